"""The tile kernels refill an LDS buffer behind a workgroup barrier, so a wave's reads of that buffer must
have returned before it arrives: s_barrier itself waits for no LDS read.  Checked on the instructions of
the built library, over every path to every barrier (needs no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_12529_amd import _lib

KERNELS = ("gemm_bf16_mid", "gemm_bf16_pp", "gemm_fp8_pp")


def objdump():
    for d in ("/opt/rocm/llvm/bin", "/opt/rocm/bin"):
        p = os.path.join(d, "llvm-objdump")
        if os.path.exists(p):
            return p
    return shutil.which("llvm-objdump")


def instructions(text):
    """Listing of one kernel -> [(address, mnemonic, operands, branch target or None)]."""
    base, out = None, []
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <", line)
        if head:
            base = int(head.group(1), 16)
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):.*?(?:<[^>+]*(?:\+0x([0-9a-f]+))?>)?$", line)
        if m:
            branch = m.group(1) == "s_branch" or m.group(1).startswith("s_cbranch")
            target = base + int(m.group(4) or "0", 16) if branch else None
            out.append((int(m.group(3), 16), m.group(1), m.group(2), target))
    return out


def reads_outstanding_at_barriers(ins):
    """Largest number of LDS instructions that may be outstanding at each s_barrier, over all paths.
    They complete in order, so lgkmcnt(n) leaves at most n of them."""
    index = {a: i for i, (a, *_) in enumerate(ins)}
    state = [None] * len(ins)
    work, barriers = [(0, 0)], {}
    while work:
        i, n = work.pop()
        while i < len(ins) and (state[i] is None or state[i] < n):
            state[i] = n
            addr, op, args, target = ins[i]
            if op.startswith("ds_"):
                n = min(n + 1, 64)   # bounded, so a loop without a wait ends the walk too
            elif op == "s_waitcnt":
                lg = re.search(r"lgkmcnt\((\d+)\)", args)
                n = min(n, int(lg.group(1))) if lg else n
            elif op == "s_barrier":
                barriers[addr] = max(barriers.get(addr, 0), n)
            elif target is not None:
                work.append((index[target], n))
                if op == "s_branch":
                    break
            elif op == "s_endpgm":
                break
            i += 1
    return barriers


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    tool = objdump()
    if tool is None:
        pytest.skip("llvm-objdump not found")
    d = tmp_path_factory.mktemp("isa")
    lib = shutil.copy(_lib.LIB_PATH, d)
    subprocess.run([tool, "--offloading", lib], check=True, capture_output=True, cwd=d)
    found = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([tool, "-d", os.path.join(d, f)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            name = re.match(r"[0-9a-f]+ <(\S+)>", part)
            if name and any(k in name.group(1) for k in KERNELS):
                found[name.group(1)] = part
    return found


def test_the_walk_counts_reads_over_loops():
    listing = """0000000000000100 <k>:
\tds_read_b128 v[0:3], v5    // 000000000100: 00
\ts_waitcnt lgkmcnt(0)       // 000000000104: 00
\ts_barrier                  // 000000000108: 00
\tds_read_b128 v[0:3], v5    // 00000000010C: 00
\ts_cbranch_scc1 65533       // 000000000110: 00 <k+0x8>
\ts_endpgm                   // 000000000114: 00
"""
    assert reads_outstanding_at_barriers(instructions(listing)) == {0x108: 64}
    waited = listing.replace("ds_read_b128 v[0:3], v5    // 00000000010C", "s_waitcnt lgkmcnt(0)  // 00000000010C")
    assert reads_outstanding_at_barriers(instructions(waited)) == {0x108: 0}


@pytest.mark.parametrize("kernel", KERNELS)
def test_lds_reads_return_before_the_barrier_that_frees_their_buffer(kernels, kernel):
    ours = {n: t for n, t in kernels.items() if kernel in n}
    assert ours, f"no {kernel} in the library"
    for name, text in ours.items():
        at = reads_outstanding_at_barriers(instructions(text))
        assert len(at) >= 2, name
        assert max(at.values()) == 0, f"{name}: LDS reads outstanding at a barrier: { {hex(a): n for a, n in at.items() if n} }"
