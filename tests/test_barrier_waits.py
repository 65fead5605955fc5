"""Every work-group barrier of the device code waits for the wave's own LDS
operations first: a store still on its way when the wave passes the barrier may
land after another wave's access behind it. The compiler inserts that wait for
__syncthreads, and has dropped it at a loop's head whose preceding stores came
over the back edge only (the dense accumulator of the final chunks then lost
columns). Checked on the disassembly of the built library, over all paths."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_22866_amd.build import LIB

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
INSN = re.compile(r"^\s+(\S.*?)\s*//\s*([0-9A-F]+):")
BRANCH = re.compile(r"s_c?branch\w*\s+(\d+)$")


def _kernels(tmp_path):
    """(name, [(address, instruction)]) of every function of the library's gfx950 code."""
    lib = shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    for f in sorted(os.listdir(tmp_path)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        name, body = None, []
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(.*)>:", line)
            if head:
                if body:
                    yield name, body
                name, body = head.group(1), []
            m = INSN.match(line)
            if m:
                body.append((int(m.group(2), 16), m.group(1)))
        if body:
            yield name, body


def unwaited_barriers(body):
    """Barriers that some path reaches with LDS operations outstanding, as
    {address: instructions}. (Cross-lane moves that go through the LDS unit touch
    no LDS memory.)"""
    at = {a: i for i, (a, _) in enumerate(body)}
    pend = [None] * len(body)
    pend[0] = frozenset()
    work, bad = [0], {}
    while work:
        i = work.pop()
        a, s = body[i]
        p = pend[i]
        if s.startswith("s_waitcnt"):
            m = re.search(r"lgkmcnt\((\d+)\)", s)
            if (m and m.group(1) == "0") or s == "s_waitcnt 0":
                p = frozenset()
        elif re.match(r"(ds_(?!bpermute|permute|swizzle)|flat_)", s):
            p = p | {s.split()[0]}
        elif s.startswith("s_barrier") and p:
            bad[a] = bad.get(a, frozenset()) | p
        m = BRANCH.match(s)
        succ = [] if s.startswith(("s_branch", "s_endpgm", "s_setpc")) else [i + 1]
        if m:
            d = int(m.group(1))
            succ.append(at[a + 4 + 4 * (d - 65536 if d >= 32768 else d)])
        for j in succ:
            if j < len(body) and (pend[j] is None or not p <= pend[j]):
                pend[j] = p | (pend[j] or frozenset())
                work.append(j)
    return bad


def test_checker_sees_a_store_over_the_back_edge():
    head = [(0, "s_waitcnt lgkmcnt(0)"), (4, "s_barrier"), (8, "ds_read_b32 v1, v2"), (12, "s_waitcnt lgkmcnt(0)"),
            (16, "ds_write_b32 v1, v2")]
    loop_to_barrier = [(20, "s_cbranch_vccnz 65531"), (24, "s_endpgm")]  # 20 + 4 - 4 * 5 = 4
    loop_to_wait = [(20, "s_cbranch_vccnz 65530"), (24, "s_endpgm")]
    assert unwaited_barriers(head + loop_to_barrier) == {4: frozenset({"ds_write_b32"})}
    assert unwaited_barriers(head + loop_to_wait) == {}


def test_barriers_wait_for_lds(tmp_path):
    if not (os.path.exists(OBJDUMP) and os.path.exists(LIB)):
        pytest.skip("needs llvm-objdump and the built library")
    n_barriers, bad = 0, {}
    for name, body in _kernels(tmp_path):
        n_barriers += sum(s.startswith("s_barrier") for _, s in body)
        found = unwaited_barriers(body)
        if found:
            bad[name] = found
    assert n_barriers > 100
    assert not bad, bad
