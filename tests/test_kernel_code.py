"""What the compiled kernels have to hold by construction, read from the gfx950 code of the built library (CPU only).

A barrier orders LDS accesses of different waves only if each wave has waited for its own before it: an access that is
merely issued may still execute behind another wave's write on the far side.  Nothing that runs shows such a missing wait
reliably, so it is looked for in the code: on every path to every s_barrier, no LDS access may be open."""
import re
import shutil
import subprocess

import pytest

from paper_2410_17043_amd import _lib

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
LANE_EXCHANGE = ("ds_bpermute", "ds_permute", "ds_swizzle")        # through the LDS crossbar, but no memory


def open_lds_accesses_at_barriers(code):
    """code: [(offset, instruction, operands, branch target offset or None)] of one kernel.  Returns the offsets of the
    barriers that some path reaches with an LDS access open.  LDS instructions complete in order, so what can be open
    behind lgkmcnt(n) are the n newest; a state is the kinds of the open ones, oldest first."""
    at = {off: i for i, (off, _, _, _) in enumerate(code)}
    seen = [set() for _ in code]
    bad = set()
    work = [(0, ())]
    while work:
        i, state = work.pop()
        while i < len(code) and state not in seen[i]:
            seen[i].add(state)
            off, op, args, target = code[i]
            if op.startswith("ds_"):
                state = (state + (not op.startswith(LANE_EXCHANGE),))[-15:]
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                if m or args.strip() == "0":
                    n = int(m.group(1)) if m else 0
                    state = state[len(state) - n:] if n < len(state) else state
            if not any(state):
                state = ()                                         # only memory accesses matter: keeps the states few
            if op == "s_barrier" and state:
                bad.add(off)
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if target is not None:
                if op == "s_branch":
                    i = at[target]
                    continue
                work.append((at[target], state))
            i += 1
    return sorted(bad)


def disassemble(path):
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--mcpu=gfx950", str(path)], check=True, capture_output=True, text=True).stdout
    kernels, code, base = {}, None, 0
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]{16}) <(.+)>:$", line)
        if m:
            base, code = int(m.group(1), 16), kernels.setdefault(m.group(2), [])
            continue
        m = re.match(r"^\t(\S+)(?: (.*?))?\s*// ([0-9A-F]+):(.*)$", line)
        if m and code is not None:
            op, target = m.group(1), None
            if op == "s_branch" or op.startswith("s_cbranch"):
                t = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>\s*$", m.group(4))
                target = int(t.group(1) or "0", 16)
            code.append((int(m.group(3), 16) - base, op, m.group(2) or "", target))
    return kernels


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    d = tmp_path_factory.mktemp("code")
    shutil.copy(_lib.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(d.glob("lib.so.*gfx950")):
        out.update(disassemble(f))
    return out


def test_the_search_sees_an_open_access_and_the_wait_that_closes_it():
    read, barrier, end = (0, "ds_read_b128", "v[0:3], v4", None), (8, "s_barrier", "", None), (12, "s_endpgm", "", None)
    assert open_lds_accesses_at_barriers([read, barrier, end]) == [8]
    for wait, bad in (("vmcnt(4)", [8]), ("lgkmcnt(1)", [8]), ("lgkmcnt(0)", []), ("vmcnt(4) lgkmcnt(0)", [])):
        assert open_lds_accesses_at_barriers([read, (4, "s_waitcnt", wait, None), barrier, end]) == bad
    # round a loop: the access behind the barrier is open when the branch comes back to it
    loop = [(0, "s_barrier", "", None), (4, "ds_write_b64", "v0, v[2:3]", None), (8, "s_cbranch_scc1", "", 0), end]
    assert open_lds_accesses_at_barriers(loop) == [0]
    assert open_lds_accesses_at_barriers([(0, "ds_bpermute_b32", "v0, v1, v2", None), barrier, end]) == []


def test_no_lds_access_is_open_at_a_barrier(kernels):
    barriers = {name: sum(op == "s_barrier" for _, op, _, _ in code) for name, code in kernels.items()}
    assert sum(barriers.values()) > 100 and any("gemm_bf16_kernel" in n for n, b in barriers.items() if b)   # the code was found and read
    found = {name: [hex(o) for o in open_lds_accesses_at_barriers(code)] for name, code in kernels.items() if barriers[name]}
    assert {n: b for n, b in found.items() if b} == {}
