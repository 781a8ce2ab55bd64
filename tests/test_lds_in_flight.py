"""CPU: no kernel touches the result registers of an LDS read before the wait for it.

Fragment reads written as inline assembly are in flight when the compiler takes them as done.  Where their values are not used any more
it may put something else into their registers, which the read then overwrites.  The built library's own device code is walked over
every branch, with the queue of LDS operations that may be outstanding (they return in order)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1901_09290_amd import binding as B

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
MOST = 40  # operations that are followed; lgkmcnt counts to 15


def _registers(text):
    out = {int(n) for n in re.findall(r"\bv(\d+)\b", text)}
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return frozenset(out)


def touched_in_flight(listing):
    """listing: (address, instruction, branch target or None) of one kernel -> instructions that use a register whose read is outstanding."""
    at = {a: i for i, (a, _, _) in enumerate(listing)}
    targets = {t for _, _, t in listing if t is not None}
    found, seen, work = [], set(), [(0, ())]
    while work:
        i, queue = work.pop()
        while i < len(listing):
            address, text, target = listing[i]
            op = text.split()[0]
            if address in targets or target is not None:
                if (i, queue) in seen:
                    break
                seen.add((i, queue))
            if op == "s_endpgm":
                break
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", text)
                if m:
                    queue = queue[len(queue) - min(len(queue), int(m.group(1))):]
            else:
                reads = op.startswith("ds_") and (op.startswith(("ds_read", "ds_bpermute", "ds_permute", "ds_swizzle")) or "_rtn" in op)
                used = _registers(text.split(",", 1)[-1] if reads else text)  # (two reads into one register return in order)
                if used and any(used & r for r in queue):
                    found.append(f"{address:x}: {text}")
                if op.startswith("ds_"):
                    queue = (queue + (_registers(text.split(",")[0]) if reads else frozenset(),))[-MOST:]
            if target is not None:
                if op == "s_branch":
                    i = at[target]
                    continue
                work.append((at[target], queue))
            i += 1
    return sorted(set(found))


def _kernels(path):
    """Name and listing of every kernel of a code object that reads LDS."""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout
    for start, name, body in re.findall(r"^([0-9a-f]{16}) <(\w+)>:\n(.*?)(?=^\S|\Z)", text, re.S | re.M):
        listing = []
        for line in body.splitlines():
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(?:.*<\w+\+0x([0-9a-f]+)>)?", line)
            if m:
                branch = m.group(1).startswith(("s_branch", "s_cbranch"))
                listing.append((int(m.group(2), 16), m.group(1), int(start, 16) + int(m.group(3), 16) if branch and m.group(3) else None))
        if any(t.startswith("ds_read") for _, t, _ in listing):
            yield name, listing


def test_the_walk_sees_a_register_that_is_touched_too_early():
    def run(*lines):
        return touched_in_flight([(4 * i, *(l if isinstance(l, tuple) else (l, None))) for i, l in enumerate(lines)])
    read = ["ds_read_b64_tr_b16 v[4:5], v1", "ds_read_b64_tr_b16 v[6:7], v1 offset:512"]
    assert run(*read, "s_waitcnt lgkmcnt(1)", "v_mov_b32 v9, v4", "s_endpgm") == []
    assert len(run(*read, "s_waitcnt lgkmcnt(1)", "v_mov_b32 v9, v6", "s_endpgm")) == 1       # read too early
    assert len(run(*read, "v_and_b32 v5, 63, v0", "s_waitcnt lgkmcnt(0)", "s_endpgm")) == 1   # overwritten by the read
    assert len(run(*read, ("s_cbranch_scc0 2", 20), "s_waitcnt lgkmcnt(0)", "v_mov_b32 v9, v4", "v_mov_b32 v9, v7", "s_endpgm")) == 1  # on one path


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_no_register_is_touched_while_its_lds_read_is_in_flight(tmp_path):
    if not os.path.exists(B._SO):
        from paper_1901_09290_amd import build as hip_build
        hip_build.build()
    so = shutil.copy(B._SO, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", so], capture_output=True, check=True, cwd=tmp_path)
    objects = sorted(str(p) for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    kernels = [k for o in objects for k in _kernels(o)]
    assert {"k_wgrad_row3", "k_stem_wgrad"} <= {m.group(1) for m in (re.match(r"_ZN2pt\d+(k_\w+?)(?:I|E)", n) for n, _ in kernels) if m}
    bad = {name: found for name, listing in kernels for found in [touched_in_flight(listing)] if found}
    assert not bad, bad
