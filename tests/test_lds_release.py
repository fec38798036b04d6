"""Kernels whose LDS is refilled by loads with an LDS destination behind a hand-written barrier: a wave's reads of what is
refilled must have returned when it reaches the barrier, and the compiler, which waits for a read only before its result is used, does
not see to that.  Checked in the machine code of the source: no LDS instruction may be outstanding at any barrier."""
import os
import re
import subprocess

from paper_2407_02891_amd import build as hip_build


def _kernels(text):
    """{kernel: [(line number, instruction or label)]}"""
    found, body = {}, None
    for number, line in enumerate(text.splitlines(), 1):
        if m := re.match(r"(_Z\w+):", line):
            body = found.setdefault(m[1], [])
            continue
        if line.startswith(".Lfunc_end"):
            body = None
        line = line.split(";")[0].strip()
        if body is not None and line and (not line.startswith(".") or line.endswith(":")):
            body.append((number, line))
    return found


def _outstanding(body):
    """{line of an s_barrier: most LDS instructions that may not have returned there}, over all paths.  They return in order, so a wait
    for a count of n leaves at most n (scalar loads share the counter and can only make it stricter)."""
    blocks, order = {"": []}, [""]
    for number, line in body:
        if line.endswith(":"):
            order.append(line[:-1])
            blocks[order[-1]] = []
        else:
            blocks[order[-1]].append((number, line))
    entry, at, work = {"": 0}, {}, [""]
    while work:
        block = work.pop()
        n, falls, to = entry[block], True, []
        for number, line in blocks[block]:
            op, _, rest = line.partition(" ")
            if op.startswith("ds_"):
                n = min(n + 1, 15)
            elif op == "s_waitcnt" and (m := re.search(r"lgkmcnt\((\d+)\)", rest)):
                n = min(n, int(m[1]))
            elif op == "s_barrier":
                at[number] = max(at.get(number, 0), n)
            elif op.startswith("s_cbranch"):
                to.append((rest.strip(), n))
            elif op in ("s_branch", "s_endpgm"):
                to += [(rest.strip(), n)] if op == "s_branch" else []
                falls = False
                break
        if falls and block != order[-1]:
            to.append((order[order.index(block) + 1], n))
        for target, count in to:
            if entry.get(target, -1) < count:
                entry[target] = count
                work.append(target)
    return at


def test_the_check_itself():
    def most(*lines):
        return list(_outstanding(list(enumerate(lines))).values())

    read = "ds_read_b128 v[0:3], v4"
    assert most(read, "s_waitcnt vmcnt(1)", "s_barrier") == [1]
    assert most(read, "s_waitcnt vmcnt(1) lgkmcnt(0)", "s_barrier") == [0]
    assert most(read, read, "s_waitcnt lgkmcnt(1)", "s_barrier", "s_waitcnt lgkmcnt(0)", "s_barrier") == [1, 0]
    # around a loop, and past a branch that skips the wait
    assert most(".LBB0_1:", "s_barrier", "s_waitcnt lgkmcnt(0)", read, "s_cbranch_scc1 .LBB0_1", "s_endpgm") == [1]
    assert most(read, "s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", ".LBB0_1:", "s_barrier", "s_endpgm") == [1]


def test_many_vector_kernels_read_before_a_refill(tmp_path):
    out = tmp_path / "wide.s"
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + [
        "--cuda-device-only", "-S", os.path.join(hip_build.CSRC, "bcq_wide.hip"), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    kernels = {k: _outstanding(body) for k, body in _kernels(out.read_text()).items() if "bcq_wide" in k}
    assert len(kernels) == 50 and all(len(at) == 7 for at in kernels.values())
    bad = {k: at for k, at in kernels.items() if any(at.values())}
    assert not bad, bad
