"""Inline assembly whose operands come from other lanes (DPP, row_newbcast): the register it reads must have been written at
least two instructions before, and the compiler keeps no such distance for it.  Checked in the machine code of the source."""
import os
import re
import subprocess

from paper_2407_02891_amd import build as hip_build


def _too_close(text):
    """Places where a row_newbcast operand was written less than two wait states before (waits for memory do not count)."""
    bad, seen, recent = [], 0, []  # recent: registers written 1, 2 wait states ago
    for number, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        if op == "s_waitcnt":
            continue
        if op == "s_nop":
            recent = ([None] * (int(rest, 0) + 1) + recent)[:2]
            continue
        operands = [o.strip() for o in rest.split(",")]
        if "row_newbcast" in rest:
            seen += 1
            if operands[1].split()[0] in [w for ws in recent if ws for w in ws]:
                bad.append((number, line))
        written = []
        if op.startswith("v_") and operands and (m := re.match(r"v(\d+)$|v\[(\d+):(\d+)\]$", operands[0])):
            lo, hi = (int(m[1]), int(m[1])) if m[1] else (int(m[2]), int(m[3]))
            written = ["v%d" % r for r in range(lo, hi + 1)]
        recent = ([written] + recent)[:2]
    return bad, seen


def test_the_check_itself():
    text = "v_sub_f32 v1, v2, v3\nv_fma_f32 v4, v5, v6, v7\ns_waitcnt lgkmcnt(0)\nv_fmac_f32_dpp v8, v1, v9 row_newbcast:3\n"
    assert len(_too_close(text)[0]) == 1
    assert not _too_close(text.replace("s_waitcnt lgkmcnt(0)", "v_mov_b32 v10, v11"))[0]
    assert not _too_close(text.replace("s_waitcnt lgkmcnt(0)", "s_nop 0"))[0]
    assert len(_too_close("v_pk_mov_b32 v[0:1], v[2:3], v[4:5]\nv_mov_b32_dpp v8, v1 row_newbcast:3\n")[0]) == 1


def test_quantiser_keeps_the_distance(tmp_path):
    out = tmp_path / "quant.s"
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + [
        "--cuda-device-only", "-S", os.path.join(hip_build.CSRC, "bcq_quant.hip"), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    bad, seen = _too_close(out.read_text())
    assert seen > 100
    assert not bad, bad[:10]
