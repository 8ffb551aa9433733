"""Host-side check of the compiled gfx950 code for two hazards around the tile copies (LDS-DMA loads issued as
assembly text, which the compiler's hazard recogniser does not look into):
  * a vector-memory instruction must not read a scalar register within five wait states of a vector-ALU write to it
    (v_readlane restoring a spilled scalar, v_readfirstlane, v_cmp): the copy would fetch from a stale address;
  * an LDS-DMA instruction needs one wait state after a scalar write of M0, five after a vector-ALU one.
The kernels' sources are compiled to assembly here (no GPU needed).  What is asked of every copy does not depend on the
path that leads to it: each scalar register that it reads, M0 among them, has been written by a scalar instruction in
the same stretch of straight-line code, after any vector-ALU write.  (A scalar result needs no wait states, and a scalar
instruction that reads a vector-written register is interlocked.)  The scanner itself is pinned on hand-written snippets
that contain the mistakes."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2605_14877_amd import build as hb

SOURCES_WITH_COPIES = ["attend.hip", "attend_short.hip", "attend_f32.hip", "attend_f32_split.hip", "calibrate.hip", "probe.hip"]
NO_SCALAR_RESULT = ("s_cmp", "s_cbranch", "s_branch", "s_waitcnt", "s_nop", "s_barrier", "s_endpgm", "s_setprio",
                    "s_sleep", "s_bitcmp", "s_setpc", "s_inst_prefetch", "s_sethalt")


def _sregs(tok):
    tok = tok.strip(",")
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", tok)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", tok)
    if m:
        return {int(m.group(1))}
    if tok in ("vcc", "m0"):
        return {tok}
    return set()


def scan(asm_text):
    """Returns (number of copy instructions seen, list of hazard descriptions)."""
    scalar_age = {}  # scalar register -> wait states since a scalar instruction of this stretch wrote it
    copies, hazards = 0, []
    for no, raw in enumerate(asm_text.split("\n"), 1):
        line = raw.split(";")[0].strip()
        if line.endswith(":"):
            scalar_age = {}  # reached from elsewhere too
            continue
        if not line or line.startswith("."):
            continue
        toks = line.split()
        op, args = toks[0], toks[1:]
        if op.startswith("global_load_lds") or (op.startswith("buffer_load") and "lds" in args):
            copies += 1
            base = {"m0"}
            for a in args:
                base |= _sregs(a)
            for r in sorted(base, key=str):
                name = r if r == "m0" else f"s{r}"
                if r not in scalar_age:
                    hazards.append(f"line {no}: {line}: {name} not written by a scalar instruction on the way here")
                elif r == "m0" and scalar_age[r] < 1:
                    hazards.append(f"line {no}: {line}: m0 written by the instruction right before")
        step = int(args[0]) + 1 if op == "s_nop" else 1
        scalar_age = {r: a + step for r, a in scalar_age.items()}
        if args and op.startswith("s_") and not op.startswith(NO_SCALAR_RESULT):
            loaded = op.startswith(("s_load", "s_buffer_load"))  # arrives later, and not from the scalar ALU
            for r in _sregs(args[0]):
                if loaded:
                    scalar_age.pop(r, None)
                else:
                    scalar_age[r] = 0
        elif op.startswith("v_"):
            for a in args[:2]:  # a scalar result stands first, or second (carry out, v_div_scale)
                for r in _sregs(a):
                    if a == args[0] or op.startswith(("v_add_co", "v_sub_co", "v_subrev_co", "v_addc_co", "v_subb_co",
                                                      "v_subbrev_co", "v_div_scale", "v_mad_u64", "v_mad_i64")):
                        scalar_age.pop(r, None)
    return copies, hazards


def test_scanner_sees_planted_mistakes():
    stale = """
    s_mov_b32 m0, s11
    v_readlane_b32 s6, v255, 4
    v_readlane_b32 s7, v255, 5
    s_nop 0
    global_load_lds_dwordx4 v213, s[6:7]
    """
    n, hz = scan(stale)
    assert n == 1 and len(hz) == 2 and "s6" in hz[0] and "s7" in hz[1]
    fixed = stale.replace("s_nop 0", "s_mov_b64 s[8:9], s[6:7]").replace("v213, s[6:7]", "v213, s[8:9]")
    assert scan(fixed) == (1, [])
    # the copy of a loop's first block: its registers were written in front of the loop, or at its end by the vector ALU
    for before in ("s_mov_b64 s[8:9], s[6:7]\n    .LBB0_1:", ".LBB0_1:\n    v_readlane_b32 s9, v1, 0"):
        n, hz = scan(f"""
    {before}
    s_mov_b32 m0, s11
    s_nop 0
    global_load_lds_dwordx4 v213, s[8:9]
    """)
        assert n == 1 and len(hz) == 2 and "s8" in hz[0] and "s9" in hz[1]
    for m0, word in (("s_mov_b32 m0, s11", "right before"), ("v_readfirstlane_b32 m0, v3\n    s_nop 0", "not written"),
                     ("s_mov_b32 m0, s11\n    .LBB0_2:\n    s_nop 0\n    s_add_u32 s4, s2, 0x1000\n    s_addc_u32 s5, s3, 0",
                      "not written")):
        n, hz = scan(f"""
    s_add_u32 s4, s2, 0x1000
    s_addc_u32 s5, s3, 0
    {m0}
    global_load_lds_dwordx4 v2, s[4:5]
    """)
        assert n == 1 and len(hz) == 1 and "m0" in hz[0] and word in hz[0], hz
    checked = """
    s_mov_b64 s[8:9], s[4:5]
    s_mov_b64 s[10:11], s[6:7]
    s_movk_i32 s12, 0x1000
    s_add_u32 m0, s3, 0x400
    s_nop 0
    buffer_load_dwordx4 v2, s[8:11], s12 offen lds
    """
    assert scan(checked) == (1, [])
    for reg, mistake in (("s9", "s_mov_b64 s[8:9], s[4:5]"), ("s12", "s_movk_i32 s12, 0x1000")):
        n, hz = scan(checked.replace(mistake, f"v_readlane_b32 {reg}, v255, 4"))
        assert n == 1 and hz and any(reg in h for h in hz)


def test_no_tile_copy_depends_on_scalars_from_the_vector_alu():
    with tempfile.TemporaryDirectory() as tmp:
        procs = []
        for src in SOURCES_WITH_COPIES:
            out = os.path.join(tmp, src + ".s")
            cmd = ["hipcc", *hb.HIP_FLAGS, "-S", "--cuda-device-only", os.path.join(hb.CSRC, src), "-o", out]
            procs.append((src, out, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        total = 0
        for src, out, pr in procs:
            log, _ = pr.communicate()
            assert pr.returncode == 0, (src, log[-2000:])
            with open(out) as f:
                copies, hazards = scan(f.read())
            assert copies > 0, src
            assert not hazards, (src, hazards[:8])
            total += copies
        print(f"{total} copy instructions checked")


def test_fp32_kernels_reduce_over_lane_groups_in_registers():
    # At the end of every block of keys: an exchange through LDS takes a round trip, and lane numbers to go with it.
    with tempfile.TemporaryDirectory() as tmp:
        for src, kernel in (("calibrate.hip", "calibrate_f32_kernel"), ("attend_f32.hip", "attend_f32_kernel")):
            out = os.path.join(tmp, src + ".s")
            subprocess.run(["hipcc", *hb.HIP_FLAGS, "-S", "--cuda-device-only", os.path.join(hb.CSRC, src), "-o", out],
                           check=True, capture_output=True)
            with open(out) as f:
                bodies = re.findall(r"^(_ZN\S*%s\S*):[^\n]*\n(.*?)^\.Lfunc_end" % kernel, f.read(), re.M | re.S)
            assert bodies, src
            for name, body in bodies:
                assert "v_permlane16_swap_b32" in body and "ds_bpermute" not in body, name
