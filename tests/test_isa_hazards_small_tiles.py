"""The 16x16 MFMAs of the decoder kernels: no result is read too early (CPU only).

The same check as for the 32x32 MFMAs.  A v_mfma_f32_16x16x4_f32 takes 8 passes
(32 cycles), so a VALU read of its result needs 12 wait states after it.
"""
import os
import re
import subprocess

import pytest

import test_isa_hazards as H


def scan16(asm):
    """As scan(), with the 16x16 results pending beside each other: a chain of
    MFMAs on several accumulators leaves each with its own distance."""
    bad = []
    for km in re.finditer(r"^(\S+):[^\n]*\n", asm, re.M):
        if km.group(1).startswith("."):
            continue
        end = asm.find(".Lfunc_end", km.end())
        if end < 0:
            continue
        pend = []            # [destination registers, wait states so far]
        for line in asm[km.end():end].split("\n"):
            t = line.split(";")[0].strip()
            if not t:
                continue
            if t.startswith("."):
                if re.match(r"^\.LBB\w*:", t):
                    pend = []
                continue
            ins = t.split()[0]
            ops = [o.strip() for o in t[len(ins):].split(",")]
            step = int(ops[0], 0) + 1 if ins == "s_nop" else 1
            if ins.startswith("v_") and not ins.startswith("v_mfma"):
                src = set()
                for o in ops[1:]:
                    src |= H._vregs(o)
                bad += [(km.group(1), t, p[1]) for p in pend if src & p[0] and p[1] < 12]
            for p in pend:
                p[1] += step
            pend = [p for p in pend if p[1] < 12]
            if ins.startswith("v_mfma_f32_16x16"):
                pend.append([H._vregs(ops[0]), 0])
    return bad


def test_scan_flags_an_early_read_and_accepts_a_drained_one():
    head = ("k:\n\tv_mfma_f32_16x16x4_f32 v[2:5], v18, v19, v[2:5]\n"
            "\tv_mfma_f32_16x16x4_f32 v[6:9], v18, v19, v[6:9]\n")
    early = head + "\ts_nop 7\n\tv_max_f32_e32 v3, 0, v2\n.Lfunc_end0:\n"
    later = head + "\ts_nop 7\n\tv_max_f32_e32 v30, 0, v29\n\tv_max_f32_e32 v3, 0, v6\n.Lfunc_end0:\n"
    drained = head + "\ts_nop 7\n\ts_nop 7\n\tv_max_f32_e32 v3, 0, v6\n.Lfunc_end0:\n"
    other = head + "\tv_max_f32_e32 v3, 0, v20\n.Lfunc_end0:\n"
    assert [b[2] for b in scan16(early)] == [9]
    assert [b[2] for b in scan16(later)] == [9]
    assert scan16(drained) == [] and scan16(other) == []


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_decoder_kernels_read_no_16x16_result_early(tmp_path):
    import importlib.util
    spec = importlib.util.spec_from_file_location("dist_build",
                                                  os.path.join(H.ROOT, "paper_1911_13225_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    flags = [f for f in b.FLAGS if f != "-fPIC"]
    out = str(tmp_path / "mlp.s")
    r = subprocess.run([b.HIPCC, *flags, "--cuda-device-only", "-S", H.SRC, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    asm = open(out).read()
    assert asm.count("v_mfma_f32_16x16x4") > 100
    bad = scan16(asm)
    assert not bad, bad[:5]
