"""The FP8 MFMAs compile to the unscaled encoding (CPU; hipcc cross-compiles
gfx950 assembly of this repository's own sources).

The kernels call the scaled builtin with both E8M0 scale operands 0, which
the compiler turns into the unscaled v_mfma_f32_{16x16x128,32x32x64}_f8f6f4
(no block scales; the fp32 scales are applied to the results).  If the
scaled form were emitted with those operands, every product would be scaled
by 2^-254; this test fails at build time instead of on the GPU."""
import concurrent.futures as cf
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_10493_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
SOURCES = ["ffn_prefill.hip", "ffn_prefill_wide.hip", "ffn_decode.hip", "ffn_decode_combine.hip"]


def _asm(src, tmp):
    out = os.path.join(tmp, src + ".s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, src), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    with open(out) as f:
        return f.read()


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_fp8_mfmas_are_unscaled(tmp_path):
    with cf.ThreadPoolExecutor(len(SOURCES)) as ex:
        asm = dict(zip(SOURCES, ex.map(lambda s: _asm(s, str(tmp_path)), SOURCES)))
    for src, text in asm.items():
        scaled = re.findall(r"v_mfma_scale_\w+", text)
        plain = re.findall(r"v_mfma_f32_(?:16x16x128|32x32x64)_f8f6f4", text)
        assert not scaled, f"{src}: scaled MFMA encoding emitted ({len(scaled)})"
        assert plain, f"{src}: no FP8 MFMA found"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("src", ["ffn_prefill_wide.hip", "router.hip"])
def test_asynchronous_loads_share_no_registers_with_the_compiler(src, tmp_path):
    """The global -> LDS loads are inline assembly that writes m0, which a clobber list cannot name (m0 is a
    reserved register): the compiler itself must use it nowhere in these files.  Nor does it insert the five wait
    states that a vector memory instruction needs after a VALU instruction wrote its scalar base."""
    code = [line.split(";")[0].strip() for line in _asm(src, str(tmp_path)).splitlines()]
    code = [c for c in code if c and not c.startswith(".") and not c.endswith(":")]
    loads = [i for i, c in enumerate(code) if c.startswith("global_load_lds")]
    assert loads
    for i in loads:
        assert re.match(r"s_mov_b32 m0, s\d+$", code[i - 2]) and code[i - 1] == "s_nop 0", code[i - 2:i + 1]
    assert sum(bool(re.search(r"\bm0\b", c)) for c in code) == len(loads)
    for i in loads:
        base = re.search(r"s\[(\d+):(\d+)\]", code[i])
        states, j = 0, i - 1
        while base and states < 5 and j >= 0:
            w = re.match(r"v_read(?:first)?lane_b32 s(\d+)", code[j])
            assert not w or not int(base[1]) <= int(w[1]) <= int(base[2]), code[j:i + 1]
            nop = re.match(r"s_nop (\d+)", code[j])
            states += 1 + (int(nop[1]) if nop else 0)
            j -= 1
