"""The Gaussian draw's arithmetic is fixed by its source, not by how a compiler
fuses it: the device header's form and the generated kernels' copy compile to
the same instructions with and without floating-point contraction, so they
agree with each other and with any build."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_26477_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _generated():
    text = open(os.path.join(CSRC, "jit.cpp")).read()
    parts = [re.search(r"static const char \*%s = R\"\((.*?)\)\";" % name, text, re.S).group(1)
             for name in ("kPrelude", "kNoisePrelude")]
    return "\n".join(parts) + ("\nextern \"C\" __global__ void draw(const u64 *s, float *o) "
                               "{ int i = __builtin_amdgcn_workitem_id_x(); o[i] = nzv(s[i], (u64)i); }\n")


SOURCES = {
    "header": ('#include "device_common.hpp"\nextern "C" __global__ void draw(const uint64_t *s, float *o) '
               '{ int i = threadIdx.x; o[i] = qaia::noise_value(s[i], (uint64_t)i); }\n'),
    "generated": None,
}


@pytest.mark.parametrize("which", list(SOURCES))
def test_draw_does_not_depend_on_contraction(tmp_path, which):
    src = tmp_path / "draw.hip"
    src.write_text(SOURCES[which] or _generated())
    code = []
    for contract in ("off", "fast"):
        out = tmp_path / (contract + ".s")
        subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-S",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=" + contract,
                        "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(out)],
                       check=True, capture_output=True)
        body = out.read_text().split("draw:", 1)[1].split(".section", 1)[0]
        lines = [line.split(";")[0].strip() for line in body.splitlines()]
        code.append([line for line in lines if line and not line.startswith(".")])
    assert any("v_cos_f32" in line or "v_sin_f32" in line or "v_log_f32" in line for line in code[0])
    assert code[0] == code[1]
