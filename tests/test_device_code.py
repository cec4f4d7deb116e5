"""Device code compiled for gfx950 and read as assembly: what cannot be told from results."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MULZ = """
#include "models.h"
__global__ void product(float w, float v, float *o) {
  *o = smc2::mulz(smc2::frcp(w), smc2::frcp(v));
}
"""


def _assembly(source, tmp_path):
    from paper_2407_17296_amd import build
    path = tmp_path / "t.hip"
    path.write_text(source)
    r = subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", str(path), "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return [ln.strip() for ln in r.stdout.splitlines() if re.match(r"\t[sv]_|\tds_|\tglobal_", ln)]


def test_zero_product_waits_for_the_transcendental_unit(tmp_path):
    """A VALU instruction must not read a transcendental result in the very next cycle: something
    else stands between the second reciprocal and the product that reads it."""
    code = _assembly(MULZ, tmp_path)
    mul = [i for i, ln in enumerate(code) if ln.startswith("v_mul_legacy_f32")]
    assert len(mul) == 1
    assert not code[mul[0] - 1].startswith("v_rcp_f32"), code
