"""The step kernels' passes over the directions (compile checks, host only): a
collision cannot be written on a pass that does not form its weights."""
import os
import subprocess

import pytest

from paper_1904_00866_amd import build as B

PROBE = '''
#include "elbm_step_impl.hpp"
using namespace elbm;
__global__ void probe(const Site<2, StoreF32, double>* v, const SiteDev<2, StoreF32Dev>* w, double* o) {
  double s = 0.0;
  %s
  *o = s;
}
'''
ALPHA = "[&](double x, double fe) { s += x * fe; }"
COLLISION = "[&](int, double invW, double, double fe, double g) { s += invW * (fe - g); }"
SHORT = "[&](int, double invW, double fe, double g) { s += invW * (fe - g); }"


def _compiles(tmp_path, body):
    src = tmp_path / "probe.hip"
    src.write_text(PROBE % body)
    cmd = [B.hipcc(), *B.flags(), "--cuda-device-only", "-fsyntax-only", str(src)]
    return subprocess.run(cmd, capture_output=True, text=True, cwd=os.path.dirname(B.LIB))


def test_passes_that_exist(tmp_path):
    r = _compiles(tmp_path, f"v->sweep<true>({ALPHA}); v->sweep<false>({ALPHA}); "
                            f"w->sweep<true>({ALPHA}); v->sweep_collision({SHORT});")
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("body", [f"v->sweep<true>({COLLISION});", f"w->sweep<true>({COLLISION});",
                                  f"v->each<true>({COLLISION});"])
def test_no_collision_on_a_pass_without_weights(tmp_path, body):
    assert _compiles(tmp_path, body).returncode != 0
