"""The autotuner times the launches that a step makes: where a step's plane
analyses go on to the next synthesis, one synthesis launch per candidate (its
first H psi) against three analyses.  A child process tunes with the HIP
runtime's kernel log on; the launches are counted there."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
from paper_2106_03872_amd import ks, synth
import torch
s = ks.system_from_synth(synth.system(synth.cubic_spec("tf", {n}, {L}, 6, 2, 9600)), precision={prec})
s.autotune(6)
torch.cuda.synchronize()
print("tuned")
"""


@pytest.mark.parametrize("n,h,precision,syntheses", [(24, 0.33, 0, 1), (24, 0.33, 1, 1), (48, 0.6, 0, 3)])
def test_tuner_times_the_form_of_a_step(n, h, precision, syntheses):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    print(f"[case] tuner form {n} spacing {h} precision {precision}", file=sys.stderr, flush=True)
    env = dict(os.environ, AMD_LOG_LEVEL="3", AMD_LOG_MASK="128", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CHILD.format(n=n, L=h * n, prec=precision)], env=env, cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "tuned" in r.stdout, r.stderr[-2000:]
    launched = [line for line in r.stderr.splitlines() if "ShaderName" in line]
    if not launched:
        pytest.skip("the HIP runtime logs no kernel names here")
    inv = sum("plane_inv_kernel" in line for line in launched)
    fwd = sum("plane_fwd_kernel" in line for line in launched)
    assert inv > 0 and 3 * inv == syntheses * fwd
