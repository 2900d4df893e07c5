"""Which steps run the next plane synthesis inside the plane analysis, and
that they give the same either way.

* FP64 planes of 60, 72 and 80 points: launches of more than 2048 blocks keep
  the two launches (four syntheses a step instead of one a call); the first
  orbitals then equal, bit for bit, those of a state of few orbitals.
* Spheres whose coefficients do not fit the y-batch (72 points in FP64 at a
  spacing of 0.5 bohr, 48 at 0.6, 40 in complex64 at 0.6) keep the two
  launches; 48 in complex64 at 0.6 has the room.  Three steps against the FP64
  oracle."""
import sys

import numpy as np
import pytest

from oracle import ks_oracle as ko
from paper_2106_03872_amd import synth

from gpu_common import oracle_ham, orbitals_device, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2106_03872_amd import ks as ksmod
    return ksmod


def _steps(ks, s, c, nsteps):
    """orbitals after nsteps of one call, and the launches of plane_inv"""
    st = ks.State(s, c.shape[0])
    st.upload(c)
    s.set_kernel_timing(True)
    st.propagate(0.04, nsteps)
    torch.cuda.synchronize()
    n = s.kernel_times()["plane_inv"][1]
    s.set_kernel_timing(False)
    out = st.download()
    st.close()
    return out, n


@pytest.mark.parametrize("n1,chained", [(60, False), (64, True), (72, False), (80, False)])
def test_large_fp64_launches(ks, n1, chained):
    print(f"[case] plane next {n1}", file=sys.stderr, flush=True)
    few = 5
    spec = synth.Spec(name=f"pn{n1}", n=(8, n1, n1), L=(3.2, 0.31 * n1, 0.31 * n1), ecut=10.0, norb=few, natoms=1,
                      seed=9400 + n1)
    sysm = synth.system(spec)
    c = orbitals_device(spec)
    planes = ks.system_from_synth(sysm).info()["nplanes"]
    repeat = 2048 // (few * planes) + 1
    s = ks.system_from_synth(sysm, max_norb=few * repeat)
    a, n_few = _steps(ks, s, c, 2)
    assert n_few == 1
    b, n_many = _steps(ks, s, c.repeat(repeat, 1, 1, 1), 2)
    assert n_many == (1 if chained else 8)
    assert bool((b.reshape((repeat,) + tuple(a.shape)) == a[None]).all())
    assert rel_err(a.cpu().numpy(), ko.taylor4_step(oracle_ham(sysm), c.cpu().numpy(), 0.04, 2)) < 1e-12
    s.close()


@pytest.mark.parametrize("n1,h,precision,launches", [(72, 0.5, 0, 12), (48, 0.6, 0, 12), (48, 0.6, 1, 1), (40, 0.6, 1, 12)])
def test_wide_spheres(ks, n1, h, precision, launches):
    print(f"[case] plane next, wide sphere {n1} spacing {h} precision {precision}", file=sys.stderr, flush=True)
    spec = synth.Spec(name=f"pw{n1}", n=(8, n1, n1), L=(3.2, h * n1, h * n1), ecut=10.0, norb=5, natoms=1, seed=9500 + n1)
    sysm = synth.system(spec)
    c = orbitals_device(spec)
    s = ks.system_from_synth(sysm, precision=precision)
    got, n = _steps(ks, s, c, 3)
    assert n == launches
    ref = ko.taylor4_step(oracle_ham(sysm), c.cpu().numpy(), 0.04, 3)
    assert rel_err(got.cpu().numpy(), ref) < (1e-12 if precision == 0 else 1e-5)
    s.close()
