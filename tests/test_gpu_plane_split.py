"""The plane passes' work split (threads, y- and z-batches, orbitals taken
together) for every plane size: seven orbitals, so that the last iteration of
a block holds fewer orbitals than it can take, on a sphere inside the band
|m| < n/4 and on a wider one whose columns exceed the z-batch, with orbital
groups of 1, 2 and 64 per block.  H psi against the FP64 oracle at 1e-12
(mixed precision 1e-5) and bit-identical across the groups."""
import sys

import numpy as np
import pytest

from oracle import ks_oracle as ko
from paper_2106_03872_amd import synth

from gpu_common import oracle_ham, orbitals_device, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [8, 12, 16, 20, 24, 32, 40, 48, 60, 64, 72, 80, 96, 120, 128]
WIDE_MAX = 80     # a wide sphere of larger FP64 planes exceeds the 160 KB of LDS


@pytest.fixture(scope="module")
def ks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2106_03872_amd import ks as ksmod
    return ksmod


@pytest.mark.parametrize("n1,h", [(n, 0.31) for n in SIZES] + [(n, 0.42) for n in SIZES if n <= WIDE_MAX])
def test_plane_split_parity(ks, n1, h):
    print(f"[case] plane split {n1} h={h}", file=sys.stderr, flush=True)
    L1 = max(h * n1, 4.8)
    spec = synth.Spec(name=f"ps{n1}", n=(16, n1, n1), L=(6.4, L1, L1), ecut=10.0, norb=7, natoms=1, seed=8300 + n1)
    sysm = synth.system(spec)
    ham = oracle_ham(sysm)
    c = orbitals_device(spec)
    ref = ko.ham_apply(ham, c.cpu().numpy())
    for precision, tol in ((ks.KS_FP64, 1e-12), (ks.KS_MIXED, 1e-5)):
        s = ks.system_from_synth(sysm, precision=precision)
        first = None
        for group in (1, 2, 64):
            s.set_tuning(8, group)
            got = s.ham_apply(c).cpu().numpy()
            assert rel_err(got, ref) < tol, (precision, group)
            assert first is None or np.array_equal(got, first), (precision, group)
            first = got
        s.close()
