"""Projection rows of a lane: few and many atoms on one grid (slots of fewer
rows than a group of four, and tiles whose lanes hold more than the sixteen rows
that stay in registers), one to four projectors per atom, tiles of 16, 32 and 64
pencils.  H psi against the FP64 oracle at 1e-12 (mixed precision 1e-5)."""
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


@pytest.mark.parametrize("n,natoms", [((24, 24, 24), 1), ((24, 24, 24), 20), ((32, 20, 20), 9), ((48, 24, 24), 24),
                                      ((120, 16, 16), 20)])
@pytest.mark.parametrize("nproj", [1, 3, 4])
def test_projection_rows(ks, n, natoms, nproj):
    print(f"[case] projection rows {n} {natoms} {nproj}", file=sys.stderr, flush=True)
    spec = synth.Spec(name="pr", n=n, L=tuple(0.33 * m for m in n), ecut=10.0, norb=5, natoms=natoms,
                      seed=9000 + n[0] + natoms)
    sysm = synth.system(spec)
    sysm.proj.beta = np.ascontiguousarray(sysm.proj.beta[:, :nproj])
    sysm.proj.d = np.ascontiguousarray(sysm.proj.d[:, :nproj])
    c = orbitals_device(spec)
    ref = ko.ham_apply(oracle_ham(sysm), c.cpu().numpy())
    for precision, tol in ((ks.KS_FP64, 1e-12), (ks.KS_MIXED, 1e-5)):
        s = ks.system_from_synth(sysm, precision=precision)
        assert rel_err(s.ham_apply(c).cpu().numpy(), ref) < tol
        s.close()
