"""The x-apply pass that sums the projections itself (few orbitals) against
the separate sum (many): the same three orbitals alone and repeated 201 times
give bit-identical H psi, which for the three equals the oracle's at 1e-12
(mixed precision 1e-5).  Grids on which an atom spans fewer and more than
eight x-tiles, with one and with four projectors per atom."""
import sys

import numpy as np
import pytest

from oracle import ks_oracle as ko
from paper_2106_03872_amd import synth

from gpu_common import oracle_ham, orbitals_device, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

REPEAT = 201    # 603 orbitals: past the 6 MB of partial sums on both grids


@pytest.fixture(scope="module")
def ks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2106_03872_amd import ks as ksmod
    return ksmod


@pytest.mark.parametrize("n,L,natoms", [((24, 24, 24), (8.0, 8.0, 8.0), 5), ((20, 40, 40), (6.6, 13.2, 13.2), 4)])
@pytest.mark.parametrize("nproj", [1, 4])
def test_x_apply_sums_projections(ks, n, L, natoms, nproj):
    print(f"[case] xsums {n} nproj {nproj}", file=sys.stderr, flush=True)
    spec = synth.Spec(name="xs", n=n, L=L, ecut=10.0, norb=3, natoms=natoms, seed=8500 + n[1])
    sysm = synth.system(spec)
    sysm.proj.beta = np.ascontiguousarray(sysm.proj.beta[:, :nproj])
    sysm.proj.d = np.ascontiguousarray(sysm.proj.d[:, :nproj])
    c = orbitals_device(spec)
    ref = ko.ham_apply(oracle_ham(sysm), c.cpu().numpy())
    many = c.repeat(REPEAT, 1, 1, 1)
    for precision, tol in ((ks.KS_FP64, 1e-12), (ks.KS_MIXED, 1e-5)):
        s = ks.system_from_synth(sysm, max_norb=3 * REPEAT, precision=precision)
        few = s.ham_apply(c)
        assert rel_err(few.cpu().numpy(), ref) < tol
        got = s.ham_apply(many).reshape((REPEAT,) + tuple(few.shape))
        assert bool((got == few[None]).all())
        s.close()
