"""The density's orbital groups of small launches (few orbitals on a small grid:
more groups than one per eight orbitals, their partial densities in U): densities
of two steps and of the boxes against the FP64 oracle at 1e-12 (mixed precision
1e-5), for orbital counts around the group sizes and for passes of three
orbitals, where U holds few partial densities."""
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


@pytest.mark.parametrize("n,norb", [((24, 24, 24), k) for k in (1, 2, 8, 9, 17)] + [((8, 12, 12), 5), ((48, 40, 40), 19)])
@pytest.mark.parametrize("chunk", [0, 3])
def test_density_groups(ks, n, norb, chunk):
    print(f"[case] density groups {n} {norb} chunk {chunk}", file=sys.stderr, flush=True)
    spec = synth.Spec(name="dg", n=n, L=tuple(max(0.33 * m, 4.8) for m in n), ecut=10.0, norb=norb, natoms=2,
                      seed=8800 + n[0] + norb)
    sysm = synth.system(spec)
    ham = oracle_ham(sysm)
    c = orbitals_device(spec)
    occ_np = np.linspace(0.3, 2.0, norb)
    occ = torch.from_numpy(occ_np).cuda()
    r0 = ko.density(ham, c.cpu().numpy(), occ_np)
    r1 = ko.taylor4_step(ham, c.cpu().numpy(), 0.04)
    r2 = ko.taylor4_step(ham, r1, 0.04)
    refs = [ko.density(ham, r, occ_np) for r in (r1, r2)]
    for precision, tol in ((ks.KS_FP64, 1e-12), (ks.KS_MIXED, 1e-5)):
        s = ks.system_from_synth(sysm, precision=precision, chunk=chunk)
        assert rel_err(s.density(c, occ).cpu().numpy()[None], r0[None]) < tol
        st = ks.State(s, norb)
        st.upload(c)
        rho = torch.empty((2,) + n, dtype=torch.float64, device="cuda")
        st.propagate(0.04, 2, occ, rho)
        for i in range(2):
            assert rel_err(rho[i].cpu().numpy()[None], refs[i][None]) < tol
        st.close()
        s.close()
