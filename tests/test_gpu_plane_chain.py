"""The plane analysis that goes on to the next plane synthesis (Taylor steps):
three steps of one call, with densities and norms, against the FP64 oracle at
1e-12 (mixed precision 1e-5, densities and norms likewise) and against three
calls of one step each, whose first synthesis is a launch of its own, at 1e-13
(mixed 1e-6).  Every plane size, so that G = 1 .. 8 orbitals are taken together
with a remainder of seven; 128 has no room for the coefficients and keeps the
two launches.  With an atom (the density inside the projection pass) and
without."""
import sys

import numpy as np
import pytest

from oracle import ks_oracle as ko
from paper_2106_03872_amd import synth

from gpu_common import oracle_ham, orbitals_device, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [8, 12, 16, 20, 24, 32, 40, 48, 60, 64, 72, 80, 96, 120, 128]


@pytest.fixture(scope="module")
def ks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2106_03872_amd import ks as ksmod
    return ksmod


@pytest.mark.parametrize("natoms", [0, 1])
@pytest.mark.parametrize("n1", SIZES)
def test_steps_chained(ks, n1, natoms):
    print(f"[case] plane chain {n1} natoms={natoms}", file=sys.stderr, flush=True)
    L1 = max(0.31 * n1, 4.8)
    spec = synth.Spec(name=f"pc{n1}", n=(16, n1, n1), L=(6.4, L1, L1), ecut=10.0, norb=7, natoms=1, seed=8600 + n1)
    sysm = synth.system(spec)
    ham = oracle_ham(sysm)
    if not natoms:
        ham = ko.Hamiltonian(ham.grid, sysm.vloc)
    c = orbitals_device(spec)
    occ = torch.full((spec.norb,), 2.0, dtype=torch.float64, device="cuda")
    ref, dens = c.cpu().numpy(), []
    for _ in range(3):
        ref = ko.taylor4_step(ham, ref, 0.04)
        dens.append(ko.density(ham, ref, occ.cpu().numpy()))
    for precision, tol, tol_calls in ((ks.KS_FP64, 1e-12, 1e-13), (ks.KS_MIXED, 1e-5, 1e-6)):
        s = ks.system_from_synth(sysm, precision=precision)
        if not natoms:
            s.set_projectors(np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros((0, 4)), np.zeros((0, 4)))
        out = []
        for calls in (1, 3):
            st = ks.State(s, spec.norb)
            st.upload(c)
            rho = torch.zeros((3,) + spec.n, dtype=torch.float64, device="cuda")
            nrm = torch.zeros((3, spec.norb), dtype=torch.float64, device="cuda")
            k = 3 // calls
            for i in range(calls):
                st.propagate(0.04, k, occ, rho[i * k:(i + 1) * k], nrm[i * k:(i + 1) * k])
            out.append([t.cpu().numpy() for t in (st.download(), rho, nrm)])
            st.close()
        (a, rho, nrm), split = out
        assert rel_err(a, ref) < tol
        for i in range(3):
            assert rel_err(rho[i], dens[i]) < tol
        assert np.max(np.abs(nrm[2] - ko.norms(ham, ref))) < tol
        for x, y in zip((a, rho, nrm), split):
            assert rel_err(x, y) < tol_calls
        s.close()
