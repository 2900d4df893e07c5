"""Orthonormalisation and subspace eigenproblem at orbital counts around their
block sizes (32-column Cholesky blocks, 16-index Jacobi blocks): the Cholesky
orthonormalised orbitals against the oracle's within the first-order bound of
the overlap's condition, orthonormal to 1e-12; one steepest-descent iteration's
Ritz values within 1e-10 of the oracle's and its orbitals orthonormal to 1e-11."""
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


def _overlap_error(c):
    m = c.cpu().numpy().reshape(c.shape[0], -1)
    return np.abs(m.conj() @ m.T - np.eye(c.shape[0])).max()


@pytest.mark.parametrize("norb", [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 65])
def test_subspace_block_edges(ks, norb):
    print(f"[case] subspace {norb}", file=sys.stderr, flush=True)
    spec = synth.Spec(name="ss", n=(24, 24, 24), L=(8.0, 8.0, 8.0), ecut=10.0, norb=norb, natoms=2, seed=8900 + norb)
    sysm = synth.system(spec)
    ham = oracle_ham(sysm)
    gs = ks.system_from_synth(sysm)
    c = orbitals_device(spec)
    cn = c.cpu().numpy()
    sv = np.linalg.svd(np.where(ham.grid.chi, cn, 0).reshape(norb, -1), compute_uv=False)
    cond = (sv[0] / sv[-1]) ** 2
    gs.orthonormalize(c)
    assert rel_err(c.cpu().numpy(), ko.orthonormalize(ham, cn)) < max(1e-12, 1e-14 * cond * np.sqrt(norb))
    assert _overlap_error(c) < 1e-12
    st = ks.State(gs, norb)
    st.upload(c)
    eig, _ = st.eigensolve(1)
    _, e, _ = ko.sd_iteration(ham, c.cpu().numpy())
    assert np.abs(eig[0].cpu().numpy() - e).max() < 1e-10 * np.abs(e).max()
    assert _overlap_error(st.download()) < 1e-11
    st.close()
    gs.close()
