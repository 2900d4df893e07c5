"""A batch that mixes systems with projectors and systems whose projectors
were never set (they hold no projection tables): every state as stepped
alone, bit for bit, and the one without projectors against the oracle."""
import sys

import numpy as np
import pytest

from oracle import ks_oracle as ko
from paper_2106_03872_amd import synth

from gpu_common import rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2106_03872_amd import ks as ksmod
    return ksmod


def _states(ks, specs, precision):
    out = []
    for k, spec in enumerate(specs):
        sysm = synth.system(spec)
        s = ks.System(spec.n, spec.L, spec.ecut, spec.norb, precision=precision)
        s.set_vloc(torch.from_numpy(sysm.vloc).cuda())
        if k != 1:
            p = sysm.proj
            s.set_projectors(p.npts, p.idx, p.beta, p.d)
        st = ks.State(s, spec.norb)
        st.upload(torch.from_numpy(synth.orbitals_box(spec)).cuda())
        out.append((sysm, s, st))
    return out


# tiles of 64 pencils (24^3) and of 32 (48^3); batches that sum the projections
# inside the x-apply pass (24 / 32, 48 / 6) and in a launch of their own
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n,norb", [(24, 32), (24, 200), (48, 6), (48, 30)])
def test_batch_with_projectors_never_set(ks, n, norb, precision):
    print(f"[case] batch, projectors never set, {n} norb {norb} precision {precision}", file=sys.stderr, flush=True)
    specs = [synth.cubic_spec(f"np{k}", n, 0.33 * n, norb + k, 3, 9100 + k) for k in range(3)]
    alone, batched = _states(ks, specs, precision), _states(ks, specs, precision)
    for _, _, st in alone:
        st.propagate(0.05, 2)
    b = ks.Batch([st for _, _, st in batched])
    b.propagate(0.05, 2)
    torch.cuda.synchronize()
    for (_, _, a), (_, _, c) in zip(alone, batched):
        assert torch.equal(a.download(), c.download())
    b.close()
    sysm, _, st = batched[1]
    spec = specs[1]
    ham = ko.Hamiltonian(ko.Grid(spec.n, spec.L, spec.ecut), sysm.vloc, [], np.zeros((0, 4)))
    ref = ko.taylor4_step(ham, synth.orbitals_box(spec)[:4], 0.05, 2)
    assert rel_err(st.download()[:4].cpu().numpy(), ref) < (1e-12 if precision == 0 else 1e-5)
    for _, s, st in alone + batched:
        st.close()
        s.close()
