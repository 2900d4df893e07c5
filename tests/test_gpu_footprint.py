"""ks_plan_footprint against what a system takes from its pool: the projection
tables (the growth at ks_system_set_projectors, for every tile shape of the
grid) and the system with a resident state as a whole, for passes of one
orbital and of eight, where the tables are not hidden by the pass buffers."""
import sys

import numpy as np
import pytest

from paper_2106_03872_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ks():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2106_03872_amd import ks as ksmod
    return ksmod


@pytest.mark.parametrize("chunk", [1, 8])
@pytest.mark.parametrize("n,natoms,nproj", [(16, 1, 4), (24, 5, 4), (48, 32, 1), (64, 64, 4), (96, 1, 4), (96, 128, 4),
                                            (96, 300, 4)])
def test_footprint_covers_the_projection_tables(ks, n, natoms, nproj, chunk):
    print(f"[case] footprint {n} atoms {natoms} nproj {nproj} chunk {chunk}", file=sys.stderr, flush=True)
    spec = synth.cubic_spec("fp", n, 0.3125 * n, chunk, natoms, 9300 + n)
    p = synth.system(spec).proj
    beta, d = np.ascontiguousarray(p.beta[:, :nproj]), np.ascontiguousarray(p.d[:, :nproj])
    npoints = int(p.npts.sum())
    plan = lambda pts: ks.plan_footprint(spec.n, spec.L, spec.ecut, chunk, pts, nproj, chunk=chunk)
    for shape in range(4):
        pool = ks.Pool(1 << 30)
        s = ks.System(spec.n, spec.L, spec.ecut, chunk, pool=pool, chunk=chunk)
        if shape and n != 96:
            with pytest.raises(ks.KSError):
                s.set_tuning(8, 8, x_shape=shape)
        else:
            s.set_tuning(8, 8, x_shape=shape)
            before = pool.usage()[0]
            s.set_projectors(p.npts, p.idx, beta, d)
            assert pool.usage()[0] - before <= plan(npoints) - plan(0)
            st = ks.State(s, chunk)
            assert pool.usage()[0] <= plan(npoints)
            st.close()
        s.close()
        pool.close()
