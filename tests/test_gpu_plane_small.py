"""Plane blocks that take several orbitals at once and the small launches that
take one per block instead: seven orbitals (one each) against the same seven
repeated past every line, so that the last block of a group has a remainder,
bit for bit, and against the oracle; H psi from and to boxes and a step of a
state, in the band and past it."""
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


@pytest.mark.parametrize("h", [0.31, 0.42])
@pytest.mark.parametrize("n1", [8, 12, 20, 32, 40])
def test_one_or_several_orbitals_per_block(ks, n1, h):
    print(f"[case] plane small {n1} spacing {h}", file=sys.stderr, flush=True)
    L1 = max(h * n1, 4.8)
    spec = synth.Spec(name=f"pl{n1}", n=(16, n1, n1), L=(6.4, L1, L1), ecut=10.0, norb=7, natoms=1, seed=9650 + n1)
    sysm = synth.system(spec)
    ham = oracle_ham(sysm)
    c = orbitals_device(spec)
    ref, ref_step = ko.ham_apply(ham, c.cpu().numpy()), ko.taylor4_step(ham, c.cpu().numpy(), 0.04)
    repeat = 61     # 427 orbitals, odd: no multiple of 2, 3, 4 or 8
    for precision, tol in ((ks.KS_FP64, 1e-12), (ks.KS_MIXED, 1e-5)):
        s = ks.system_from_synth(sysm, max_norb=7 * repeat, precision=precision)
        assert 7 * s.info()["nplanes"] <= 256 and 7 * repeat * s.info()["nplanes"] > 1024
        for group in (8, 64):
            s.set_tuning(8, group)
            few = s.ham_apply(c)
            assert rel_err(few.cpu().numpy(), ref) < tol
            many = s.ham_apply(c.repeat(repeat, 1, 1, 1)).reshape((repeat,) + tuple(few.shape))
            assert bool((many == few[None]).all())
            out = []
            for x in (c, c.repeat(repeat, 1, 1, 1)):
                st = ks.State(s, x.shape[0])
                st.upload(x)
                st.propagate(0.04, 1)
                out.append(st.download())
                st.close()
            assert rel_err(out[0].cpu().numpy(), ref_step) < tol
            assert bool((out[1].reshape((repeat,) + tuple(few.shape)) == out[0][None]).all())
        s.close()
