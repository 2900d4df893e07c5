"""Which launches sum the projections inside the x-apply pass (no launch of
the separate sum), and that H psi is bit-identical either way: two orbitals
against the same two repeated past the line, for every n0, within the band and
past it, where an atom spans up to 17 tiles (more than one trip of eight of the
sum); the line of 6 MB of partial sums with blocks to spare; the launches that
never do (complex64 past 32 points, the other tile shapes).  The two orbitals
also against the FP64 oracle at 1e-12 (complex64 1e-5)."""
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


def _apply(s, c):
    """H psi and whether the projections were summed in a launch of their own"""
    s.set_kernel_timing(True)
    h = s.ham_apply(c)
    torch.cuda.synchronize()
    n = s.kernel_times()["proj_reduce"][1]
    s.set_kernel_timing(False)
    return h, n > 0


def _limit(n0, half, precision):
    if n0 <= 32:
        return 2048 if n0 < 32 or precision or half else 768
    if precision:
        return 0
    return (1792 if n0 <= 48 else 1024 if n0 == 64 else 768) if half else 768


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n0,h0", [(n, 0.31) for n in (16, 20, 24, 32, 40, 48, 60, 64, 72, 80, 96, 120, 128)]
                         + [(n, 0.42) for n in (24, 32, 40, 48, 64, 80)])
def test_sums_inside_and_apart(ks, n0, h0, precision):
    print(f"[case] sums rule {n0} spacing {h0} precision {precision}", file=sys.stderr, flush=True)
    spec = synth.Spec(name=f"sr{n0}", n=(n0, 24, 24), L=(h0 * n0, 7.5, 7.5), ecut=10.0, norb=2, natoms=2, seed=9700 + n0)
    sysm = synth.system(spec)
    tiles = 9 if n0 <= 32 else 18
    limit = _limit(n0, h0 < 0.4, precision)
    repeat = (limit // tiles) // 2 + 1
    s = ks.system_from_synth(sysm, max_norb=2 * repeat, precision=precision)
    info = s.info()
    assert info["x_half"] == (h0 < 0.4)
    if n0 > 32:
        assert 2 * 8 < info["nslots"] <= 2 * 17   # an atom spans more than eight tiles
    c = orbitals_device(spec)
    few, apart_few = _apply(s, c)
    many, apart_many = _apply(s, c.repeat(repeat, 1, 1, 1))
    assert (apart_few, apart_many) == (limit == 0, True)
    assert bool((many.reshape((repeat,) + tuple(few.shape)) == few[None]).all())
    ref = ko.ham_apply(oracle_ham(sysm), c.cpu().numpy())
    assert rel_err(few.cpu().numpy(), ref) < (1e-12 if precision == 0 else 1e-5)
    s.close()


def test_six_megabytes_of_partial_sums(ks):
    print("[case] sums rule, 6 MB", file=sys.stderr, flush=True)
    spec = synth.cubic_spec("sm", 32, 10.0, 2, 24, 9801)
    sysm = synth.system(spec)
    s = ks.system_from_synth(sysm, max_norb=128)
    info = s.info()
    # about slots^2 / atoms values of 16 bytes per projector and orbital, 16 tiles
    per_orbital = info["nslots"] ** 2 / spec.natoms * 4 * 16
    assert 32 * per_orbital < 0.9 * (6 << 20) and 128 * per_orbital > 1.1 * (6 << 20) and 128 * 16 <= 2048
    c = orbitals_device(spec)
    few, apart_few = _apply(s, c.repeat(16, 1, 1, 1))
    many, apart_many = _apply(s, c.repeat(64, 1, 1, 1))
    assert (apart_few, apart_many) == (False, True)
    assert torch.equal(few[:2], many[126:])
    s.close()


@pytest.mark.parametrize("shape", [1, 2, 3])
def test_other_shapes_sum_apart(ks, shape):
    print(f"[case] sums rule, shape {shape}", file=sys.stderr, flush=True)
    spec = synth.Spec(name="ss", n=(96, 12, 12), L=(30.0, 4.8, 4.8), ecut=10.0, norb=2, natoms=1, seed=9900)
    sysm = synth.system(spec)
    s = ks.system_from_synth(sysm)
    c = orbitals_device(spec)
    s.set_tuning(8, 8, x_shape=shape)
    h, apart = _apply(s, c)
    assert apart
    assert rel_err(h.cpu().numpy(), ko.ham_apply(oracle_ham(sysm), c.cpu().numpy())) < 1e-12
    s.close()
