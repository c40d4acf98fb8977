"""Fused pairs of sweeps along neighbouring dimensions d, d + 1 >= 1 whose
displacements depend on the dimensions below d alone (the split step's v1 and
v2 sweeps; section II splitting, section II-A update): bitwise the two sweeps
one by one, over column counts around a wave, extents around the rows of a
lane and of a wave, one and two shifts per wave and spread ones, every tier and
degree."""
import numpy as np
import pytest

from gpu_helpers import have_gpu
from test_gpu_strang import _bits, _state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    if not have_gpu():
        pytest.skip("no HIP device")
    import paper_1603_07008_amd as sl
    sl.lib()
    return sl


def _both(sl, ns, k, tier, d, mask, amp, ndouble=1, nsteps=1, offset=0.0, seed=1, pairs=1):
    import torch
    rng = np.random.default_rng(seed)
    n = int(np.prod([ns[e] for e in range(len(ns)) if mask >> e & 1] or [1]))
    seq = [(d + i, mask, torch.from_numpy(offset + rng.uniform(-amp, amp, n)).cuda())
           for i in range(2)]
    plan = sl.Plan(ns, k, tier, ndouble=ndouble)
    st = _state(plan, seed)
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = tuple(torch.full_like(t, float("nan")) for t in st)
        plan.timing_enable(True)
        out.append((a, b)[plan.split_steps(seq, nsteps, a, b)])
        assert plan.timing_read(-2)[0] == (2 - pairs * fuse) * nsteps
        plan.timing_enable(False)
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(_bits(x), _bits(y)), (ns, k, tier)
    plan.close()


@pytest.mark.parametrize("ns", [(48, 2, 4), (64, 3, 5), (63, 17, 49), (65, 9, 7), (100, 8, 48),
                                (192, 16, 97)])
@pytest.mark.parametrize("amp,offset", [(0.4, 0.0), (0.2, -3.5), (9.0, 0.0)])
def test_extents_and_shifts(sl, ns, amp, offset):
    for tier in ("fp32", "bf16"):
        # 65 columns leave half of two waves idle: one sweep after the other
        _both(sl, ns, 2, tier, 1, 1, amp, nsteps=2, offset=offset, pairs=int(ns[0] != 65))


@pytest.mark.parametrize("tier", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("ndouble", [0, 1])
@pytest.mark.parametrize("amp", [0.4, 7.0])
def test_tiers_and_degrees(sl, tier, k, ndouble, amp):
    _both(sl, (60, 11, 13), k, tier, 1, 1, amp, ndouble=ndouble)


@pytest.mark.parametrize("ns,d,mask", [((12, 8, 6, 7), 2, 3), ((12, 8, 6, 7), 2, 2),
                                       ((60, 9, 6, 7), 1, 1), ((4, 3, 5, 2, 6), 2, 0),
                                       ((4, 3, 5, 2, 6), 3, 0b101)])
def test_dimensions_and_masks(sl, ns, d, mask):
    pairs = int(ns != (4, 3, 5, 2, 6) or d == 3)
    _both(sl, ns, 1, "fp32", d, mask, 0.4, pairs=pairs)
    _both(sl, ns, 2, "bf16", d, mask, 3.0, pairs=pairs)


@pytest.mark.parametrize("nsteps", [1, 2, 3])
def test_result_buffer_not_asked_for(sl, nsteps):
    """With a NULL result_buffer the pairs leave the result where the separate
    sweeps do."""
    import ctypes
    import torch
    plan = sl.Plan((64, 9, 10), 2, "fp32")
    s = torch.full((64,), 0.3, dtype=torch.float64, device="cuda")
    st = _state(plan, 3)
    seq = (sl.SweepDesc * 2)(*[sl.SweepDesc(1 + i, 1, s.data_ptr()) for i in range(2)])
    out = []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = tuple(torch.empty_like(t) for t in st)
        rc = sl.lib().sldg_split_steps(plan._h, seq, 2, nsteps, *[
            ctypes.c_void_p(t.data_ptr()) for t in (*a, *b)], None)
        assert rc == 0
        out.append(a)                                 # two sweeps a step: back in buffer 0
    torch.cuda.synchronize()
    for x, y in zip(*out):
        assert torch.equal(_bits(x), _bits(y))
    plan.close()
