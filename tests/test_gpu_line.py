"""Split steps of 1D problems (section III's advection study), many sweeps in
one launch: bitwise the sweeps one by one, over line lengths around a wave, a
workgroup and the cells of a lane, both LDS layouts, every tier and degree,
sequences of several displacements, and more sweeps than one launch takes."""
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


def _both(sl, n, k, tier, nsteps, shifts, ndouble=1, adjoint=False):
    import torch
    seq = [(0, 0, torch.full((1,), s, dtype=torch.float64, device="cuda")) for s in shifts]
    plan = sl.Plan((n,), k, tier, ndouble=ndouble)
    st = _state(plan, n + k)
    out, where = [], []
    for fuse in (False, True):
        plan.set_fusion(fuse)
        a = tuple(t.clone() for t in st)
        b = tuple(torch.full_like(t, float("nan")) for t in st)
        run = plan.split_steps_adjoint if adjoint else plan.split_steps
        where.append(run(seq, nsteps, a, b))
        out.append((a, b)[where[-1]])
    torch.cuda.synchronize()
    assert where[0] == where[1] == nsteps * len(shifts) % 2
    for x, y in zip(*out):
        assert torch.equal(_bits(x), _bits(y)), (n, k, tier)
    plan.close()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 256, 257, 1000, 1025, 2049, 4096, 4097])
@pytest.mark.parametrize("k,tier", [(3, "fp64"), (2, "fp32"), (1, "bf16")])
def test_lengths(sl, n, k, tier):
    _both(sl, n, k, tier, 5, [0.37])


@pytest.mark.parametrize("tier", ["fp64", "fp32", "bf16", "fp16"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("ndouble", [0, 1, 2])
def test_tiers_and_sequences(sl, tier, k, ndouble):
    _both(sl, 70, k, tier, 3, [0.4, -2.7, 81.5], ndouble=min(ndouble, k + 1))
    _both(sl, 333, k, tier, 4, [-0.25, 0.0], ndouble=min(ndouble, k + 1))


@pytest.mark.parametrize("tier", ["fp64", "bf16"])
def test_adjoint(sl, tier):
    _both(sl, 130, 2, tier, 3, [0.4, -2.7], adjoint=True)


@pytest.mark.parametrize("nsteps,shifts", [(16385, [0.3]), (5462, [0.3, -0.1, 1.2])])
def test_several_launches(sl, nsteps, shifts):
    _both(sl, 20, 2, "fp32", nsteps, shifts)
