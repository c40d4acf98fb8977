"""Guard bands around the buffers of the fused passes: X V X, column pairs (the
fused pass and the two line sweeps, the second in place), 1D steps and a batch's
passes write every cell of their output, nothing beside it and nothing of their
input, at smooth and at spread shifts."""
import numpy as np
import pytest

from gpu_helpers import have_gpu
from test_gpu_guard import run_guarded, state_inputs, state_specs
from test_gpu_passes import _uniform
from test_gpu_strang import _seq

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sl():
    if not have_gpu():
        pytest.skip("no HIP device")
    import paper_1603_07008_amd as sl
    sl.lib()
    return sl


def _guarded(sl, plan, seq, nsteps=1, adjoint=False):
    run = plan.split_steps_adjoint if adjoint else plan.split_steps

    def op(ins, outs):
        assert run(seq, nsteps, tuple(ins), tuple(outs)) == 1
    run_guarded(lambda: list(state_inputs(sl, plan, 3)), state_specs(sl, plan), op)
    plan.close()


@pytest.mark.parametrize("tier,k", [("fp64", 1), ("fp32", 2), ("bf16", 3), ("fp16", 1)])
@pytest.mark.parametrize("ns", [(1, 7), (63, 5), (130, 41), (21, 6, 5)])
@pytest.mark.parametrize("amp", [0.4, 20.0])
def test_x_v_x(sl, tier, k, ns, amp):
    seq = _seq(ns, 2, 1, 1.5 * ns[0], amp, 2)
    seq[2] = seq[0]                       # (one table: three do not fit a grid of 1 x 7)
    for adjoint in (False, True):
        _guarded(sl, sl.Plan(ns, k, tier), seq, adjoint=adjoint)


@pytest.mark.parametrize("tier,k", [("fp64", 2), ("fp32", 1), ("bf16", 2), ("fp16", 3)])
@pytest.mark.parametrize("ns", [(60, 11, 13), (112, 151, 101), (304, 51, 59)])
@pytest.mark.parametrize("amp", [0.4, 1.5, 30.0])
def test_column_pair(sl, tier, k, ns, amp):
    _guarded(sl, sl.Plan(ns, k, tier),
             [(1, 1, _uniform(ns[0], amp, 1)), (2, 1, _uniform(ns[0], amp, 2))])


@pytest.mark.parametrize("tier,k,n", [("fp64", 2, 64), ("fp64", 3, 3000), ("bf16", 1, 4095)])
def test_line(sl, tier, k, n):
    _guarded(sl, sl.Plan((n,), k, tier), [(0, 0, _uniform(1, 5.0, 1))], nsteps=3)


@pytest.mark.parametrize("rows", [0, 4, 16])
def test_batch(sl, rows):
    import torch
    from paper_1603_07008_amd.batch import Batch
    grids = [((33, 40), 1), ((64, 65), 2), ((130, 31), 3), ((5, 2), 1)]
    plans = [sl.Plan(ns, k, "bf16") for ns, k in grids]
    seqs = [_seq(ns, 2, 1, 2.0, 3.0, i) for i, (ns, _) in enumerate(grids)]
    b = Batch([g[0] for g in grids], [g[1] for g in grids], "bf16")

    def op(ins, outs):
        pairs = [[(x[2 * i], x[2 * i + 1]) for i in range(len(grids))] for x in (ins, outs)]
        b.bind(*pairs)
        b.set_sequence([(seqs[0][q][0], [(s[q][1], s[q][2]) for s in seqs]) for q in range(3)])
        b.set_pass_tuning(0, rows)
        assert b.run(1) == 1
    run_guarded(lambda: [t for i, p in enumerate(plans) for t in state_inputs(sl, p, i)],
                [s for p in plans for s in state_specs(sl, p)], op)
    b.close()
