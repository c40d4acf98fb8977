"""Which calls the differentiable split steps issue: every step of the forward
pass and its transpose runs once, whatever the checkpoint interval (a stub
plan in place of the device)."""
import pytest
import torch

from paper_1603_07008_amd import autograd as AG


class StubPlan:
    tier = "fp64"

    def __init__(self):
        self.forward = self.adjoint = 0

    def empty_state(self):
        return torch.zeros(4, dtype=torch.float64), torch.zeros(2, 4, dtype=torch.float64)

    def _steps(self, nsteps, src, dst):
        assert isinstance(nsteps, int) and nsteps > 0
        for a, b in zip(src, dst):
            b.copy_(a + nsteps)
        return 1

    def split_steps(self, seq, nsteps, src, dst):
        self.forward += nsteps
        return self._steps(nsteps, src, dst)

    def split_steps_adjoint(self, seq, nsteps, src, dst):
        self.adjoint += nsteps
        return self._steps(nsteps, src, dst)


@pytest.mark.parametrize("every", [None, 0, 1, 3, 4, 10, 100, -1, -3, 4.0, 2.5])
@pytest.mark.parametrize("nsteps", [0, 1, 10])
@pytest.mark.parametrize("frozen", [False, True])
def test_every_step_runs_once(every, nsteps, frozen):
    plan = StubPlan()
    m = torch.zeros(4, dtype=torch.float64, requires_grad=True)
    h = torch.zeros(2, 4, dtype=torch.float64, requires_grad=True)
    fn = (lambda state: []) if frozen else None
    out, _ = AG.split_steps(plan, [], nsteps, m, h, checkpoint_every=every, frozen_shifts_fn=fn)
    assert plan.forward == nsteps and torch.all(out == nsteps)
    out.sum().backward()
    assert plan.adjoint == nsteps


@pytest.mark.parametrize("every,starts", [(None, [0]), (4, [0, 4, 8]), (-4, [0, 4, 8]),
                                          (4.0, [0, 4, 8]), (2.5, [0, 5])])
def test_calls_start_at_the_checkpoints(every, starts):
    runs = AG._runs(10, every, False)
    assert [n for n, _ in runs] == starts
    assert sum(c for _, c in runs) == 10
