"""A solver class that redefines the calls a rollout makes is called for each of
them (adjoint.Rollout, on the CPU): the native sequences of Solver stand only
for Solver's own methods."""
import pytest
import torch

from paper_2203_12946_amd.adjoint import Rollout
from paper_2203_12946_amd.eselbm import Solver


class CountingSolver(Solver):
    """Solver's interface without a device; counts the calls of a rollout."""
    D, Q, cells = 3, 1, 4
    compute_dtype = storage_dtype = torch.float32

    def __init__(self):
        self.calls = []

    def empty_state(self):
        return torch.zeros(4)

    empty_velocity = empty_adjoint = empty_seed = empty_state

    def set_velocity_field(self, uv):
        pass

    def step(self, f, out, n, tau):
        self.calls.append("step")
        out.copy_(f + 1)

    def dissipation_loss_uv(self, uv, loss=None, weight=None, seed=None, force_grad=None):
        self.calls.append("loss")

    def adjoint_step(self, f_n, lam, out, tau, force_grad=None, seed_next=None):
        self.calls.append("adjoint")
        out.copy_(lam)

    def adjoint_step_diss(self, f_n, lam, uv_next, weight, out, tau, force_grad=None):
        self.calls.append("adjoint_diss")
        out.copy_(lam)

    def _refuse(self, *a, **k):
        raise AssertionError("a native sequence in place of the class's own methods")

    step_series = adjoint_series = _refuse


@pytest.mark.parametrize("diss", [None, 1e-3])
def test_an_overriding_class_is_called_for_every_step(diss):
    s = CountingSolver()
    ro = Rollout(s, 0.1, 7, 3, diss_weight=diss)
    fN = ro.forward(torch.zeros(4), None if diss is None else torch.zeros(1, dtype=torch.float64))
    assert int(fN[0]) == 7
    assert s.calls.count("step") == 7 and s.calls.count("loss") == (7 if diss else 0)
    s.calls.clear()
    ro.backward(torch.ones(4), diss_grad=1.0 if diss else 0.0)
    assert s.calls.count("adjoint_diss" if diss else "adjoint") == 7
    assert s.calls.count("step") == 4  # two segments of three recomputed from their checkpoints


def test_an_instance_method_counts_too():
    """A step replaced on one object (a wrapper that logs, for instance)."""
    class Plain(CountingSolver):
        step = Solver.step
        set_velocity_field = Solver.set_velocity_field
        dissipation_loss_uv = Solver.dissipation_loss_uv

    s = Plain()
    with pytest.raises(AssertionError):
        Rollout(s, 0.1, 2, 1).forward(torch.zeros(4))
    s.step = lambda f, out, n, tau: s.calls.append("step")
    Rollout(s, 0.1, 2, 1).forward(torch.zeros(4))
    assert s.calls == ["step", "step"]
