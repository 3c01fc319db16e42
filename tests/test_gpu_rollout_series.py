"""The native sequences of a rollout (include/eselbm_rollout.h): argument errors
of any of their calls come before the first is made, and a rollout through
them equals one through single calls."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPE = (6, 70)


@pytest.fixture(scope="module")
def es():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12946_amd import eselbm
    return eselbm


def _solver(es, dtype="f32"):
    s = es.Solver("D2Q9", SHAPE, dtype=dtype)
    f = s.init_equilibrium(torch.ones(SHAPE, dtype=torch.float64, device="cuda"),
                           torch.full((2,) + SHAPE, 0.01, dtype=torch.float64, device="cuda"))
    return s, f


@pytest.mark.parametrize("bad", ["own_input", "null_state", "overlap", "null_velocity"])
def test_step_series_checks_every_call_first(es, bad):
    s, f = _solver(es)
    both = torch.full((2, 9) + SHAPE, 7.0, device="cuda")
    outs, uvs = [both[0], both[1], s.empty_state()], [s.empty_velocity().fill_(7.0) for _ in range(3)]
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    ptr = [t.data_ptr() for t in outs]
    uvp = [t.data_ptr() for t in uvs]
    if bad == "own_input":
        ptr[2] = ptr[1]
    elif bad == "null_state":
        ptr[2] = None
    elif bad == "overlap":
        ptr[2] = ptr[1] + 4
    else:
        uvp[2] = None
    field = s.empty_velocity().fill_(7.0)
    s.set_velocity_field(field)
    arr = ctypes.c_void_p * 3
    status = es.lib.eselbm_rollout_steps(s._h, f.data_ptr(), arr(*ptr), arr(*uvp), 3, 0.1, loss.data_ptr(), 1.0,
                                         es._stream())
    torch.cuda.synchronize()
    assert status == 1
    assert float(loss) == 0.0
    assert all(bool((t == 7.0).all()) for t in [both, field] + uvs)
    # the registered field is the one before the refused call
    s.step(f, outs[0], 1, 0.1)
    assert bool((field != 7.0).all())


def test_step_series_refuses_a_loss_it_cannot_take(es):
    s, f = _solver(es, "f16s")
    outs, uvs = [s.empty_state().fill_(7.0)], [s.empty_velocity()]
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    with pytest.raises(es.EselbmError):
        s.step_series(f, outs, 0.1, uvs, loss, 1.0)
    assert bool((outs[0] == 7.0).all())


@pytest.mark.parametrize("bad", ["null_state", "aliased_velocity"])
def test_adjoint_series_checks_every_call_first(es, bad):
    s, f = _solver(es)
    lam, other = s.empty_adjoint().fill_(1.0), s.empty_adjoint().fill_(7.0)
    uv = s.empty_velocity().zero_()
    states, uvs = [f.data_ptr()] * 3, [uv.data_ptr()] * 3
    if bad == "null_state":
        states[2] = None
    else:
        uvs[2] = other.data_ptr()  # the third step's result goes into it
    arr = ctypes.c_void_p * 3
    status = es.lib.eselbm_rollout_adjoints(s._h, arr(*states), arr(*uvs), 3, 1.0, lam.data_ptr(), other.data_ptr(), 0.1,
                                            None, es._stream())
    torch.cuda.synchronize()
    assert status == 1
    assert bool((lam == 1.0).all()) and bool((other == 7.0).all())


class OneCallAtATime:
    """A solver without the native sequences: the rollout's Python loops."""

    def __init__(self, s):
        self._s = s

    def __getattr__(self, name):
        if name in ("step_series", "adjoint_series"):
            raise AttributeError(name)
        return getattr(self._s, name)


@pytest.mark.parametrize("nsteps,ckpt,keep", [(7, 3, 1), (6, 3, 2), (5, 1, 1), (4, 9, 1), (9, 2, None)])
@pytest.mark.parametrize("D,dtype,force,diss", [
    (2, "f32", False, None), (2, "f32", False, 1e-3), (2, "f64", False, 1e-3), (2, "f32s", False, 1e-3),
    (3, "f32", True, 1e-3), (3, "f32", True, None), (3, "f64", False, None)])
def test_native_sequences_equal_single_calls(es, D, dtype, force, diss, nsteps, ckpt, keep):
    """State, loss and gradients to the bit: the same launches in the same order."""
    from paper_2203_12946_amd.adjoint import Rollout
    shape = (12, 70) if D == 2 else (4, 6, 66)
    g = torch.Generator(device="cuda").manual_seed(5)
    s = es.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype)
    rho = 1 + 1e-2 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.02 * torch.randn((D,) + shape, generator=g, device="cuda", dtype=torch.float64)
    f0 = s.init_equilibrium(rho, u)
    lam = torch.randn(f0.shape, generator=g, device="cuda", dtype=torch.float64).to(s.compute_dtype)
    F = 1e-5 * torch.randn((D,) + shape, generator=g, device="cuda") if force else None
    if force:
        s.set_force(F)
    out = []
    for solver in (s, OneCallAtATime(s)):
        ro = Rollout(solver, 0.02, nsteps, ckpt, diss_weight=diss, keep_segments=keep)
        loss = None if diss is None else torch.zeros(1, dtype=torch.float64, device="cuda")
        fg = torch.zeros_like(F) if force else None
        fN = ro.forward(f0, loss)
        grad = ro.backward(lam, diss_grad=0.7 if diss else 0.0, force_grad=fg)
        again = ro.backward(lam, diss_grad=0.7 if diss else 0.0)  # with every segment recomputed
        out.append([t.clone() for t in (fN, grad, again, loss, fg) if t is not None])
    assert all(torch.equal(a, b) for a, b in zip(*out))
