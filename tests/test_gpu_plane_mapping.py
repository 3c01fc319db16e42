"""Steps whose lanes run through whole planes (ragged rows on grids beyond the
smallest, and the FP64 D3Q27 step on short rows), in every variant of the step.

FP64 against the oracle, one step, within 1e-14 (a few roundings of
populations below 0.3).  The 4-byte formats against the row-mapped step, to the
bit: the state repeated along x until the row is whole blocks takes the row
mapping and has the same cells.  F16-shifted against the F32-shifted step of
the same state: its arithmetic is single precision with series cut far below
its storage, so the two agree to one FP16 rounding step of a deviation.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2203_12946_amd import workloads as W
from tests._states import three_regime_state

pytestmark = pytest.mark.gpu

TAU = 3e-3


@pytest.fixture(scope="module")
def es():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12946_amd import eselbm
    return eselbm


def _stored(f, dtype):
    """(what the solver stores, the populations it stands for)"""
    w = oracle.lattice(f.ndim - 1)[1].reshape((-1,) + (1,) * (f.ndim - 1))
    if dtype == "f64":
        return f, f
    if dtype == "f32":
        v = f.astype(np.float32)
        return v, v.astype(np.float64)
    v = (f - w).astype(np.float32)
    return v, w + v.astype(np.float64)


def _check(s, a, out, ref, alpha=None, uv=None):
    """``out`` (and the fields) = one step of ``a``: against the oracle
    (``ref()``: state, alpha) in FP64, against the row-mapped step of the
    repeated state otherwise."""
    if s.dtype_code == 0:
        f, ra = ref()
        err = float(np.max(np.abs(out.cpu().numpy() - f)))
        assert err <= 1e-14, err
        if alpha is not None:
            assert np.max(np.abs(alpha.cpu().numpy() - ra)) <= 1e-10
            r, u = oracle.moments(f)
            assert np.max(np.abs(uv.double().cpu().numpy() - np.concatenate([u, r[None]]))) <= 1e-7
        return
    n = 256 // math.gcd(256, s.nx)
    big = a.repeat((1,) * s.D + (n,))
    rows = type(s)(s.lattice, big.shape[1:], dtype={1: "f32", 3: "f32s"}[s.dtype_code], mode=s.mode)
    if s._walls is not None:
        rows.set_walls(*s._walls)
    if s._force is not None:
        rows.set_force(s._force.repeat((1,) * s.D + (n,)))
    got = rows.empty_state()
    fields = []
    if alpha is not None:
        fields = [(torch.empty(big.shape[1:], dtype=s.compute_dtype, device="cuda"), alpha), (rows.empty_velocity(), uv)]
        rows.set_alpha_field(fields[0][0])
        rows.set_velocity_field(fields[1][0])
    rows.step(big, got, 1, TAU)
    for x, y in fields:
        assert torch.equal(x[..., :s.nx], y) and torch.equal(x[..., -s.nx:], y)
    assert torch.equal(got[..., :s.nx], out) and torch.equal(got[..., -s.nx:], out)


# rows of one partial wave, of several waves and a tail, just past a block; two
# planes and one; FP64 D3Q27 rows of whole waves
@pytest.mark.parametrize("shape", [(41, 43, 44), (3, 79, 301), (3, 90, 257), (32, 16, 64), (4, 45, 192),
                                   (513, 522), (1030, 257), (831, 320)])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s"])
def test_periodic_and_walls(es, shape, dtype):
    D = len(shape)
    stored, f0 = _stored(three_regime_state(D, shape, 3), dtype)
    s = es.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype)
    a = torch.from_numpy(np.ascontiguousarray(stored)).cuda()
    b = s.empty_state()
    s._walls = None
    s.step(a, b, 1, TAU)
    ref = lambda: oracle.step(f0, 1, TAU, want_alpha=True)[:2]  # noqa: E731
    _check(s, a, b, ref)
    # the diagnostic variant: the same state to the bit, the fields, the sums
    alpha = torch.empty(shape, dtype=s.compute_dtype, device="cuda")
    uv = s.empty_velocity()
    s.set_alpha_field(alpha)
    s.set_velocity_field(uv)
    s.set_stats(True)
    c = s.empty_state()
    s.step(a, c, 1, TAU)
    st = s.stats()
    assert torch.equal(b, c) and st["n_cells"] == s.cells and st["n_nonpos"] == 0
    assert abs(st["mass"] - f0.sum()) <= 1e-6 * s.cells
    _check(s, a, c, ref, alpha, uv)
    # in place, the same bits as two lattices
    s.set_alpha_field(None)
    s.set_velocity_field(None)
    s.set_stats(False)
    d = a.clone()
    s.step(d, d, 2, TAU)
    s.step(b, c, 1, TAU)
    assert torch.equal(c, d)
    # walls on y alone, and on every axis (FP64: rows cannot be repeated there)
    lid = {(1, 1): (0.05,) + (0.01,) * (D - 1)}
    for mask in ([False, True] + [False] * (D - 2), [True] * D):
        if mask[0] and dtype != "f64":
            continue
        s._walls = (mask, lid)
        s.set_walls(*s._walls)
        s.step(a, b, 1, TAU)
        _check(s, a, b, lambda: (oracle.step_walls(f0, 1, TAU, mask, lid), None))


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("shape", [(41, 43, 44), (3, 79, 301), (513, 522)])
def test_f16(es, shape, walls):
    D = len(shape)
    w = oracle.lattice(D)[1].reshape((-1,) + (1,) * D)
    a = torch.from_numpy((three_regime_state(D, shape, 5) - w).astype(np.float16)).cuda()
    out = []
    for dtype in ("f16s", "f32s"):
        s = es.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype)
        if walls:
            s.set_walls([True] * D, {(1, 1): (0.05,) + (0.01,) * (D - 1)})
        b = s.empty_state()
        s.step(a.to(s.storage_dtype), b, 1, TAU)
        out.append(b.float())
    # one rounding step: 2^-10 of the value, 2^-24 below the normal range
    assert bool(torch.all((out[0] - out[1]).abs() <= 2.0 ** -10 * out[1].abs() + 2.0 ** -24))


@pytest.mark.parametrize("shape", [(41, 43, 44), (513, 522)])
def test_es_bgk_mirror_and_force(es, shape):
    D = len(shape)
    lat = "D2Q9" if D == 2 else "D3Q27"
    f0 = three_regime_state(D, shape, 7)
    a = torch.from_numpy(f0).cuda()
    s = es.Solver(lat, shape, dtype="f64")
    b = s.empty_state()
    s.set_prandtl(0.71)
    s.step(a, b, 1, TAU)
    _check(s, a, b, lambda: (oracle.step_esbgk(f0, 1, TAU, 0.71), None))
    s.set_prandtl(1.0)
    s.set_mode("elbm")
    s.step(a, b, 1, TAU)
    _check(s, a, b, lambda: (oracle.step(f0, 1, TAU, mode="elbm"), None))
    s = es.Solver(lat, shape, dtype="f32")
    s._walls = None
    s.set_force(torch.from_numpy(W.random_force(shape, D, amplitude=1e-4, seed=4)).float().cuda())
    a, b = a.float(), s.empty_state()
    s.step(a, b, 1, TAU)
    _check(s, a, b, None)
