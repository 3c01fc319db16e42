"""The statistics' read-back where the order of calls or a cell's values are out
of the ordinary."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def es():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12946_amd import eselbm
    return eselbm


def _state(es, D, shape, dtype, seed=3):
    """A solver and a perturbed equilibrium in its storage type."""
    rng = np.random.default_rng(seed)
    f = oracle.init_equilibrium(1 + 1e-2 * rng.standard_normal(shape), 0.02 * rng.standard_normal((D,) + shape))
    s = es.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype)
    return s, torch.from_numpy(f).to(s.storage_dtype).cuda()


def _H(f):
    f = f.double().cpu().numpy()
    w = oracle.lattice(f.ndim - 1)[1].reshape((-1,) + (1,) * (f.ndim - 1))
    return float(np.sum(f * (np.log(f / w) - 1)))


def test_H_between_a_capture_and_its_replays(es):
    """A captured step's reset has not run: H asked for before the first replay
    is that of the registered state, not added to an earlier one; and so is
    H after every replay, asked for once and twice."""
    s, a = _state(es, 2, (20, 70), "f64")
    b = s.empty_state()
    s.set_stats(True)

    def check(state):
        for _ in range(2):
            # every term to a few roundings of a sum of some 12600 terms below 1
            assert abs(s.stats(with_H=True)["H"] - _H(state)) <= 1e-12 * abs(_H(state))

    s.step(a, b, 1, 0.1)
    check(b)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.step(b, a, 1, 0.1)
    check(a)
    for _ in range(3):
        g.replay()
        check(a)
        b.copy_(a)
    s.step(a, b, 1, 0.1)
    check(b)


def test_H_after_a_capture_on_a_new_handle(es):
    s, a = _state(es, 2, (20, 70), "f64")
    b = s.empty_state()
    s.set_stats(True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.step(a, b, 1, 0.1)
    b.copy_(a)
    assert abs(s.stats(with_H=True)["H"] - _H(b)) <= 1e-12 * abs(_H(b))


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
def test_H_of_infinite_and_huge_populations(es, dtype):
    """A population beyond every range takes the logarithm, as the others of its
    cell: inf gives inf, NaN gives NaN, and a double beyond the range of float
    its own term."""
    s, a = _state(es, 2, (6, 70), "f64")
    w = oracle.lattice(2)[1].reshape(9, 1, 1)
    if dtype != "f64":
        s = es.Solver("D2Q9", (6, 70), dtype=dtype)
        a = torch.from_numpy(a.cpu().numpy() - (w if dtype.endswith("s") else 0.0)).to(s.storage_dtype).cuda()
    b = s.empty_state()
    s.set_stats(True)
    s.step(a, b, 1, 0.1)

    def H(value):
        # H is that of the registered output as it is now
        old = b[4, 3, 33].clone()
        b[4, 3, 33] = value
        h = s.stats(with_H=True)["H"]
        b[4, 3, 33] = old
        return h

    base = H(b[4, 3, 33].clone())
    assert np.isfinite(base)
    assert H(float("inf")) == float("inf")
    assert np.isnan(H(float("nan")))
    if dtype == "f64":
        big = 1e200
        term = big * (np.log(big / w[4, 0, 0]) - 1)
        # one term, to a few roundings, beside which the others vanish
        assert abs(H(big) - term) <= 8 * 2.0 ** -52 * term


def test_H_on_both_sides_of_the_series_in_one_wave(es):
    """|z| = |f - w| / (f + w) drawn for every population: cells at the series'
    end (0.36 to its bound 0.375), beyond it, and waves of both with one
    population beyond among 26 within."""
    rng = np.random.default_rng(11)
    shape, w = (3, 5, 130), oracle.lattice(3)[1].reshape(27, 1, 1, 1)
    for dtype in ("f64", "f32"):
        s = es.Solver("D3Q27", shape, dtype=dtype)
        b = s.empty_state()
        s.set_stats(True)
        s.step(torch.from_numpy(w * np.ones((27,) + shape)).to(s.storage_dtype).cuda(), b, 1, 0.1)
        for band in ((0.36, 0.3749), (0.3751, 0.6), "mixed"):
            lo, hi = (0.30, 0.3749) if band == "mixed" else band
            z = rng.uniform(lo, hi, (27,) + shape) * rng.choice([-1.0, 1.0], (27,) + shape)
            if band == "mixed":
                # every seventh cell has one population beyond the bound
                cells = np.arange(np.prod(shape)) % 7 == 3
                z.reshape(27, -1)[rng.integers(0, 27, cells.sum()), np.flatnonzero(cells)] = 0.45
            b.copy_(torch.from_numpy(w * (1 + z) / (1 - z)))
            f = b.double().cpu().numpy()
            at = np.abs(f - w) / (f + w)
            if band == "mixed":
                beyond = (at > 0.375).any(axis=0).reshape(-1)
                assert 0 < beyond[:64].sum() < 64
            else:
                assert (at <= 0.375).all() if hi < 0.375 else (at > 0.375).all()
            terms = f * (np.log(f / w) - 1)
            # each term to a few roundings, summed in FP64
            assert abs(s.stats(with_H=True)["H"] - np.sum(terms)) <= 1e-13 * np.sum(np.abs(terms)), (dtype, band)


@pytest.mark.parametrize("mode", ["higher", "lower"])
def test_a_NaN_path_length_shows(es, mode):
    """A cell with strictly positive populations, one of them so small that its
    path length overflows to NaN, among healthy cells: alpha_max is NaN and
    alpha_min that of the others."""
    s, a = _state(es, 2, (6, 70), "f64")
    s.set_mode(mode)
    b, alpha = s.empty_state(), torch.empty((6, 70), dtype=torch.float64, device="cuda")
    a[4, 3, 33] = 1e-320  # the rest population, which does not move
    s.set_alpha_field(alpha)
    s.set_stats(True)
    s.step(a, b, 1, 0.1)
    st = s.stats()
    al = alpha.cpu().numpy()
    assert st["n_nonpos"] == 0 and np.isnan(al).sum() == 1 and np.isnan(al[3, 33])
    assert np.isnan(st["alpha_max"]) and np.isnan(st["alpha_mean"])
    assert st["alpha_min"] == np.nanmin(al)
