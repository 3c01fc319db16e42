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
