"""The H pass (FP64 sum over the state) against NumPy's logarithms, summed
pairwise (a sequential sum of the largest case's 10^7 equal terms is itself off
by 2e-13), on states whose populations lie well inside, at and beyond the range
of its series, asked for once and twice.  Tolerance 1e-13 of
sum |f (log(f/w) - 1)|: every term is evaluated to a few FP64 roundings and
summed in FP64."""
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


# |z| = |f - w| / (f + w): the series ends at 0.375; (0.1, 0.5) mixes both in a wave
@pytest.mark.parametrize("zs", [(1e-4, 1e-2), (0.3, 0.374), (0.374, 0.376), (0.376, 0.6), (0.1, 0.5)])
@pytest.mark.parametrize("D,shape", [(2, (5, 70)), (3, (3, 5, 65)), (2, (1100, 1000))])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
def test_h_matches_the_oracle(es, D, shape, dtype, zs):
    rng = np.random.default_rng(1)
    w = oracle.lattice(D)[1].reshape((-1,) + (1,) * D)
    # a uniform lattice at rest is its own next state: H of the step's output
    # is H of a known state, scaled in density for every cell alike
    z = rng.uniform(*zs) * rng.choice([-1.0, 1.0])
    f = np.broadcast_to(w * (1 + z) / (1 - z), (w.size,) + shape).copy()
    f *= 1 + 1e-6 * rng.standard_normal(shape)
    s = es.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype)
    a = torch.from_numpy(f - w if dtype.endswith("s") else f).to(s.storage_dtype).cuda()
    b = s.empty_state()
    s.set_stats(True)

    def check(state, h):
        g = state.double().cpu().numpy() + (w if dtype.endswith("s") else 0.0)
        terms = g * (np.log(g / w) - 1)
        assert abs(h - float(np.sum(terms))) <= 1e-13 * float(np.sum(np.abs(terms)))

    s.step(a, b, 1, 0.1)
    h1, h2 = s.stats(with_H=True)["H"], s.stats(with_H=True)["H"]
    check(b, h1)
    assert abs(h2 - h1) <= 1e-13 * abs(h1)
    s.step(b, a, 1, 0.1)
    assert s.stats(with_H=False)["H"] == 0.0
    check(a, s.stats(with_H=True)["H"])
