"""A cell's closed-form path length depends on the cell alone: the step of a
translated lattice is the translated step, to the bit.

Most cells lie in the extended series' range, beyond the common series' bound;
one column lies beyond the extended series, so that some waves hold such cells
and others do not, and the translation moves cells from the one to the other.
"""
import numpy as np
import pytest
import torch

import oracle
from tests._states import unstream

pytestmark = pytest.mark.gpu

TAU = 3e-3


def _state(D, shape, amp, far):
    """Pulled cells of relative perturbations ``amp``, in the column x = 20 ``far``."""
    rng = np.random.default_rng(11)
    u = 0.03 * rng.standard_normal((D,) + shape)
    g = oracle.init_equilibrium(1 + 0.01 * rng.standard_normal(shape), u)
    a = np.full(shape, amp)
    a[..., 20] = far
    return unstream(g * (1 + a * rng.uniform(-1, 1, g.shape)))


# rows of whole waves and of partial ones, and lanes through whole planes
@pytest.mark.parametrize("shape", [(6, 128), (5, 300), (520, 514), (4, 6, 128), (3, 7, 150), (30, 45, 66)])
@pytest.mark.parametrize("mode", ["higher", "lower"])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s", "f16s"])
def test_translation(dtype, mode, shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12946_amd import eselbm
    D = len(shape)
    f = _state(D, shape, *((0.03, 0.2) if dtype == "f64" else (0.07, 0.4)))
    if dtype in ("f32s", "f16s"):
        f = f - oracle.lattice(D)[1].reshape((-1,) + (1,) * D)
    s = eselbm.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype, mode=mode)
    s.set_stats(True)
    a = torch.from_numpy(f).cuda().to(s.storage_dtype)
    alpha = [torch.empty(shape, dtype=s.compute_dtype, device="cuda") for _ in range(2)]
    out = []
    for k, fin in enumerate((a, a.roll(60, -1))):
        s.set_alpha_field(alpha[k])
        b = s.empty_state()
        s.step(fin, b, 1, TAU)
        out.append(b)
    st = s.stats()
    assert st["n_exact"] > 0.5 * s.cells and st["n_nonpos"] == 0
    assert torch.equal(alpha[0].roll(60, -1), alpha[1])
    assert torch.equal(out[0].roll(60, -1), out[1])
