"""An even count of steps leaves the newest state in both lattices, the bits of
single steps, whichever stores its copies take: grids on both sides of the
store rule's lines (smallest, fitting the last-level cache, beyond it), with
fields that start on cache lines and that do not, on two lattices and in place.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

TAU = 3e-3


@pytest.mark.parametrize("dtype,shape", [
    ("f32", (64, 64)), ("f64", (512, 512)), ("f64", (1024, 1024)), ("f32", (2049, 2047)), ("f32", (2113, 2111)),
    ("f16s", (2999, 3001)), ("f64", (61, 61, 61)), ("f32", (96, 96, 96)), ("f32", (131, 97, 203)),
    ("f32s", (108, 128, 128)), ("f64", (131, 97, 203)), ("f16s", (151, 151, 151))])
def test_both_copies_and_single_steps(dtype, shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12946_amd import eselbm
    D = len(shape)
    s = eselbm.Solver("D2Q9" if D == 2 else "D3Q27", shape, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(4)
    rho = 1 + 0.01 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.02 * torch.randn((D,) + shape, generator=g, device="cuda", dtype=torch.float64)
    f0 = s.init_equilibrium(rho, u)
    one, two = s.empty_state(), s.empty_state()
    s.step(f0, one, 1, TAU)
    s.step(one, two, 1, TAU)
    a, b = f0.clone(), torch.full_like(f0, float("nan"))
    s.step(a, b, 2, TAU)
    assert torch.equal(a, two) and torch.equal(b, two)
    a = f0.clone()
    s.step(a, a, 2, TAU)
    assert torch.equal(a, two)
