"""Host check of the ES-BGK quasi-equilibrium solve (tests/collision_check.hip,
built for the host with hipcc from the kernels' own headers; no GPU): on
strictly positive cells, from near the equilibrium to far from it, an accepted
quasi-equilibrium is finite, no cell is refused that the factored Newton solve
accepts, and the result is as close to the double-precision solve.
"""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not pathlib.Path(hipcc).exists():
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("collision") / "collision_check"
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only",
                           "-I", str(ROOT / "include"), str(ROOT / "tests" / "collision_check.hip"), "-o", str(exe)])
    return exe


def _solve(checker, D, dtype, pr, tau, spread):
    cells = 40000 if D == 2 else 10000
    r = subprocess.run([str(checker), "qe", str(D), dtype, str(pr), str(tau), str(cells), "1", str(spread)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    accepted, *rest = (float(v) for v in r.stdout.split())
    assert accepted > cells / 2
    return rest


@pytest.mark.parametrize("spread", [0.05, 0.5, 1.0, 2.0])
@pytest.mark.parametrize("pr,tau", [(1.4, 1.0), (0.71, 1.0), (3.0, 1.0), (0.5, 1e-3)])
@pytest.mark.parametrize("dtype", ["f32", "f32s", "f64"])
@pytest.mark.parametrize("D", [2, 3])
def test_accepted_quasi_equilibria_are_solutions(checker, D, dtype, pr, tau, spread):
    nonfinite, refused, err, err_newton = _solve(checker, D, dtype, pr, tau, spread)
    assert nonfinite == 0
    assert refused == 0
    # both solves end at the rounding of the residual, formed in the same type
    # by the same sums: a factor of four for the cells' spread.  In double the
    # reference is that Newton solve itself: the single-precision one's error,
    # by the ratio of the roundings, stands in.
    if dtype == "f64":
        err_newton = _solve(checker, D, "f32", pr, tau, spread)[3] * 2.0 ** -29
    assert err <= 4 * err_newton, (err, err_newton)
