"""The direct pressure solve (transforms along y and z on the matrix cores,
tridiagonal systems along x) against the oracle's solver, at the edges of
its tiles: below, at and past the 16/8-deep slices, the 32/64/128-wide
tiles, the rows per wavefront of the tridiagonal kernel and its longest
line, over every kind of open and closed side.

Tolerances: the solve stops at ||r|| <= cg_tol ||b||.  FP64 at 1e-13 and
condition numbers up to about 1e5 leave the solution within 1e-10 (the
suite's bound for a solved FP64 pressure); FP32 within 1e-5 (the suite's
bound for an FP32 pressure)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.bc import Geometry  # noqa: E402
from oracle.pressure import PressureSolver  # noqa: E402
from tests.helpers import rel, to_np  # noqa: E402
from uf_layouts import default_config  # noqa: E402
from uf_layouts.configs import BC_INLET, BC_OUTLET, BC_SLIP, BC_WALL, PC_MG  # noqa: E402

O, I, W, S = BC_OUTLET, BC_INLET, BC_WALL, BC_SLIP
CASES = [
    ((2, 2, 1), [I, O, W, S, W, S]),
    ((3, 5, 2), [O, I, O, I, W, S]),
    ((8, 16, 16), [I, I, O, O, W, S]),        # one wavefront per line, whole tiles
    ((9, 17, 13), [O, O, I, O, W, S]),        # one past each
    ((17, 33, 31), [I, W, W, S, O, S]),       # the only outlet on the ground
    ((129, 31, 33), [I, O, I, O, W, O]),      # 16 rows per wavefront, ragged last one
    ((40, 65, 65), [O, I, W, W, O, O]),       # second tile along y and z
    ((6, 130, 129), [I, O, O, O, W, S]),      # third tile along y, second along z
    ((257, 9, 18), [O, I, S, S, W, S]),       # 32 rows per wavefront
    ((512, 6, 8), [I, O, I, I, W, S]),        # the longest line
]


def solve(shape, bc, dtype, tol, x0=None):
    import paper_2204_01117_amd as U
    cfg = default_config(*shape, 2.0, dy=1.7, dz=2.3, dt=0.1, dtype=dtype, bc=bc, precond=PC_MG, cg_tol=tol,
                         cg_maxit=50)
    rng = np.random.default_rng(sum(shape))
    b = rng.normal(size=shape).astype(np.float32)
    g = U.Grid(cfg)
    x, st = g.pressure_solve(torch.as_tensor(b), x0)
    g.close()
    ps = PressureSolver(Geometry(dict(cfg)), method="auto")
    ref, _ = ps.solve(b.astype(np.float64).ravel(), np.zeros(b.size))
    return to_np(x), ref.reshape(shape), st


@pytest.mark.parametrize("dtype,tol,bound", [("f32", 1e-6, 1e-5), ("f64", 1e-13, 1e-10)])
@pytest.mark.parametrize("shape,bc", CASES)
def test_direct_solve_matches_oracle(shape, bc, dtype, tol, bound):
    x, ref, st = solve(shape, bc, dtype, tol)
    print(shape, dtype, "iterations", st["cg_iters"], "rel", rel(x, ref), flush=True)
    assert st["converged"] == 1 and st["cg_rel_residual"] <= tol
    assert st["cg_iters"] <= 4      # the CG takes at least eight on these
    assert rel(x, ref) <= bound


def test_direct_solve_from_a_guess_and_past_the_line_limit():
    """A guess is improved, not replaced; a line past 512 rows takes the CG."""
    shape, bc = (24, 20, 18), [I, O, O, O, W, S]
    x, ref, st = solve(shape, bc, "f64", 1e-13)
    y, _, st2 = solve(shape, bc, "f64", 1e-13, x0=torch.as_tensor(1.001 * x))
    assert st2["converged"] == 1 and rel(y, ref) <= 1e-10
    x, ref, st = solve((520, 6, 8), bc, "f64", 1e-13)
    assert st["converged"] == 1 and st["cg_iters"] > 4 and rel(x, ref) <= 1e-9


@pytest.mark.parametrize("dtype,bound", [("f32", 1e-5), ("f64", 1e-10)])
@pytest.mark.parametrize("shape,bc", CASES[2:])
def test_direct_solve_smoothing_iteration(shape, bc, dtype, bound):
    """A threshold just below what the first iteration leaves is met by an
    iteration of sweeps (within 4.5 times it), one far below by products;
    the iterate is then the solution to the same bounds."""
    _, _, st = solve(shape, bc, dtype, 0.5)
    assert st["cg_iters"] == 1
    r0 = st["cg_rel_residual"]
    for ratio in (2.0, 4.4, 20.0):
        x, ref, st = solve(shape, bc, dtype, r0 / ratio)
        print(shape, dtype, "ratio", ratio, "iterations", st["cg_iters"], "left", st["cg_rel_residual"] / r0,
              flush=True)
        assert st["converged"] == 1 and st["cg_rel_residual"] <= r0 / ratio
        assert 2 <= st["cg_iters"] <= 4
        assert rel(x, ref) <= bound
