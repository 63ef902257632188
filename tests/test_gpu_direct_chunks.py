"""The direct solve where the device decides: a chunk of several iterations
whose status the host has not read enqueues products and smoothing sweeps
for each, of which one kind returns at once.  Against the solve of a fresh
grid, whose host reads the status after each iteration and enqueues one
kind: the same iterations and the same bits, for a solve that ends after
products, after a smoothing iteration, after the products that follow a
smoothing iteration which fell short, and after products twice; in chunks
shorter than the solve, as long and longer, through uf_step and through
uf_batch's captured solves (replayed several times)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from uf_layouts import default_config, porosity_field, random_city  # noqa: E402

# tolerance as a fraction of the residual that the first products leave ->
# (iterations, of which with products): a smoothing iteration is tried up to
# a factor of 4.5, and reduces the residual of these grids 3.1 to 4.4 times
ENDS = [(0.9, 1, 1), (3.0, 2, 1), (4.45, 3, 2), (50.0, 2, 2)]


def grid(n, tol, maxit=50):
    import paper_2204_01117_amd as U
    cfg = default_config(*n, 2.0, dt=0.04, dtype="f32", u_ref=6.0, wind_dir_deg=32.0, cg_tol=tol, cg_maxit=maxit)
    g = U.Grid(cfg)
    boxes, trees, _ = random_city(*n, 2.0, 2.0, 2.0, 1, 3, 4)
    g.set_porosity(torch.as_tensor(porosity_field(*n, 2.0, 2.0, 2.0, boxes, trees)))
    return g


def same(a, b):
    return all(torch.equal(a[f], b[f]) for f in a)


@pytest.mark.parametrize("n", [(120, 6, 8), (24, 40, 33), (17, 33, 31)])
def test_unread_chunks(n):
    import paper_2204_01117_amd as U
    rng = np.random.default_rng(1)
    g = grid(n, 1e-6)
    g.step(2)
    start = {f: t.clone() for f, t in g.state().items()}
    g.close()
    for f in "uvw":
        start[f] += 0.3 * torch.as_tensor(rng.standard_normal(tuple(start[f].shape))).to(start[f])
    g = grid(n, 1e-30, maxit=1)
    g.set_state(start)
    left = g.step(1, allow=(4,))["cg_rel_residual"]
    g.close()
    for c, iters, products in ENDS:
        tol = left / c

        def alone(state):
            """The step of a fresh grid: chunks of one iteration, each status read."""
            g = grid(n, tol)
            g.timer_enable(["ds_row"])
            g.set_state(state)
            d = g.step(1)
            out = (d["cg_iters"], {f: t.clone() for f, t in g.state().items()}, g.timer_read("ds_row")[1] // 2)
            g.close()
            return out

        want = alone(start)
        assert (want[0], want[2]) == (iters, products), c
        # the same flow with the pressure that solves it: its solve ends at once or after one iteration
        solved = dict(start, p=want[1]["p"])
        short = alone(solved)
        assert short[0] <= 1
        g = grid(n, tol)
        g.set_state(start)
        g.step(1)
        # a chunk is as long as the solve before it: as long as needed, longer, shorter, as long
        for state, (count, fields, _) in ((start, want), (solved, short), (start, want), (start, want)):
            g.set_state(state)
            d = g.step(1)
            assert d["cg_iters"] == count and same(g.state(), fields), (c, d)
        # the captured solve holds as many iterations as the grid's last one took; replayed with eager work between
        batch = U.Batch([g])
        for state, (count, fields, _) in ((start, want), (start, want), (solved, short), (start, want), (start, want)):
            g.set_state(state)
            d = batch.step(1)[0]
            assert d["cg_iters"] == count and same(g.state(), fields), (c, d)
        batch.close()
        g.close()
