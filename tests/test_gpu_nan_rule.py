"""One NaN face: a step writes non-finite values at the same positions on
every path.  ``Grid.step`` takes a component per block on small grids, tiles
that march along x from 2.5e5 cells in FP32 (with blocks of their own for the
corners beside the sides) and several planes per thread from 4.5e5;
``Batch.step`` takes a thread per corner throughout.  A NaN velocity clamps
its trace to a position whose samples are finite, so a path that forgot to
put the NaN back would write a finite value there.

Positions are compared, not values: no tolerance."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from uf_layouts import default_config, porosity_field, random_city  # noqa: E402

# (nx - 2, ...): beside a side along x; (..., ny - 1, ...): on one along y
PLACES = [("u", (0.5, 0.5, 0.5)), ("v", (0.5, 2, 0.5)), ("w", (2, 0.5, 0.5)), ("u", (-2, 0.5, 1)),
          ("v", (0.5, -1, -1))]


@pytest.mark.parametrize("n,dtype", [((20, 16, 12), "f32"), ((20, 16, 12), "f64"), ((72, 70, 52), "f32"),
                                     ((72, 100, 64), "f32"), ((80, 76, 68), "f64")])
def test_one_nan_face(n, dtype):
    import paper_2204_01117_amd as U
    cfg = default_config(*n, 2.0, dt=0.09, dtype=dtype, u_ref=6.0, wind_dir_deg=32.0)
    boxes, trees, _ = random_city(*n, 2.0, 2.0, 2.0, 1, 4, 5)
    phi = torch.as_tensor(porosity_field(*n, 2.0, 2.0, 2.0, boxes, trees))
    grids = [U.Grid(cfg) for _ in range(2)]
    for g in grids:
        g.set_porosity(phi)
    grids[0].step(2)
    state = {f: t.clone() for f, t in grids[0].state().items()}
    batch = U.Batch(grids[1:])
    for f, at in PLACES:
        idx = tuple(int(a * m) if isinstance(a, float) else a % m for a, m in zip(at, n))
        st = dict(state)
        st[f] = state[f].clone()
        st[f][idx] = float("nan")
        for g in grids:
            g.set_state(st)
        assert grids[0].step(1, allow=(5,))["status"] == "UF_ENONFINITE"
        assert batch.step(1, allow=(5,))[0]["status"] == "UF_ENONFINITE"
        one, many = grids[0].state(), grids[1].state()
        for q in one:
            a, b = ~torch.isfinite(one[q]), ~torch.isfinite(many[q])
            assert torch.equal(a, b), (n, dtype, f, idx, q, int(a.sum()), int(b.sum()))
        assert all(bool((~torch.isfinite(one[q])).any()) for q in "uvw")
    batch.close()
    for g in grids:
        g.close()
