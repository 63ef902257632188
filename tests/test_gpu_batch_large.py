"""uf_batch against uf_step, bit for bit, from the sizes on where a grid's
own step takes other kernels than the batch's thread per corner: tiles that
march along x (advection from 2.5e5 cells, k-omega from 2.5e6, FP32),
several planes per thread (diffusion, drag and projection from 4.5e5), with
sides of every kind, an outlet above (diffusion and drag stay with the
thread per corner) and an inlet there (no planes, no marching); and a flow
so fast that traces leave the neighbouring cells."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from uf_layouts import default_config, porosity_field, random_city  # noqa: E402
from uf_layouts.configs import BC_INLET, BC_OUTLET, BC_SLIP, BC_WALL  # noqa: E402

O, I, W, S = BC_OUTLET, BC_INLET, BC_WALL, BC_SLIP
CASES = [
    ((72, 70, 52), [I, O, S, S, W, S], "f32"),      # 2.6e5: advection marches
    ((90, 80, 66), [I, O, I, O, W, S], "f32"),      # 4.8e5: planes
    ((90, 80, 66), [O, I, O, I, W, S], "f64"),      # planes in FP64
    ((90, 80, 66), [I, O, S, S, W, I], "f32"),      # an inlet above
    ((90, 80, 66), [I, O, W, S, S, O], "f32"),      # an outlet above
    ((150, 240, 70), [I, O, S, S, W, S], "f32"),    # 2.5e6: everything; full rows of a tile
    ((150, 240, 71), [I, O, I, O, W, W], "f32"),    # two tiles along z
    ((200, 290, 43), [O, I, S, S, W, O], "f32"),
    ((127, 1000, 20), [I, O, W, S, W, S], "f32"),
    ((61, 301, 144), [O, O, W, W, W, S], "f32"),
]


@pytest.mark.parametrize("speed", [1.0, 8.0])
@pytest.mark.parametrize("n,bc,dtype", CASES)
def test_batch_equals_steps(n, bc, dtype, speed):
    import paper_2204_01117_amd as U
    rng = np.random.default_rng(sum(n))
    cfg = default_config(*n, 2.0, dy=2.1, dz=1.9, dt=0.05, dtype=dtype, bc=bc, u_ref=4.0, wind_dir_deg=20.0,
                         cg_tol=1e-6 if dtype == "f32" else 1e-10, cg_maxit=200)
    boxes, trees, _ = random_city(*n, 2.0, 2.1, 1.9, 3, 10, 10)
    phi = torch.as_tensor(porosity_field(*n, 2.0, 2.1, 1.9, boxes, trees))
    grids = [U.Grid(cfg) for _ in range(2)]
    start = grids[0].state()
    for f in start:
        noise = torch.as_tensor(rng.standard_normal(tuple(start[f].shape))).to(start[f])
        start[f] = start[f] * speed + 0.5 * speed * noise if f in "uvw" else start[f] * (1 + 0.1 * noise.abs())
    for g in grids:
        g.set_porosity(phi)
        g.set_state(start)
    batch = U.Batch(grids[1:])
    for step in range(2):
        grids[0].step(1)
        batch.step(1)
        one, many = grids[0].state(), grids[1].state()
        for f in one:
            assert bool(torch.isfinite(one[f]).all()), (step, f)
            assert torch.equal(one[f], many[f]), (step, f, float((one[f] - many[f]).abs().max()),
                                                  int((one[f] != many[f]).sum()))
    batch.close()
    for g in grids:
        g.close()
