"""The tiled smoothed-object kernels (4 x 4 columns, 64 levels, 8 objects at a
time, lists of 256) against the oracle at their edges: ragged tiles, more
objects in reach of a tile than a batch, more objects than a list round,
objects out of reach of every tile, floating and ground-standing ones.

The forward's operations are the oracle's up to the association of products
(FP64 rounding: 1e-14, as tests/test_gpu_design.py).  The gradient is
compared with the sum of phibar dphi/dp from the oracle's porosity by
central differences of step 1e-5 m: truncation about (1e-5 / width)^2 / 6 of
the third derivative's scale and rounding 1e-16 / 1e-5 per cell give about
1e-9 of the largest entry; the bound is 1e-7."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.smooth import smooth_porosity as oracle_smooth  # noqa: E402


def objects(rng, n, h, nb, nc, spread=1.0):
    L = [n[a] * h[a] for a in range(3)]
    bx, cy = [], []
    for _ in range(nb):
        c, w = rng.uniform(0, spread, 2) * L[:2], rng.uniform(1, 6, 2)
        z0 = 0.0 if rng.random() < 0.7 else rng.uniform(0.1, 0.4) * L[2]
        bx.append([c[0] - w[0], c[0] + w[0], c[1] - w[1], c[1] + w[1], z0, z0 + rng.uniform(1, 5), rng.uniform(0, 0.6)])
    for _ in range(nc):
        c = rng.uniform(0, spread, 2) * L[:2]
        z0 = 0.0 if rng.random() < 0.7 else rng.uniform(0.1, 0.4) * L[2]
        cy.append([c[0], c[1], rng.uniform(0.5, 3), z0, z0 + rng.uniform(1, 5), rng.uniform(0.2, 0.7)])
    return bx, cy


@pytest.mark.parametrize("n,nb,nc,width,spread", [
    ((4, 4, 64), 2, 1, 0.5, 1.0),       # one whole tile
    ((5, 9, 65), 3, 2, 0.5, 1.0),       # one past it along every axis
    ((23, 18, 7), 12, 9, 1.0, 0.3),     # more objects in reach than a batch holds
    ((40, 31, 20), 150, 140, 0.3, 1.0), # more objects than a list round
    ((30, 12, 16), 3, 3, 0.05, 4.0),    # most objects out of reach
])
def test_tiles_match_oracle(n, nb, nc, width, spread):
    import paper_2204_01117_amd as U
    h = (1.0, 1.2, 0.9)
    rng = np.random.default_rng(sum(n))
    bx, cy = objects(rng, n, h, nb, nc, spread)
    ref = oracle_smooth(n, h, bx, cy, width)
    phi = U.smooth_porosity(n, h, bx, cy, width, dtype="f64").cpu().numpy()
    assert np.abs(phi - ref).max() <= 1e-14
    pb = rng.normal(size=n)
    gb, gc = U.smooth_porosity_grad(n, h, bx, cy, width, torch.as_tensor(pb).cuda())
    g2 = U.smooth_porosity_grad(n, h, bx, cy, width, torch.as_tensor(pb).cuda())
    assert np.array_equal(gb, g2[0]) and np.array_equal(gc, g2[1])
    scale = max(np.abs(gb).max(), np.abs(gc).max())
    e = 1e-5
    for rows, grad in ((bx, gb), (cy, gc)):
        for o in rng.choice(len(rows), size=min(3, len(rows)), replace=False):
            for q in range(len(rows[o])):
                if q == (4 if rows is bx else 3) and rows[o][q] <= 0.0:
                    assert grad[o, q] == 0.0     # ground-standing: no lower step
                    continue
                keep = rows[o][q]
                rows[o][q] = keep + e
                hi = oracle_smooth(n, h, bx, cy, width)
                rows[o][q] = keep - e
                lo = oracle_smooth(n, h, bx, cy, width)
                rows[o][q] = keep
                # cells whose object changes between the two have no derivative there
                fd = ((hi - lo) / (2 * e) * pb)
                mid = oracle_smooth(n, h, bx, cy, width)
                smooth = np.abs(hi + lo - 2 * mid) <= 1e-7
                assert smooth.mean() > 0.999
                if smooth.all():
                    assert abs(fd.sum() - grad[o, q]) <= 1e-7 * scale, (o, q, fd.sum(), grad[o, q])
