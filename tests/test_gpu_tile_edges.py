"""Edges of the tiles that the seed of the plane objective and the gradient of
the smoothed objects work in, against autograd of the same formulas (torch,
FP64, CPU).

Seed: a block evaluates 16 x 16 columns and owns the faces of 15 x 15, so nx
and ny on either side of 15 and 30 (where the last tile owns the closing
face alone), with a plane at the lowest and the highest pair of layers; the
rest is zeroed in 16-byte stores, so outputs of every length modulo them
(checked by the whole output).  Tolerances as tests/test_gpu_plane_seed.py
derives them: 1e-13 of the largest value in FP64, 4e-7 in FP32.

Smoothed objects: every parameter of every object is compared.  A cell's term
has about ten roundings, of exponents up to 40 long: 1e-14 of it; an
object's parameter sums at most a few thousand cells, each term at most the
largest entry's scale: 1e-10 of the largest."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from uf_layouts import default_config  # noqa: E402

PLANES = [((14, 15, 4), 0.5), ((15, 16, 3), 2.5), ((16, 14, 2), 0.9), ((15, 15, 5), 4.5), ((30, 15, 6), 2.0),
          ((29, 31, 3), 1.7), ((1, 30, 7), 6.5), ((45, 1, 2), 1.5)]


@pytest.mark.parametrize("dtype,bound", [("f32", 4e-7), ("f64", 1e-13)])
@pytest.mark.parametrize("n,zc", PLANES)
def test_plane_seed_tiles(n, zc, dtype, bound):
    import paper_2204_01117_amd as U
    rng = np.random.default_rng(sum(n))
    g = U.Grid(default_config(*n, 2.0, dz=1.5, dt=0.05, dtype=dtype))
    phi = torch.as_tensor(rng.uniform(0.0, 1.0, n))
    g.set_porosity(phi)
    st = g.state()
    g.set_state(dict(st, **{f: torch.as_tensor(rng.normal(size=tuple(st[f].shape))) for f in "uvw"}))
    st = g.state()
    u = [st[f].double().cpu().requires_grad_() for f in "uvw"]
    p = phi.to(st["u"].dtype).double().requires_grad_()
    pb = torch.zeros(n, dtype=torch.float64, device="cuda")
    _, grads = g.plane_objective(zc * 1.5, s_target=1.0, s_min=0.8, w_penalty=3.0, grad=True, phibar=pb)
    k0 = min(max(int(np.floor(zc - 0.5)), 0), n[2] - 2)
    t = zc - 0.5 - k0
    at = lambda q: (1 - t) * q[:, :, k0] + t * q[:, :, k0 + 1]
    c = [at(0.5 * (q.narrow(a, 0, n[a]) + q.narrow(a, 1, n[a]))) for a, q in enumerate(u)]
    s = torch.sqrt(sum(q ** 2 for q in c) + 1e-12)
    (4.0 * (at(p) * ((s - 1.0) ** 2 + 3.0 * torch.clamp(0.8 - s, min=0.0) ** 2)).sum()).backward()
    for a, b, tol in zip(list(grads) + [pb], u + [p], [bound] * 3 + [1e-13]):
        assert float((a.double().cpu() - b.grad).abs().max()) <= tol * float(b.grad.abs().max())
    g.close()


def objects(rng, L, nb, nc, lo, hi):
    """Objects whose centres lie in the fraction lo to hi of the ground plan."""
    bx, cy = [], []
    for _ in range(nb):
        c, w = rng.uniform(lo, hi, 2) * L[:2], rng.uniform(1, 4, 2)
        z0 = 0.0 if rng.random() < 0.5 else rng.uniform(0.1, 0.4) * L[2]
        bx.append([c[0] - w[0], c[0] + w[0], c[1] - w[1], c[1] + w[1], z0, z0 + rng.uniform(1, 5), rng.uniform(0, 0.6)])
    for _ in range(nc):
        c = rng.uniform(lo, hi, 2) * L[:2]
        z0 = 0.0 if rng.random() < 0.5 else rng.uniform(0.1, 0.4) * L[2]
        cy.append([c[0], c[1], rng.uniform(0.5, 3), z0, z0 + rng.uniform(1, 5), rng.uniform(0.2, 0.7)])
    return bx, cy


@pytest.mark.parametrize("n,parts,width", [
    ((9, 5, 65), [(2, 1, 0.0, 1.0)], 0.5),
    ((23, 18, 7), [(12, 9, 0.2, 0.5)], 1.0),                         # several batches reach a tile
    ((16, 12, 8), [(256, 0, 5.0, 6.0), (3, 2, 0.3, 0.7)], 0.3),      # the second round of the list alone
    ((16, 12, 8), [(5, 0, 0.3, 0.7), (251, 40, 5.0, 6.0)], 0.3),     # the first alone, of two
    ((31, 33, 20), [(700, 324, 0.0, 1.0)], 0.4),                     # as many objects as the gradient takes
])
def test_smooth_gradient_every_parameter(n, parts, width):
    import paper_2204_01117_amd as U
    h = (1.0, 1.2, 0.9)
    rng = np.random.default_rng(sum(n))
    L = np.array(n) * h
    bx, cy = [], []
    for nb, nc, lo, hi in parts:
        b, c = objects(rng, L, nb, nc, lo, hi)
        bx += b
        cy += c
    pb = rng.normal(size=n)
    gb, gc = U.smooth_porosity_grad(n, h, bx, cy, width, torch.as_tensor(pb).cuda())
    px, py, pz = ((torch.arange(m, dtype=torch.float64) + 0.5) * d for m, d in zip(n, h))
    sig = lambda t: torch.sigmoid(t / width)
    tb = torch.tensor(bx, dtype=torch.float64).reshape(-1, 7).requires_grad_()
    tc = torch.tensor(cy, dtype=torch.float64).reshape(-1, 6).requires_grad_()
    phi = torch.ones(n, dtype=torch.float64)
    owner = torch.full(n, -1)
    values = []
    for q, r in enumerate(list(tb) + list(tc)):
        if q < len(bx):
            flat = (sig(px - r[0]) * sig(r[1] - px))[:, None] * (sig(py - r[2]) * sig(r[3] - py))[None, :]
            z0, z1, po = r[4], r[5], r[6]
        else:
            flat = sig(r[2] - torch.sqrt((px[:, None] - r[0]) ** 2 + (py[None, :] - r[1]) ** 2))
            z0, z1, po = r[3], r[4], r[5]
        lev = sig(z1 - pz) * (sig(pz - z0) if float(z0) > 0 else 1.0)
        v = 1.0 - flat[:, :, None] * lev * (1.0 - po)
        less = v.detach() < phi      # the first object that reaches the minimum holds the cell
        phi = torch.where(less, v.detach(), phi)
        owner = torch.where(less, torch.tensor(q), owner)
        values.append(v)
    loss = sum((torch.where(owner == q, v, torch.zeros_like(v)) * torch.as_tensor(pb)).sum() for q, v in enumerate(values))
    loss.backward()
    scale = max(float(t.grad.abs().max()) for t in (tb, tc) if t.numel())
    assert scale > 0
    for got, t in ((gb, tb), (gc, tc)):
        if t.numel():
            assert np.abs(got - t.grad.numpy()).max() <= 1e-10 * scale
