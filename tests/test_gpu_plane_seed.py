"""The plane objective's gradient with respect to the state and the porosity
against autograd of the same formula in FP64 (torch, CPU), at the edges of
the seed kernel's blocks of 1024 faces: the fewest layers (most columns in a
block), columns longer than a block, ragged planes.

Tolerance: about thirty roundings of FP64 arithmetic, 30 * 2^-53 < 1e-14,
between quantities no larger than the compared one times ten: 1e-13 of the
largest value; FP32 grids, from the same FP32 state, round both cells' terms,
at most three times the largest result, and their sum: 7 * 2^-24 = 4e-7."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from uf_layouts import default_config  # noqa: E402


@pytest.mark.parametrize("dtype,bound", [("f32", 4e-7), ("f64", 1e-13)])
@pytest.mark.parametrize("n,zc", [((3, 1030, 2), 1.0), ((2, 7, 2), 0.5), ((4, 3, 1100), 1050.3), ((5, 33, 17), 16.5),
                                  ((1, 1, 5), 2.2), ((9, 64, 64), 1.5)])
def test_plane_seed_matches_autograd(n, zc, dtype, bound):
    import paper_2204_01117_amd as U
    cfg = default_config(*n, 2.0, dz=1.5, dt=0.05, dtype=dtype)
    rng = np.random.default_rng(sum(n))
    g = U.Grid(cfg)
    phi = torch.as_tensor(rng.uniform(0.0, 1.0, n))
    g.set_porosity(phi)
    st = g.state()
    g.set_state(dict(st, **{f: torch.as_tensor(rng.normal(size=tuple(st[f].shape))) for f in "uvw"}))
    st = g.state()
    u = [st[f].double().cpu().requires_grad_() for f in "uvw"]
    p = phi.to(st["u"].dtype).double().requires_grad_()
    z = zc * 1.5
    pb = torch.zeros(n, dtype=torch.float64, device="cuda")
    J, grads = g.plane_objective(z, s_target=1.0, s_min=0.8, w_penalty=3.0, grad=True, phibar=pb)
    c = [0.5 * (u[0][:-1] + u[0][1:]), 0.5 * (u[1][:, :-1] + u[1][:, 1:]), 0.5 * (u[2][:, :, :-1] + u[2][:, :, 1:])]
    k0 = min(max(int(np.floor(z / 1.5 - 0.5)), 0), n[2] - 2)
    t = z / 1.5 - 0.5 - k0
    at = lambda q: (1 - t) * q[:, :, k0] + t * q[:, :, k0 + 1]
    s = torch.sqrt(sum(at(q) ** 2 for q in c) + 1e-12)
    ref = 2.0 * 2.0 * (at(p) * ((s - 1.0) ** 2 + 3.0 * torch.clamp(0.8 - s, min=0.0) ** 2)).sum()
    ref.backward()
    print(n, dtype, J, float(ref.detach()), flush=True)
    assert abs(J - float(ref.detach())) <= 1e-12 * abs(J)
    for a, b in zip(list(grads) + [pb], u + [p]):
        scale = float(b.grad.abs().max())
        tol = 1e-13 if a is pb else bound
        assert float((a.double().cpu() - b.grad).abs().max()) <= tol * scale
    g.close()
