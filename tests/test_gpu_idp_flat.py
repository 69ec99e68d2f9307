"""The projection's iterates on flat and narrow grids, whose axes the solver may
take in another order: axes of one cell in every place, few rows and many planes
(the tiles then lie in x and z; also on a coarser level), against the numpy
conjugate gradients of the iterates' test, to its 1e-10; the whole projection with
its face displacements on a flat grid and on the same grid lying in x and y."""
import numpy as np
import pytest

from paper_2504_00745_amd import workloads as wl
from test_gpu_idp_iterations import G, reference  # noqa: F401 (G: a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precond", [1, 0])
@pytest.mark.parametrize("shape", [(40, 1, 90), (90, 40, 1), (1, 40, 90), (1, 1, 700), (1, 700, 1), (700, 1, 1), (530, 1, 520),
                                   (300, 2, 50), (271, 3, 341), (90, 7, 33), (1030, 5, 520), (9, 7, 40), (7, 7, 100)])
def test_iterates(G, shape, precond):  # noqa: F811
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[idp flat] {shape} precond {precond}")
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(nx * ny + nz))
    at = rng.uniform(0.3, 1.0, shape)
    lab = (rng.random(shape) < 0.02).astype(np.uint8) * 2
    lab[rng.random(shape) < 0.02] = 1
    axis = int(np.argmax(shape))  # an air layer across the longest axis
    np.moveaxis(lab, axis, 0)[3 * shape[axis] // 4:] = 1
    s = np.where(lab == 0, rng.normal(0, 0.1, shape), 0.0)
    ctx = gic.Context(wl._params((nx, ny, nz), 0.01, 0.01, 1e-4, (0.0, 0.0, 0.0)), 1, "fp64", r_max=0.0025)
    work = gic.idp_workspace(ctx)
    iters = 4 if at.size > 1 << 20 else 7
    for m in (iters, iters + 1):  # an odd and an even count: the buffers change places
        q = torch.zeros(ctx.G, dtype=torch.float64, device="cuda")
        it, rel = gic.gic_idp_solve(ctx, G.dev(at.reshape(-1)), torch.as_tensor(lab.reshape(-1)).to("cuda"),
                                    G.dev(s.reshape(-1)), q, work, max_iter=m, tol=0.0, check_every=3, precond=precond)
        want, wrel = reference(at, lab, s, m, precond)
        assert it == m
        got = q.view(shape).cpu().numpy()
        assert np.linalg.norm(got - want) <= 1e-10 * np.linalg.norm(want)
        assert abs(rel - wrel) <= 1e-9 * wrel
        assert not got[lab != 0].any()


def test_projection_of_a_flat_grid(G):  # noqa: F811
    """nx x 1 x nz against nx x nz x 1: the same cells in the same places."""
    import torch
    from paper_2504_00745_amd import gic
    nx, nz = 70, 45
    rng = np.random.Generator(np.random.PCG64(8))
    afx = (rng.uniform(0.0, 0.6, nx * nz) * 2 ** 32).astype(np.int64)
    star = rng.uniform(0.4, 1.0, nx * nz)
    lab = (rng.random(nx * nz) < 0.1).astype(np.uint8)
    out = []
    for n in ((nx, 1, nz), (nx, nz, 1)):
        ctx = gic.Context(wl._params(n, 0.01, 0.01, 1e-4, (0.0, 0.0, 0.0)), 1, "fp64", r_max=0.0025)
        e = lambda m: torch.full((m,), -7.0, dtype=torch.float64, device="cuda")  # noqa: E731
        f = [e((n[0] + 1) * n[1] * n[2]), e(n[0] * (n[1] + 1) * n[2]), e(n[0] * n[1] * (n[2] + 1))]
        q = torch.zeros(ctx.G, dtype=torch.float64, device="cuda")
        it, rel = gic.gic_density_projection(ctx, torch.as_tensor(afx).cuda(), G.dev(star), torch.as_tensor(lab).cuda(), q, *f,
                                             gic.idp_workspace(ctx), tol=1e-10)
        out.append((it, rel, q, f))
    (ia, ra, qa, fa), (ib, rb, qb, fb) = out
    assert ia == ib and ra <= 1e-10 and torch.equal(qa, qb)
    assert torch.equal(fa[0], fb[0]) and torch.equal(fa[2], fb[1])
    assert not fa[1].any() and not fb[2].any()
