"""The projection's iterates, step by step, against plain numpy conjugate
gradients with the same preconditioner (the V-cycle as defined: halved levels,
piecewise-constant transfers, one damped Jacobi sweep before and after, 48
sweeps on the coarsest level; or the diagonal), on grids that take every pass
of the solver: levels blocked in runs of planes (the finest, and a coarser one
of 2^18 cells), levels of a thread per cell, the one-workgroup levels from
their smallest to their largest, thin grids whose levels shrink by two, odd
extents.  After m iterations the two differ by rounding only: each iteration
adds a few units of 2^-53 times the few hundred terms of its dot products and
sweeps, far below the 1e-10 of the bar."""
import numpy as np
import pytest

from paper_2504_00745_amd import workloads as wl

pytestmark = pytest.mark.gpu

OMEGA = 2.0 / 3.0


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_00745_amd import gic
    gic.lib()
    import gpu_util
    return gpu_util


class Level:
    def __init__(self, ac, scale):
        self.ac, self.scale = ac, scale
        self.fluid = ac > 0
        self.beta = []
        diag = np.zeros_like(ac)
        for ax in range(3):
            m = ac.shape[ax] - 1
            lo, hi = [slice(None)] * 3, [slice(None)] * 3
            lo[ax], hi[ax] = slice(0, m), slice(1, m + 1)
            a, b = ac[tuple(lo)], ac[tuple(hi)]
            w = np.where((a != 0) & (b != 0), 0.5 * (np.abs(a) + np.abs(b)), 0.0)
            self.beta.append((tuple(lo), tuple(hi), w))
            diag[tuple(lo)] += w
            diag[tuple(hi)] += w
        with np.errstate(divide="ignore"):
            self.dinv = np.where(self.fluid, np.where(diag > 0, 1.0 / (scale * diag), 0.0), 1.0)

    def A(self, v):
        v = np.where(self.fluid, v, 0.0)
        out = np.zeros_like(v)
        for lo, hi, w in self.beta:
            f = w * (v[lo] - v[hi])
            out[lo] += f
            out[hi] -= f
        return self.scale * out


def blocks(a, fill=0.0):
    """(8, coarse shape): the children of every coarse cell."""
    pad = np.pad(a, [(0, m % 2) for m in a.shape], constant_values=fill)
    z, y, x = [m // 2 for m in pad.shape]
    return pad.reshape(z, 2, y, 2, x, 2).transpose(1, 3, 5, 0, 2, 4).reshape(8, z, y, x)


def hierarchy(ac):
    levels = [Level(ac, 1.0)]
    while levels[-1].ac.size > 256:
        c = blocks(levels[-1].ac)
        n = (c != 0).sum(0)
        mean = np.abs(c).sum(0) / np.maximum(n, 1)
        levels.append(Level(np.where((c < 0).any(0), -mean, np.where((c > 0).any(0), mean, 0.0)), 4.0 * levels[-1].scale))
    return levels


def vcycle(levels, l, b):
    L = levels[l]
    if l == len(levels) - 1:
        e = np.zeros_like(b)
        for _ in range(48):
            e = np.where(L.fluid, e + OMEGA * L.dinv * (b - L.A(e)), 0.0)
        return e
    e = OMEGA * L.dinv * b
    res = np.where(L.fluid, b - L.A(e), 0.0)
    bc = np.where(levels[l + 1].fluid, blocks(res).sum(0), 0.0)
    ec = np.where(levels[l + 1].fluid, vcycle(levels, l + 1, bc), 0.0)
    up = ec.repeat(2, 0).repeat(2, 1).repeat(2, 2)[tuple(slice(0, m) for m in b.shape)]
    u = np.where(L.fluid, e + up, 0.0)
    return np.where(L.fluid, u + OMEGA * L.dinv * (b - L.A(u)), b)


def reference(at, lab, s, iters, precond):
    levels = hierarchy(np.where(lab == 0, at, np.where(lab == 1, -at, 0.0)))
    L = levels[0]
    M = (lambda r: vcycle(levels, 0, r)) if precond and len(levels) > 1 else (lambda r: L.dinv * r)
    q, r = np.zeros_like(s), np.where(lab == 0, s, 0.0)
    z = M(r)
    d, rz = z.copy(), (r * z).sum()
    for _ in range(iters):
        w = np.where(L.fluid, L.A(d), d)
        alpha = rz / (d * w).sum()
        q += alpha * d
        r -= alpha * w
        z = M(r)
        rz, old = (r * z).sum(), rz
        d = z + (rz / old) * d
    return q, np.linalg.norm(r) / np.linalg.norm(s)


@pytest.mark.parametrize("precond", [1, 0])
@pytest.mark.parametrize("shape", [(32, 32, 32), (17, 16, 15), (41, 35, 37), (61, 66, 131), (9000, 1, 1), (2, 300, 5),
                                   (128, 130, 130), (5, 5, 11), (33, 47, 64)])
def test_iterates(G, shape, precond):
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[idp iterates] {shape} precond {precond}")
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(nx * ny + nz))
    at = rng.uniform(0.3, 1.0, shape)
    lab = (rng.random(shape) < 0.02).astype(np.uint8) * 2
    lab[rng.random(shape) < 0.02] = 1
    lab[3 * nz // 4:] = 1
    s = np.where(lab == 0, rng.normal(0, 0.1, shape), 0.0)
    p = wl._params((nx, ny, nz), 0.01, 0.01, 1e-4, (0.0, 0.0, 0.0))
    ctx = gic.Context(p, 1, "fp64", r_max=0.0025)
    work = gic.idp_workspace(ctx)
    iters = 4 if at.size > 1 << 20 else 7  # an odd and an even count: the buffers change places
    for m in (iters, iters + 1):
        q = torch.zeros(ctx.G, dtype=torch.float64, device="cuda")
        it, rel = gic.gic_idp_solve(ctx, G.dev(at.reshape(-1)), torch.as_tensor(lab.reshape(-1)).to("cuda"),
                                    G.dev(s.reshape(-1)), q, work, max_iter=m, tol=0.0, check_every=3, precond=precond)
        want, wrel = reference(at, lab, s, m, precond)
        assert it == m
        got = q.view(shape).cpu().numpy()
        assert np.linalg.norm(got - want) <= 1e-10 * np.linalg.norm(want)
        assert abs(rel - wrel) <= 1e-9 * wrel
        assert not got[lab != 0].any()
