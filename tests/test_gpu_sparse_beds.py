"""Brick kernels on beds of about one granule per cell, where they run one
wave per brick (gather, direct contact, P2G), and the per-granule P2G: a
ragged jittered lattice of 72,283 granules (past the size from which the wave
form is taken) with one brick replaced by a clump of 216 (a wave loops over
its brick; its shell overflows the wave's LDS array).

The references are the kernels that run a thread per granule without bricks
(reorder, G2P, drag, the contact from the neighbour list, integrate) and the
oracle's integer P2G; every comparison is bit for bit, on the first call
(both forms launched, the device picks one) and on later ones (the count of
occupied bricks has reached the host)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_00745_amd import gic
    gic.lib()
    import gpu_util
    return gpu_util


def bed(dims, clump=True, seed=3):
    rng = np.random.Generator(np.random.PCG64(seed))
    sp = 0.003
    g = np.stack(np.meshgrid(*[np.arange(m) for m in dims], indexing="ij")).reshape(3, -1).astype(float)
    r = rng.uniform(0.75e-3, 1.44e-3, g.shape[1])
    x = (g + 0.5) * sp + rng.uniform(-1, 1, g.shape) * np.maximum(sp / 2 - r / 1.03, 0.0)
    if clump:  # brick (2, 3, 4): 6^3 granules of 0.4 diameters spacing in place of its own
        lo = np.array([8, 12, 16]) * sp
        inside = np.all((x > lo[:, None]) & (x < lo[:, None] + 4 * sp), axis=0)
        h = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij")).reshape(3, -1)
        y = lo[:, None] + (h + 0.5) * (4 * sp / 6) + rng.uniform(-1e-5, 1e-5, h.shape)
        x = np.concatenate([x[:, ~inside], y], axis=1)
        r = np.concatenate([r[~inside], np.full(216, 1.003e-3)])
    p = rng.permutation(x.shape[1])
    x, r = np.ascontiguousarray(x[:, p]), np.ascontiguousarray(r[p])
    n = [m + 3 for m in dims]
    cfg = dict(kn=1e5, restitution=0.5, kt_ratio=1.0, mu=0.5, rho_s=2500.0, eta_f=1e-3, c_drag=1.0, alpha_max=0.74,
               walls=0x3F, n=n, dx=sp, nc=list(n), cell=sp, dt=2e-5, g=[0.0, 0.0, -9.81])
    v = rng.normal(0.0, 5.0, x.shape)  # some stencils leave their brick's tile in one move
    u = rng.normal(0.0, 0.1, (3, int(np.prod(n))))
    return cfg, x, v, r, u


def setup(G, gic, cfg, x, v, r, u, prec, r_max=1.5e-3):
    import torch
    n = x.shape[1]
    ctx = gic.Context(cfg, n, prec, r_max=r_max)
    i32 = lambda m: torch.empty(m, dtype=torch.int32, device="cuda")  # noqa: E731
    s = dict(ctx=ctx, n=n, X=G.dev(x), V=G.dev(v), R=G.dev(r), U=G.dev(u, ctx.real), key=i32(n), order=i32(n),
             cb=i32(ctx.K), ce=i32(ctx.K))
    gic.gic_sort_cells(ctx, s["X"], s["key"], s["order"], s["cb"], s["ce"])
    s["Xs"], s["Vs"], s["Rs"] = (torch.empty_like(s[k]) for k in "XVR")
    gic.gic_reorder(ctx, s["order"], s["X"], s["V"], s["R"], None, s["Xs"], s["Vs"], s["Rs"], None)
    return s


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("dims", [(41, 43, 41), (13, 11, 9)])
def test_sparse_bed_matches_per_granule_kernels(G, orc, prec, dims):
    """(13, 11, 9): the 256-thread forms of the same kernels."""
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[sparse] {dims} {prec}")
    cfg, x, v, r, u = bed(dims, clump=dims[0] > 16)
    s = setup(G, gic, cfg, x, v, r, u, prec)
    ctx, n, cells = s["ctx"], s["n"], (s["cb"], s["ce"])
    real = ctx.real
    e = lambda m, t=real: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    A, M = e(ctx.G, torch.int64), e(3 * ctx.G, torch.int64)
    ao, mo = orc.p2g_fixed(cfg, x, v, r)
    uat, af, Fd = e(3 * n), e(n), e(3 * n)
    Fc, pairs = e(3 * n), e(8 * n, torch.int32)
    for call in range(3):
        gic.gic_p2g(ctx, s["Xs"], s["Vs"], s["Rs"], *cells, A, M)
        torch.cuda.synchronize()  # from the second call on the count of bricks is known
        assert np.array_equal(A.cpu().numpy(), ao) and np.array_equal(M.view(3, -1).cpu().numpy(), mo), call
        # alpha only
        B = e(ctx.G, torch.int64)
        gic.gic_p2g(ctx, s["Xs"], s["Vs"], s["Rs"], *cells, B, None)
        assert torch.equal(A, B)
        gic.gic_g2p(ctx, s["Xs"], s["U"], A, None, uat, af)
        gic.gic_drag(ctx, s["Rs"], s["Vs"], uat, af, Fd)
        gic.gic_contact_forces(ctx, s["Xs"], s["Vs"], s["Rs"], *cells, Fc, pair_ids=pairs)  # from the list
        x2, v2, r2 = (torch.full_like(s[k], -1.0) for k in ("Xs", "Vs", "Rs"))
        f2, u2, a2, c2 = e(3 * n), e(3 * n), e(n), e(3 * n)
        gic.gic_gather_g2p_drag(ctx, s["order"], s["X"], s["V"], s["R"], None, x2, v2, r2, None, s["U"], A, *cells,
                                f2, u2, a2)
        assert all(torch.equal(p, q) for p, q in ((x2, s["Xs"]), (v2, s["Vs"]), (r2, s["Rs"]), (u2, uat), (a2, af),
                                                  (f2, Fd))), call
        gic.gic_gather_g2p_fluid(ctx, s["order"], s["X"], s["V"], s["R"], None, x2, v2, r2, None, s["U"], A, *cells, f2)
        assert torch.equal(f2, Fd)
        gic.gic_contact_forces(ctx, s["Xs"], s["Vs"], s["Rs"], *cells, c2)
        assert torch.equal(c2, Fc), call
        x3, v3 = s["Xs"].clone(), s["Vs"].clone()
        gic.gic_integrate(ctx, s["Rs"], Fc, Fd, x3, v3)
        A3, M3 = torch.empty_like(A), torch.empty_like(M)
        gic.gic_p2g(ctx, x3, v3, s["Rs"], *cells, A3, M3)
        x4, v4, A4, M4 = s["Xs"].clone(), s["Vs"].clone(), torch.empty_like(A), torch.empty_like(M)
        gic.gic_integrate_p2g(ctx, x4, v4, s["Rs"], Fc, Fd, *cells, A4, M4)
        assert torch.equal(x3, x4) and torch.equal(v3, v4) and torch.equal(A3, A4) and torch.equal(M3, M4)
    assert (Fc != 0).any() and ctx.error()[0] in (0, 4)
    a3, m3 = orc.p2g_fixed(cfg, x3.view(3, n).cpu().numpy(), v3.view(3, n).cpu().numpy(), s["Rs"].cpu().numpy())
    assert np.array_equal(A3.cpu().numpy(), a3) and np.array_equal(M3.view(3, -1).cpu().numpy(), m3)


def test_sparse_bed_steps(G, orc):
    """gic_step (tiles stored by the per-granule P2G, escapes, assembly) gives
    the oracle's P2G of its own state after every step."""
    from paper_2504_00745_amd import gic
    cfg, x, v, r, u = bed((41, 43, 41))
    sim = gic.Simulator(cfg, x, 0.2 * v, r, u, "fp32", r_max=1.5e-3)
    for k in range(4):
        sim.step()
        c = {a: t.cpu().numpy() for a, t in sim.cur.items()}
        a, m = orc.p2g_fixed(cfg, c["x"].reshape(3, -1), c["v"].reshape(3, -1), c["r"])
        assert np.array_equal(sim.alpha.cpu().numpy(), a), k
        assert np.array_equal(sim.mom.view(3, -1).cpu().numpy(), m), k
        G.say(f"[sparse] step {k} ok")


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_sparse_wet_bed(G, orc, prec):
    """The capillary form of the wave kernel against the oracle's contact plus
    bridge forces on sampled granules, to the bar of the wet-bed tests (1e-5 /
    1e-12 of the summed term magnitudes)."""
    import torch
    from paper_2504_00745_amd import gic
    cfg, x, v, r, u = bed((41, 43, 41))
    cfg.update(sigma=0.072, vbridge=1e-4, sr_peak=0.3)
    s = setup(G, gic, cfg, x, v, r, u, prec, r_max=1.44e-3)
    ctx, n = s["ctx"], s["n"]
    rng = np.random.Generator(np.random.PCG64(8))
    sr = rng.uniform(0.0, 1.0, n).astype(np.float32).astype(np.float64)
    SR = G.dev(sr, ctx.real)[s["order"].long()].contiguous()
    F = torch.empty(3 * n, dtype=ctx.real, device="cuda")
    pos = np.empty(n, np.int64)
    pos[s["order"].cpu().numpy()] = np.arange(n)
    clump = np.nonzero(r == 1.003e-3)[0]
    idx = np.concatenate([rng.choice(n, 3000, replace=False), clump])
    Fs, fa = orc.contact_forces_sample(cfg, x, v, r, idx)
    Fb, fb = orc.capillary_forces_sample(cfg, x, r, sr, idx)
    assert (fb > 0).sum() > 200 and (fa > 0).sum() > 200
    for call in range(3):
        gic.gic_contact_capillary_forces(ctx, s["Xs"], s["Vs"], s["Rs"], SR, s["cb"], s["ce"], F)
        torch.cuda.synchronize()
        err = np.linalg.norm(F.view(3, n).double().cpu().numpy()[:, pos[idx]] - (Fs + Fb), axis=0)
        tol = 1e-5 if prec == "fp32" else 1e-12
        assert np.all(err <= tol * (fa + fb) + 1e-300), (call, np.max(err / (fa + fb + 1e-300)))
