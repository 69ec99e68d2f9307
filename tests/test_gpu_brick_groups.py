"""Kernels over groups of 2x2x2 bricks (gather, direct contact, P2G and the
assembly of its tiles), taken for sparse beds of many bricks once their count
has reached the host: a fifth of a jittered lattice in a box of an odd number of
bricks along two axes (groups that reach outside it), half of the box empty, a
clump whose shell overflows the group's LDS array.

References: the kernels that run a thread per granule without bricks (G2P, drag,
the contact from the neighbour list, integrate) and the oracle's integer P2G;
every comparison is bit for bit."""
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


def bed(dims, keep, seed=4, dx=0.003):
    """keep: share of the lattice sites that hold a granule."""
    rng = np.random.Generator(np.random.PCG64(seed))
    sp = 0.003
    g = np.stack(np.meshgrid(*[np.arange(m) for m in dims], indexing="ij")).reshape(3, -1).astype(float)
    g = g[:, rng.random(g.shape[1]) < keep]
    r = rng.uniform(0.9e-3, 1.5e-3, g.shape[1])
    x = (g + 0.5) * sp + rng.uniform(-1, 1, g.shape) * 0.4e-3
    # a clump of 16^3 granules over the cells 20 .. 25 (more than a group's shell array holds)
    lo = 20 * sp
    inside = np.all((x > lo) & (x < lo + 6 * sp), axis=0)
    h = np.stack(np.meshgrid(*[np.arange(16)] * 3, indexing="ij")).reshape(3, -1)
    y = lo + (h + 0.5) * (6 * sp / 16) + rng.uniform(-1e-5, 1e-5, h.shape)
    x, r = np.concatenate([x[:, ~inside], y], axis=1), np.concatenate([r[~inside], np.full(4096, 0.57e-3)])
    p = rng.permutation(x.shape[1])
    x, r = np.ascontiguousarray(x[:, p]), np.ascontiguousarray(r[p])
    nc = [dims[0], dims[1], dims[2] + 40]
    n = [int(np.ceil(m * sp / dx - 1e-9)) for m in nc]
    cfg = dict(kn=1e5, restitution=0.5, kt_ratio=1.0, mu=0.5, rho_s=2500.0, eta_f=1e-3, c_drag=1.0, alpha_max=0.74,
               walls=0x3F, n=n, dx=dx, nc=nc, cell=sp, dt=2e-5, g=[0.0, 0.0, -9.81])
    v = rng.normal(0.0, 5.0, x.shape)  # some stencils leave their group's tile in one move
    u = rng.normal(0.0, 0.1, (3, int(np.prod(n))))
    return cfg, x, v, r, u


@pytest.mark.parametrize("prec,dims,keep,dx", [("fp32", (105, 102, 107), 0.2, 0.003), ("fp64", (105, 102, 107), 0.2, 0.003),
                                               ("fp32", (67, 66, 69), 0.9, 0.003), ("fp32", (105, 102, 107), 0.2, 0.004)])
def test_groups_match_per_granule_kernels(G, orc, prec, dims, keep, dx):
    """The smaller bed takes groups for the node tiles and waves for the
    contact; at dx = 4 mm a brick holds 3 nodes per edge."""
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[groups] {dims} {prec} {dx}")
    cfg, x, v, r, u = bed(dims, keep, dx=dx)
    n = x.shape[1]
    r_max = 1.5e-3
    ctx = gic.Context(cfg, n, prec, r_max=r_max)
    e = lambda m, t=ctx.real: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    i32 = torch.int32
    X, V, R, U = G.dev(x), G.dev(v), G.dev(r), G.dev(u, ctx.real)
    key, order, cb, ce = e(n, i32), e(n, i32), e(ctx.K, i32), e(ctx.K, i32)
    Xs, Vs, Rs = torch.empty_like(X), torch.empty_like(V), torch.empty_like(R)
    for _ in range(2):  # the second call's kernels see the count of bricks
        gic.gic_sort_cells(ctx, X, key, order, cb, ce)
        torch.cuda.synchronize()
    gic.gic_reorder(ctx, order, X, V, R, None, Xs, Vs, Rs, None)
    A, M = e(ctx.G, torch.int64), e(3 * ctx.G, torch.int64)
    gic.gic_p2g(ctx, Xs, Vs, Rs, cb, ce, A, M)
    uat, af, Fd, Fc = e(3 * n), e(n), e(3 * n), e(3 * n)
    gic.gic_g2p(ctx, Xs, U, A, None, uat, af)
    gic.gic_drag(ctx, Rs, Vs, uat, af, Fd)
    gic.gic_contact_forces(ctx, Xs, Vs, Rs, cb, ce, Fc, pair_ids=e(48 * n, i32))  # from the list
    for call in range(3):
        x2, v2, r2 = (torch.full_like(t, -1.0) for t in (Xs, Vs, Rs))
        f2, u2, a2, c2 = e(3 * n), e(3 * n), e(n), e(3 * n)
        gic.gic_gather_g2p_drag(ctx, order, X, V, R, None, x2, v2, r2, None, U, A, cb, ce, f2, u2, a2)
        for p, q in ((x2, Xs), (v2, Vs), (r2, Rs), (u2, uat), (a2, af), (f2, Fd)):
            assert torch.equal(p, q), call
        gic.gic_gather_g2p_fluid(ctx, order, X, V, R, None, x2, v2, r2, None, U, A, cb, ce, f2)
        assert torch.equal(f2, Fd), call
        gic.gic_contact_forces(ctx, Xs, Vs, Rs, cb, ce, c2)
        torch.cuda.synchronize()
        assert torch.equal(c2, Fc), call
    assert (Fc != 0).any()


@pytest.mark.parametrize("prec,dims,keep,dx", [("fp32", (105, 102, 107), 0.2, 0.003), ("fp64", (67, 66, 69), 0.9, 0.003),
                                               ("fp32", (105, 102, 107), 0.2, 0.004)])
def test_group_tiles_assemble(G, orc, prec, dims, keep, dx):
    """gic_step: tiles of groups from the second step on, escapes, segments that
    the bed leaves; the grids are the oracle's P2G of the stepped state."""
    import torch
    from paper_2504_00745_amd import gic
    cfg, x, v, r, u = bed(dims, keep, dx=dx)
    sim = gic.Simulator(cfg, x, v, r, u, prec, r_max=1.5e-3)
    for k in range(4):
        sim.step()
        torch.cuda.synchronize()
        c = {a: t.cpu().numpy() for a, t in sim.cur.items()}
        a, m = orc.p2g_fixed(cfg, c["x"].reshape(3, -1), c["v"].reshape(3, -1), c["r"])
        assert np.array_equal(sim.alpha.cpu().numpy(), a), k
        assert np.array_equal(sim.mom.view(3, -1).cpu().numpy(), m), k
        G.say(f"[groups] step {k} ok")
