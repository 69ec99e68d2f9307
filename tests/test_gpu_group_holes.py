"""Kernels over groups of 2x2x2 bricks on beds whose groups begin with empty
bricks: the lowest brick layer (z) or the first brick row (y) of the box empty,
or a quarter of the bricks, at random, removed.  The begin of an empty brick's cells is
the next granule's position, which may be a later brick's of the same group.

References: the kernels that run a thread per granule without bricks (reorder,
G2P, drag, the contact from the neighbour list, integrate); every comparison is
bit for bit, outputs filled beforehand with a value that no result takes."""
import numpy as np
import pytest

from test_gpu_brick_groups import G, bed  # noqa: F401 (G: a fixture)

pytestmark = pytest.mark.gpu


def shifted(dims, keep, where, seed=4):
    """bed() moved up by one brick along the axis `where`, or with a quarter of its
    bricks emptied."""
    cfg, x, v, r, _ = bed(dims, keep, seed)
    rng = np.random.Generator(np.random.PCG64(seed + 100))
    nc, sp = list(cfg["nc"]), cfg["cell"]
    if where == "holes":
        b = np.floor(x / (4 * sp)).astype(int)
        nb = [(m + 3) // 4 for m in nc]
        keep_b = rng.random(nb) < 0.75
        keep_b[0, 0, 0] = False
        k = keep_b[b[0], b[1], b[2]]
        x, v, r = np.ascontiguousarray(x[:, k]), np.ascontiguousarray(v[:, k]), np.ascontiguousarray(r[k])
    else:
        x = x.copy()
        x[where] += 4 * sp
        nc[where] += 4
    cfg = dict(cfg, nc=nc, n=list(nc))
    return cfg, x, v, r, rng.normal(0.0, 0.1, (3, int(np.prod(nc))))


BIG, BIGGER = (105, 102, 107), (145, 142, 147)  # 18,954 bricks; 49,284, a quarter of them emptied


@pytest.mark.parametrize("prec,dims,keep,where", [("fp32", (67, 66, 69), 0.9, 2), ("fp32", BIG, 0.2, 2), ("fp32", BIG, 0.2, 1),
                                                  ("fp64", BIG, 0.2, 2), ("fp64", BIG, 0.2, 1), ("fp32", BIG, 0.2, 0),
                                                  ("fp32", BIGGER, 0.2, "holes"), ("fp64", BIGGER, 0.2, "holes")])
def test_gathers_and_contact(G, prec, dims, keep, where):  # noqa: F811
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[group holes] {prec} {dims} {where}")
    cfg, x, v, r, u = shifted(dims, keep, where)
    n = x.shape[1]
    ctx = gic.Context(cfg, n, prec, r_max=1.5e-3)
    e = lambda m, t=ctx.real: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    i32 = torch.int32
    X, V, R, U = G.dev(x), G.dev(v), G.dev(r), G.dev(u, ctx.real)
    ID = torch.arange(n, dtype=i32, device="cuda")
    key, order, cb, ce = e(n, i32), e(n, i32), e(ctx.K, i32), e(ctx.K, i32)
    Xs, Vs, Rs, IDs = (torch.empty_like(t) for t in (X, V, R, ID))
    for _ in range(2):  # the second call's kernels see the count of bricks
        gic.gic_sort_cells(ctx, X, key, order, cb, ce)
        torch.cuda.synchronize()
    occupied = int((ce.view(-1, 64)[:, 63] > cb.view(-1, 64)[:, 0]).sum())
    held = int((torch.nn.functional.max_pool3d(((ce.view(-1, 64)[:, 63] > cb.view(-1, 64)[:, 0]).float()
                                                .view(1, 1, *((m + 3) // 4 for m in cfg["nc"][::-1]))), 2, ceil_mode=True)).sum())
    # the group forms are taken
    assert occupied >= (4096 if prec == "fp32" else 16384) and n <= 80 * occupied and occupied >= 5 * held
    gic.gic_reorder(ctx, order, X, V, R, ID, Xs, Vs, Rs, IDs)
    A, M = e(ctx.G, torch.int64), e(3 * ctx.G, torch.int64)
    gic.gic_p2g(ctx, Xs, Vs, Rs, cb, ce, A, M)
    uat, af, Fd, Fc = e(3 * n), e(n), e(3 * n), e(3 * n)
    gic.gic_g2p(ctx, Xs, U, A, None, uat, af)
    gic.gic_drag(ctx, Rs, Vs, uat, af, Fd)
    gic.gic_contact_forces(ctx, Xs, Vs, Rs, cb, ce, Fc, pair_ids=e(48 * n, i32))  # from the list
    H = torch.rand(n, dtype=torch.float64, device="cuda")

    def fresh():
        return [torch.full_like(t, -7) for t in (Xs, Vs, Rs, IDs, Fd, uat, af, H)]

    x2, v2, r2, i2, f2, u2, a2, h2 = fresh()
    gic.gic_gather_g2p_drag(ctx, order, X, V, R, ID, x2, v2, r2, i2, U, A, cb, ce, f2, u2, a2)
    for p, q in ((x2, Xs), (v2, Vs), (r2, Rs), (i2, IDs), (u2, uat), (a2, af), (f2, Fd)):
        assert torch.equal(p, q), int((p != q).sum())
    x2, v2, r2, i2, f2, u2, a2, h2 = fresh()
    gic.gic_gather_g2p_fluid(ctx, order, X, V, R, ID, x2, v2, r2, i2, U, A, cb, ce, f2, held=H, held_out=h2)
    for p, q in ((x2, Xs), (v2, Vs), (r2, Rs), (i2, IDs), (f2, Fd), (h2, H[order.long()])):
        assert torch.equal(p, q), int((p != q).sum())
    c2 = torch.full_like(Fc, -7.0)
    gic.gic_contact_forces(ctx, Xs, Vs, Rs, cb, ce, c2)
    assert torch.equal(c2, Fc) and bool((Fc != 0).any())


@pytest.mark.parametrize("prec,dims,keep,where", [("fp32", (67, 66, 69), 0.9, 2), ("fp32", BIG, 0.2, 1), ("fp64", BIG, 0.2, 1),
                                                  ("fp64", BIGGER, 0.2, "holes")])
def test_steps_match_stages(G, prec, dims, keep, where):  # noqa: F811
    """gic_step against the per-granule stages, from the same state, step by
    step: x, v, r, id and both grids."""
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[group holes] steps {prec} {dims} {where}")
    cfg, x, v, r, u = shifted(dims, keep, where)
    n = x.shape[1]
    sim = gic.Simulator(cfg, x, v, r, u, prec, r_max=1.5e-3)
    ctx = gic.Context(cfg, n, prec, r_max=1.5e-3)  # the reference's own
    e = lambda m, t=ctx.real: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    i32 = torch.int32
    key, order, cb, ce = e(n, i32), e(n, i32), e(ctx.K, i32), e(ctx.K, i32)
    uat, af, Fd, Fc = e(3 * n), e(n), e(3 * n), e(3 * n)
    A, M = e(ctx.G, torch.int64), e(3 * ctx.G, torch.int64)
    torch.cuda.synchronize()
    for step in range(3):
        c = {k: t.clone() for k, t in sim.cur.items()}
        alpha = sim.alpha.clone()
        for t in sim.nxt.values():
            t.fill_(-7)
        sim.step()
        s = {k: torch.empty_like(t) for k, t in c.items()}
        gic.gic_sort_cells(ctx, c["x"], key, order, cb, ce)
        gic.gic_reorder(ctx, order, c["x"], c["v"], c["r"], c["id"], s["x"], s["v"], s["r"], s["id"])
        gic.gic_g2p(ctx, s["x"], sim.u, alpha, None, uat, af)
        gic.gic_drag(ctx, s["r"], s["v"], uat, af, Fd)
        gic.gic_contact_forces(ctx, s["x"], s["v"], s["r"], cb, ce, Fc, pair_ids=e(48 * n, i32))
        gic.gic_integrate(ctx, s["r"], Fc, Fd, s["x"], s["v"])
        gic.gic_p2g(ctx, s["x"], s["v"], s["r"], cb, ce, A, M)
        for k in ("x", "v", "r", "id"):
            assert torch.equal(sim.cur[k], s[k]), (step, k, int((sim.cur[k] != s[k]).sum()))
        assert torch.equal(sim.alpha, A) and torch.equal(sim.mom, M), step
    ids = torch.sort(sim.cur["id"])[0]
    assert torch.equal(ids, torch.arange(n, dtype=i32, device="cuda"))
