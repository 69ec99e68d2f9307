"""Sorts by digit passes: dense cells, large shuffled beds, keys of one to four
digits, changes between sorts, and the switch to and from the counting sort once
the record of a sort has reached the host; against numpy's stable argsort of the
oracle's keys and its ranges, bit for bit.  And the rollout's step on a bed that
takes them, against the stages."""
import numpy as np
import pytest

from test_gpu_sort_paths import G, check, config  # noqa: F401 (G: a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,n,box", [((4, 4, 4), 9, 4), ((4, 4, 4), 60001, 4), ((12, 12, 12), 300007, 12), ((44, 44, 44), 270001, 8),
                                      ((100, 30, 20), 524289, 100), ((257, 260, 264), 524309, 257), ((60, 61, 62), 1048577, 4)])
def test_digit_passes(G, orc, nc, n, box):  # noqa: F811
    """box: edge of the part of the box that holds the granules (a small part of a
    large box becomes known to be dense after the first sorts only)."""
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[sort digits] {nc} {n} {box}")
    rng = np.random.Generator(np.random.PCG64(n))
    cfg = config(nc)
    edge = np.minimum(np.array(nc, float), box)[:, None]
    ctx = gic.Context(cfg, n, "fp64", r_max=0.5)
    buf = [torch.empty(m, dtype=torch.int32, device="cuda") for m in (n, n, ctx.K, ctx.K)]
    for _ in range(3):  # other beds of the same number: shuffled each time
        x = rng.random((3, n)) * edge
        check(G, gic, orc, cfg, ctx, x, buf)
    y = x[:, buf[1].cpu().numpy()]
    for moved in (0, 1, 4096, 4097, n // 10):  # sorted, a few changes, many
        if moved > n:
            continue
        y = y.copy()
        sel = rng.choice(n, moved, replace=False)
        y[:, sel] = rng.random((3, moved)) * edge
        check(G, gic, orc, cfg, ctx, y, buf)
        y = y[:, buf[1].cpu().numpy()]
    for _ in range(17):  # until the next record
        gic.gic_sort_cells(ctx, G.dev(y), *buf)
    x = rng.random((3, n)) * np.array(nc, float)[:, None]  # spread over the whole box
    check(G, gic, orc, cfg, ctx, x, buf)
    check(G, gic, orc, cfg, ctx, y, buf)


@pytest.mark.parametrize("n,dense", [(20000, True), (524291, False), (1048579, False)])
def test_rollout_step(G, n, dense):  # noqa: F811
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[sort digits] rollout {n}")
    rng = np.random.Generator(np.random.PCG64(n))
    m = 3 if dense else int(np.ceil(n ** (1 / 3)))  # dense: 740 granules a cell
    cfg = dict(config((m + 1,) * 3), kn=1.0, dt=1e-6, g=[0.0, 0.0, -9.81])
    x = rng.random((3, n)) * m
    r = np.full(n, 0.01) * rng.uniform(0.5, 1.0, n)
    c = gic.Context(cfg, n, "fp64", r_max=0.01)
    e = lambda k, t=torch.float64: torch.empty(k, dtype=t, device="cuda")  # noqa: E731
    i32 = torch.int32
    xv = torch.cat([G.dev(x).reshape(-1), G.dev(rng.normal(0, 1, 3 * n))])
    r, u = G.dev(r), G.dev(rng.normal(0, 0.1, 3 * c.G))
    key, order, cb, ce = e(n, i32), e(n, i32), e(c.K, i32), e(c.K, i32)
    xvs, rs = e(6 * n), e(n)
    A, uat, af, Fd, Fc = e(c.G), e(3 * n), e(n), e(3 * n), e(3 * n)
    d = gic.Context(cfg, n, "fp64", r_max=0.01)
    xs, vs = xvs[:3 * n].view(3, n), xvs[3 * n:]
    gic.gic_sort_cells(d, xv[:3 * n].view(3, n), key, order, cb, ce)
    gic.gic_reorder(d, order, xv[:3 * n].view(3, n), xv[3 * n:], r, None, xs, vs, rs, None)
    gic.gic_p2g_real(d, xs, vs, rs, cb, ce, A, None)
    gic.gic_g2p(d, xs, u, None, A, uat, af)
    gic.gic_drag(d, rs, vs, uat, af, Fd)
    gic.gic_contact_forces(d, xs, vs, rs, cb, ce, Fc, pair_ids=e(64 * n, i32))
    gic.gic_integrate(d, rs, Fc, Fd, xs, vs)
    want = e(6 * n)
    gic.gic_permute(d, order, xvs, want, 6, True)
    for call in range(4):
        out, g = torch.full_like(xv, -1.0), torch.ones_like(xv)
        gic.gic_rollout_step(c, xv, r, u, out, key, order, cb, ce, xvs, rs)
        assert torch.equal(out, want), call
        gic.gic_rollout_step_vjp(c, xv, r, u, g, e(1).fill_(0.0), e(1).fill_(0.0), key, order, cb, ce, xvs, rs, e(6 * n),
                                 e(3 * n), e(n))
        torch.cuda.synchronize()
        if call:
            assert torch.equal(g, last), call
        last = g
    assert bool((Fc != 0).any()) and c.error()[0] == 0


@pytest.mark.parametrize("n,m", [(262144, 65536), (100003, 30000)])
def test_one_long_cell_among_short_ones(G, orc, n, m):  # noqa: F811
    """A cell of m of the n granules, the rest some eight a cell: bit for bit, and,
    once the record of the first sort has reached the host, not at the pace of the
    one workgroup that puts a cell in order (18 us for every 1,024 granules; a sort of
    as many granules spread evenly takes some 35 us, the digit passes some 65)."""
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[sort digits] long cell {n} {m}")
    rng = np.random.Generator(np.random.PCG64(n))
    nc = (int(np.ceil((n / 8) ** (1 / 3))),) * 3
    cfg = config(nc)
    x = rng.random((3, n)) * np.array(nc, float)[:, None]
    x[:, rng.choice(n, m, replace=False)] = rng.random((3, m)) * 0.9 + 0.05
    ctx = gic.Context(cfg, n, "fp64", r_max=0.5)
    buf = [torch.empty(k, dtype=torch.int32, device="cuda") for k in (n, n, ctx.K, ctx.K)]
    for _ in range(2):
        check(G, gic, orc, cfg, ctx, x, buf)
    y = G.dev(x)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    for _ in range(5):
        a.record()
        for _ in range(4):
            gic.gic_sort_cells(ctx, y, *buf)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / 4 * 1e3)
    G.say(f"[sort digits] us {min(times):.1f}")
    assert min(times) < 18.0 * m / 1024 / 2  # half the time of the one workgroup


def test_sorts_among_brick_lists(G, orc):  # noqa: F811
    """Stage calls whose brick lists come between the sorts: the sorts are sampled all
    the same, so a long cell is known (see above), also where a list of the same number
    of granules came first."""
    import torch
    from paper_2504_00745_amd import gic
    n, m = 262144, 65536
    G.say("[sort digits] lists between")
    rng = np.random.Generator(np.random.PCG64(3))
    cfg = dict(config((96,) * 3), kn=1.0)  # more bricks than a call takes without a list
    x = rng.random((3, n)) * 96.0
    x[:, rng.choice(n, m, replace=False)] = rng.random((3, m)) * 0.9 + 0.05
    e = lambda k, t=torch.int32: torch.empty(k, dtype=t, device="cuda")  # noqa: E731
    other = gic.Context(cfg, n, "fp64", r_max=0.5)
    tab = [e(n), e(n), e(other.K), e(other.K)]
    gic.gic_sort_cells(other, G.dev(x), *tab)
    f64 = torch.float64
    xs, r = G.dev(x)[:, tab[1].long()].contiguous(), torch.full((n,), 1e-3, dtype=f64, device="cuda")
    ctx = gic.Context(cfg, n, "fp64", r_max=0.5)
    buf = [e(n), e(n), e(ctx.K), e(ctx.K)]
    y, A = G.dev(x), e(ctx.G, torch.int64)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    for k in range(6):
        gic.gic_p2g(ctx, xs, None, r, tab[2], tab[3], A, None)  # builds a list
        a.record()
        gic.gic_sort_cells(ctx, y, *buf)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    assert all(torch.equal(p, q) for p, q in zip(tab, buf))
    G.say(f"[sort digits] us {times}")
    assert min(times[2:]) < 18.0 * m / 1024 / 2
