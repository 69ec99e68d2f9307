"""The counting sort at the edges of its paths, against numpy's stable argsort
of the oracle's keys and its searchsorted ranges, bit for bit: tables of one
and of two scan passes (32,768 cells and just beyond), cells at and beyond the
size that a workgroup sorts by digits (256), all granules in one cell, and
second sorts on the context with no, few (merged) and many (counted again)
changed keys on both sides of the size from which changes are collected
(2^18)."""
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


def config(nc):
    return dict(kn=1e5, restitution=0.5, kt_ratio=1.0, mu=0.5, rho_s=2500.0, eta_f=1e-3, c_drag=1.0, alpha_max=0.74,
                walls=0, n=list(nc), dx=1.0, nc=list(nc), cell=1.0, dt=1e-5, g=[0.0, 0.0, 0.0])


def check(G, gic, orc, cfg, ctx, x, buf):
    n = x.shape[1]
    key, order, cb, ce = buf
    gic.gic_sort_cells(ctx, G.dev(x), key, order, cb, ce)
    k = orc.cell_keys(cfg, x)
    want = np.argsort(k, kind="stable")
    assert np.array_equal(key.cpu().numpy().view(np.uint32), k)
    assert np.array_equal(order.cpu().numpy(), want)
    cells = np.arange(ctx.K, dtype=np.uint64)
    assert np.array_equal(cb.cpu().numpy(), np.searchsorted(k[want], cells, side="left"))
    assert np.array_equal(ce.cpu().numpy(), np.searchsorted(k[want], cells, side="right"))
    assert ctx.error() == (0, -1)


@pytest.mark.parametrize("nc", [(4, 4, 4), (32, 32, 32), (36, 32, 32), (7, 61, 33)])
@pytest.mark.parametrize("n,bed", [(1000, "uniform"), (70001, "uniform"), (70001, "one"), (2570, "long"),
                                   (300007, "uniform"), (300007, "one"), (262144, "uniform")])
def test_counting_sort(G, orc, nc, n, bed):
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[sort] {nc} {n} {bed}")
    rng = np.random.Generator(np.random.PCG64(n))
    box = np.array(nc, float)[:, None]
    x = rng.random((3, n)) * box
    if bed == "one":
        x = np.floor(box / 2) + 0.9 * rng.random((3, n))
    if bed == "long":  # cells of 255, 256, 257, 258 and 1,544 granules, interleaved
        cell = rng.permutation(np.repeat(np.arange(5), [255, 256, 257, 258, 1544]))
        x = rng.random((3, n)) * 0.9
        x[0] += cell % 4
        x[1] += cell // 4
    ctx = gic.Context(config(nc), n, "fp64", r_max=0.5)
    cfg = config(nc)
    buf = [torch.empty(m, dtype=torch.int32, device="cuda") for m in (n, n, ctx.K, ctx.K)]
    check(G, gic, orc, cfg, ctx, x, buf)
    y = x[:, buf[1].cpu().numpy()]  # sorted: no key changes
    check(G, gic, orc, cfg, ctx, y, buf)
    check(G, gic, orc, cfg, ctx, y, buf)
    for moved in (1, 37, 4096, 4097):
        if moved > n:
            break
        y = y.copy()
        sel = rng.choice(n, moved, replace=False)
        y[:, sel] = rng.random((3, moved)) * box
        check(G, gic, orc, cfg, ctx, y, buf)
        y = y[:, buf[1].cpu().numpy()]


def test_steps_keep_and_rebuild_ranges(G, orc):
    """Stepping calls: steps without a changed key keep the tables, a granule
    moved in place across cells (small and large beds) renews them."""
    import torch
    from paper_2504_00745_amd import gic
    for n in (5000, 270001):
        rng = np.random.Generator(np.random.PCG64(n))
        m = int(np.ceil(n ** (1 / 3)))
        cfg = dict(config((m + 1,) * 3), kn=1.0, dt=1e-9)
        g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij")).reshape(3, -1)[:, :n] + 0.5
        x = g + rng.uniform(-0.2, 0.2, g.shape)
        u = np.zeros((3, int(np.prod(cfg["n"]))))
        sim = gic.Simulator(cfg, x, np.zeros_like(x), np.full(n, 0.2), u, "fp64", r_max=0.2)
        for k in range(6):
            if k in (3, 5):
                sim.cur["x"][0, 17 * k] += 1.0
            before = sim.cur["x"].cpu().numpy()
            sim.step()
            key = orc.cell_keys(cfg, before)
            want = np.argsort(key, kind="stable")
            assert np.array_equal(sim.scratch["order"].cpu().numpy(), want), (n, k)
            cells = np.arange(sim.ctx.K, dtype=np.uint64)
            assert np.array_equal(sim.scratch["cell_begin"].cpu().numpy(),
                                  np.searchsorted(key[want], cells, side="left")), (n, k)
            assert np.array_equal(sim.scratch["cell_end"].cpu().numpy(),
                                  np.searchsorted(key[want], cells, side="right")), (n, k)
            assert torch.equal(sim.cur["x"].cpu(), torch.as_tensor(before[:, want] + 1e-9 * sim.cur["v"].cpu().numpy()))
