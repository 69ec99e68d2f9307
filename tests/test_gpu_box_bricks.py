"""Stage calls that take every brick of the box against the same calls over a
kept list of the occupied ones, bit for bit: one brick, boxes whose bricks do
not fill the XCDs' runs, a box most of which is empty."""
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


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nc,filled", [((4, 4, 4), 1.0), ((20, 21, 24), 1.0), ((64, 61, 100), 0.3), ((128, 61, 65), 1.0)])
def test_box_matches_list(G, prec, nc, filled):
    import torch
    from paper_2504_00745_amd import gic
    G.say(f"[box] {nc} {prec}")
    cell = 0.004
    rng = np.random.Generator(np.random.PCG64(11))
    n = max(40, int(0.6 * np.prod(nc) * filled))
    L = np.array(nc)[:, None] * cell
    x = (0.02 + 0.96 * rng.random((3, n))) * L
    x[2] *= filled
    r = rng.uniform(0.8e-3, 1.5e-3, n)
    cfg = dict(kn=1e5, restitution=0.5, kt_ratio=1.0, mu=0.5, rho_s=2500.0, eta_f=1e-3, c_drag=1.0, alpha_max=0.74,
               walls=0x3F, n=list(nc), dx=cell, nc=list(nc), cell=cell, dt=1e-6, g=[0.0, 0.0, -9.81])
    ctx = gic.Context(cfg, n, prec, r_max=1.5e-3)
    e = lambda m, t=ctx.real: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    i32, i64 = torch.int32, torch.int64
    X, V, R = G.dev(x), G.dev(rng.normal(0, 0.1, x.shape)), G.dev(r)
    U = G.dev(rng.normal(0, 0.1, (3, ctx.G)), ctx.real)
    key, order, cb, ce = e(n, i32), e(n, i32), e(ctx.K, i32), e(ctx.K, i32)

    def stages():
        xs, vs, rs = torch.empty_like(X), torch.empty_like(V), torch.empty_like(R)
        A, M, A2, M2 = e(ctx.G, i64), e(3 * ctx.G, i64), e(ctx.G, i64), e(3 * ctx.G, i64)
        Fd, Fc, ar = e(3 * n), e(3 * n), e(ctx.G, torch.float64)
        gic.gic_gather_g2p_drag(ctx, order, X, V, R, None, xs, vs, rs, None, U, A0, cb, ce, Fd, None, None)
        gic.gic_p2g(ctx, xs, vs, rs, cb, ce, A, M)
        gic.gic_contact_forces(ctx, xs, vs, rs, cb, ce, Fc)
        gic.gic_p2g_real(ctx, xs, vs, rs, cb, ce, ar, None)
        out = [xs.clone(), vs.clone(), rs, A, M, Fd, Fc, ar]
        gic.gic_integrate_p2g(ctx, xs, vs, rs, Fc, Fd, cb, ce, A2, M2)
        return out + [xs, vs, A2, M2]

    A0 = torch.zeros(ctx.G, dtype=i64, device="cuda")
    for _ in range(2):
        gic.gic_sort_cells(ctx, X, key, order, cb, ce)
        torch.cuda.synchronize()  # the count of occupied bricks has reached the host
    box = stages()
    gic.gic_brick_list(ctx, cb, ce)
    kept = stages()
    assert all(torch.equal(a, b) for a, b in zip(box, kept))
    assert int((kept[3] != 0).sum()) > 0 and (n < 1000 or bool((kept[6] != 0).any()))
