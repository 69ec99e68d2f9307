"""The rollout's one-call step and its reverse against the stages they stand
for, called one by one on the same state: the step bit for bit, the adjoint to
1e-11 of its largest component (the pair terms of a granule and the 27 node
terms are added in another order, a few units of 2^-53 of terms that are at most
some hundred times the sum).  Beds: a moving bidisperse bed, the same with a
cell of more than 256 granules (its order is sorted by digits and its brick's
shell overflows the LDS array), a bed past the size from which one wave runs a
brick, a single granule."""
import numpy as np
import pytest

from paper_2504_00745_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_00745_amd import gic
    gic.lib()
    import gpu_util
    return gpu_util


def bed(name):
    if name == "sparse":
        rng = np.random.Generator(np.random.PCG64(5))
        g = np.stack(np.meshgrid(np.arange(41), np.arange(42), np.arange(43), indexing="ij")).reshape(3, -1)
        r = rng.uniform(0.75e-3, 1.5e-3, g.shape[1])
        x = (g + 0.5) * 3e-3 + rng.uniform(-1, 1, g.shape) * np.maximum(1.5e-3 - r / 1.03, 0)
        p = wl._params([45, 45, 45], 3e-3, 3e-3, 1e-6, (0.0, 0.0, -9.81), c_drag=1000.0)
        d = dict(params=p, x=x, v=rng.normal(0, 0.5, x.shape), r=r, u=rng.normal(0, 0.1, (3, 45 ** 3)))
        q = rng.permutation(x.shape[1])
        return dict(d, x=np.ascontiguousarray(x[:, q]), v=d["v"], r=r[q])
    d = wl.make("c4", n_override=1 if name == "one" else 4099)
    d["v"] = 20.0 * d["v"]
    if name.startswith("fine"):  # node tiles of 11^3 (beyond four a thread) and 13^3 (beyond LDS)
        p = dict(d["params"])
        dx = p["cell"] / (1.9 if name == "fine" else 2.5)
        n = [int(np.ceil(m * p["dx"] / dx)) for m in p["n"]]
        p.update(dx=dx, n=n)
        d.update(params=p, u=np.random.Generator(np.random.PCG64(7)).normal(0, 0.1, (3, int(np.prod(n)))))
    if name == "dense":  # 300 granules in one cell, the rest as they were
        rng = np.random.Generator(np.random.PCG64(6))
        x, r = d["x"].copy(), d["r"].copy()
        x[:, :300] = 0.2 + 0.012 * rng.random((3, 300))
        r[:300] = 0.0004
        d.update(x=x, r=r)
    return d


@pytest.mark.parametrize("name", ["bidisperse", "dense", "sparse", "one", "fine", "finer"])
def test_step_and_reverse_match_stages(T, name):
    import torch
    from paper_2504_00745_amd import gic
    T.say(f"[rollout step] {name}")
    d = bed(name)
    cfg, n = d["params"], d["x"].shape[1]
    c = gic.Context(cfg, n, "fp64", r_max=max(float(d["r"].max()), 0.4 * cfg["cell"]) if name != "sparse" else 1.5e-3)
    e = lambda m, t=torch.float64: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    i32 = torch.int32
    xv = torch.cat([T.dev(d["x"]).reshape(-1), T.dev(d["v"]).reshape(-1)])
    r, u = T.dev(d["r"]), T.dev(d["u"]).reshape(-1)
    key, order, cb, ce = e(n, i32), e(n, i32), e(c.K, i32), e(c.K, i32)
    xvs, rs = e(6 * n), e(n)
    A, uat, af, Fd, Fc = e(c.G), e(3 * n), e(n), e(3 * n), e(3 * n)

    def forward_stages():
        x, v = xv[:3 * n].view(3, n), xv[3 * n:]
        gic.gic_sort_cells(c, x, key, order, cb, ce)
        gic.gic_reorder(c, order, x, v, r, None, xvs[:3 * n], xvs[3 * n:], rs, None)
        xs, vs = xvs[:3 * n].view(3, n), xvs[3 * n:]
        gic.gic_p2g_real(c, xs, vs, rs, cb, ce, A, None)
        gic.gic_g2p(c, xs, u, None, A, uat, af)
        gic.gic_drag(c, rs, vs, uat, af, Fd)
        return xs, vs

    xs, vs = forward_stages()
    gic.gic_contact_forces(c, xs, vs, rs, cb, ce, Fc, pair_ids=e(48 * n, i32))
    x1, v1 = xs.clone(), vs.clone()
    gic.gic_integrate(c, rs, Fc, Fd, x1, v1)
    want = e(6 * n)
    gic.gic_permute(c, order, torch.cat([x1.reshape(-1), v1]), want, 6, True)
    for call in range(3):  # from the second on the count of bricks has reached the host
        out = torch.full_like(xv, -1.0)
        gic.gic_rollout_step(c, xv, r, u, out, key, order, cb, ce, e(6 * n), e(n))
        torch.cuda.synchronize()
        assert torch.equal(out, want), call
    # reverse
    rng = np.random.Generator(np.random.PCG64(9))
    g0 = T.dev(rng.normal(0, 1, 6 * n))
    xs, vs = forward_stages()
    gs = e(6 * n)
    gic.gic_permute(c, order, g0, gs, 6, False)
    gx, gv, gF = gs[:3 * n], gs[3 * n:], e(3 * n)
    gic.gic_integrate_vjp(c, rs, gx, gv, gF)
    gmu, gcd, guat, gaf, gA = e(n), e(n), e(3 * n), e(n), e(c.G)
    gic.gic_contact_forces_vjp(c, xs, vs, rs, cb, ce, gF, gx, gv, gmu)
    gic.gic_drag_vjp(c, rs, vs, uat, af, gF, gv, guat, gaf, gcd)
    gic.gic_g2p_vjp(c, xs, u, A, guat, gaf, cb, ce, gx, gA)
    gic.gic_p2g_vjp(c, xs, vs, rs, gA, None, gx, gv)
    want = e(6 * n)
    gic.gic_permute(c, order, gs, want, 6, True)
    for call in range(3):
        g, mu, cd = g0.clone(), e(1).fill_(2.0), e(1).fill_(3.0)
        gic.gic_rollout_step_vjp(c, xv, r, u, g, mu, cd, key, order, cb, ce, e(6 * n), e(n), e(6 * n), e(3 * n), e(n))
        torch.cuda.synchronize()
        for a, b in ((g[:3 * n], want[:3 * n]), (g[3 * n:], want[3 * n:])):
            assert float((a - b).abs().max()) <= 1e-11 * float(b.abs().max()), call
        for got, per, base in ((mu, gmu, 2.0), (cd, gcd, 3.0)):
            assert abs(float(got) - (base + float(per.sum()))) <= 1e-12 * (base + float(per.abs().sum())), call
        if call:
            assert torch.equal(g, last)  # the same bits on every call
        last = g
    assert c.error()[0] == 0


def test_rollout_step_arguments(T):
    import torch
    from paper_2504_00745_amd import gic
    d = wl.make("c4", n_override=64)
    n = 64
    z = lambda m, t=torch.float64: torch.zeros(m, dtype=t, device="cuda")  # noqa: E731

    def call(c, xv, out):
        gic.gic_rollout_step(c, xv, z(n), z(3 * c.G), out, z(n, torch.int32), z(n, torch.int32), z(c.K, torch.int32),
                             z(c.K, torch.int32), z(6 * n), z(n))

    for over, prec in ((dict(drag_model=1), "fp64"), (dict(vmass=1), "fp64"), (dict(), "fp32")):
        c = gic.Context(dict(d["params"], rho_f=1000.0, **over), n, prec, r_max=0.006)
        with pytest.raises(gic.GicError):
            call(c, z(6 * n), z(6 * n))
    c = gic.Context(d["params"], n, "fp64", r_max=0.006)
    xv = z(6 * n)
    with pytest.raises(gic.GicError):
        call(c, xv, xv)  # xv_out aliases xv


@pytest.mark.parametrize("over", [dict(drag_model=1), dict(vmass=1)])
def test_other_forms_step_forward(T, over):
    """A rollout of a form without a reverse still steps forward."""
    import torch
    from paper_2504_00745_amd.rollout import Rollout
    d = wl.make("c4", n_override=4099)
    cfg = dict(d["params"], rho_f=1000.0, mu_f=1e-3, **over)
    a = Rollout(cfg, d["r"], d["u"], 1, r_max=0.006)
    b = Rollout(dict(cfg, drag_model=0, vmass=0), d["r"], d["u"], 1, r_max=0.006)
    xv = torch.cat([T.dev(d["x"]).reshape(-1), T.dev(d["v"]).reshape(-1)])
    out = [torch.empty_like(xv) for _ in range(2)]
    a.step(xv, out[0])
    b.step(xv, out[1])
    assert bool(torch.isfinite(out[0]).all()) and not torch.equal(out[0], out[1])
