"""Plans by the form of their sums, against the FP64 oracle.

Tolerances on the norm.  Spherical form: FP64 sums on bases truncated at 3e-11, T to 3e-9
a step, the FP32 amplitude and result of one rounding (2^-24 = 6e-8) each: 2e-7 for the
amplitude, twice that for the intensity and the gradients.  Direct form: FP32 sums of up to
1e4 products in chains of at most some hundreds, 1e-5 as for every FP32 pattern; the split
leaves out lo * lo and rounds lo, 2^-16 each of a product, 1e-4.
"""
import numpy as np
import pytest

import oracle
from paper_2202_03411_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"spherical": 2e-7, "fp32": 1e-5, "bf16x3": 1e-4}


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2202_03411_amd import msft
    return torch, msft


def _rel(a, b):
    return float(np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b)))


def _fields(grid, seed, top=0.05):
    rng = np.random.default_rng(inputs.SEED_BASE + seed)
    return (rng.uniform(0.0, top, grid).astype(np.float32) for _ in range(2))


def _check(env, grid, det, pitch, theta, precision, detector, forms, lam=45.0, pixels=400):
    """Forward and adjoint of a plan of these forms against the oracle; returns the plan's
    intensity and amplitude and its tensors, for what a test adds."""
    torch, msft = env
    print(f"[gpu] {detector} {precision} grid={grid} det={det} {forms}", flush=True)
    d, b = _fields(grid, det)
    g = np.random.default_rng(det).normal(size=det * det).astype(np.float32)
    q = oracle.qmap(lam, theta, det) if detector == "flat" else oracle.qmap_uniform(lam, theta, det)
    ok = np.flatnonzero(~np.isnan(q[:, 2]))
    pix = ok[:: max(1, ok.size // pixels)]
    d64, b64 = d.astype(np.float64), b.astype(np.float64)
    Ao = oracle.amplitude(q[pix], oracle.strength(oracle.MSFT, d64, b64, pitch, lam), pitch, 1)
    with msft.Plan(lam, theta, det, grid, pitch, precision, detector=detector) as plan:
        assert msft.msft_plan_forms(plan.handle) == forms
        dt, bt = torch.from_numpy(d).cuda(), torch.from_numpy(b).cuda()
        I, A = plan.simulate(dt, bt, amplitude=True)
        gd, gb = torch.full_like(dt, float("nan")), torch.full_like(bt, float("nan"))
        msft.msft_backward(plan.handle, dt, bt, torch.view_as_real(A).contiguous(),
                           torch.from_numpy(g).cuda(), gd, gb, plan.workspace())
        In = torch.full_like(I, float("nan"))
        try:   # refused where the direct form's scratch passes the fixed one, whichever form runs
            msft.msft_simulate_noalloc(plan.handle, dt, bt, In, None)
            assert torch.equal(I, In)
        except msft.MSFTError as e:
            assert e.status == msft.MSFT_ERR_UNSUPPORTED and np.prod(grid) > 5e5
        if detector == "flat":
            Ib = torch.full_like(I, float("nan"))
            reqs = [(plan.handle, dt, bt, Ib, None)]
            msft.msft_simulate_batch(reqs, msft.workspace_tensor(msft.msft_batch_query(reqs), "cuda"))
            assert torch.equal(I, Ib)
        torch.cuda.synchronize()
        I, A = I.cpu().numpy().astype(np.float64), A.cpu().numpy().astype(np.complex128)
        gd, gb = (t.cpu().numpy().astype(np.float64).reshape(-1, grid[2]) for t in (gd, gb))
    rng = np.random.default_rng(det + 1)
    cols = np.sort(rng.choice(grid[0] * grid[1], size=min(24, grid[0] * grid[1]), replace=False))
    od, ob = oracle.backward(oracle.MSFT, q[ok], g[ok].astype(np.float64), A[ok], d64, b64, pitch, lam, cols=cols)
    errs = [_rel(A[pix], Ao), _rel(I[pix], np.abs(Ao) ** 2), _rel(gd[cols], od), _rel(gb[cols], ob)]
    print("  amplitude %.2e intensity %.2e gradients %.2e %.2e" % tuple(errs), flush=True)
    fwd = TOL["spherical" if forms[0] == "spherical" else precision]
    adj = TOL["spherical" if forms[1] == "spherical" else "fp32"]   # the direct adjoint is FP32 in both
    assert errs[0] <= fwd and errs[1] <= 2 * fwd
    assert max(errs[2:]) <= 2 * adj


@pytest.mark.parametrize("grid,det,pitch,theta,precision,detector,forms", [
    # few pixels on many angles: the gradient direct
    ((60, 62, 90), 11, (20.0, 20.0, 20.0), 60.0, "fp32", "flat", ("spherical", "direct")),
    ((60, 62, 90), 11, (20.0, 20.0, 20.0), 60.0, "bf16x3", "flat", ("spherical", "direct")),
    ((140, 60, 100), 40, (21.375,) * 3, 60.0, "fp32", "uniform_q", ("spherical", "direct")),
    ((200, 140, 60), 40, (21.375,) * 3, 60.0, "fp32", "uniform_q", ("spherical", "direct")),
    ((200, 140, 60), 40, (21.375,) * 3, 60.0, "bf16x3", "uniform_q", ("spherical", "direct")),
    # few columns of many slices: the pattern direct
    ((14, 2, 734), 109, (3.78, 3.78, 4.567), 75.0, "fp32", "flat", ("direct", "spherical")),
    ((14, 2, 734), 109, (3.78, 3.78, 4.567), 75.0, "bf16x3", "flat", ("direct", "spherical")),
    ((28, 65, 407), 72, (5.31,) * 3, 60.0, "fp32", "uniform_q", ("direct", "spherical")),
    ((60, 62, 300), 40, (11.25,) * 3, 60.0, "bf16x3", "uniform_q", ("direct", "spherical")),
])
def test_forward_and_adjoint_of_different_forms(env, grid, det, pitch, theta, precision, detector, forms):
    _check(env, grid, det, pitch, theta, precision, detector, forms)


def test_four_hundred_nodes(env):
    # the most nodes a plan may have: the adjoint's coefficient stage takes 54 400 bytes of
    # dynamic and 24 576 of static LDS, past 64 KiB
    _check(env, (324, 30, 4), 100, (22.0, 22.0, 5.0), 80.0, "fp32", "flat", ("spherical", "spherical"))


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_direct_kernels_at_size(env, precision):
    # the flat detector's own pixels as a list of momenta, which is always summed directly:
    # 1.2e10 pixels x voxels, ragged axes (partial x, y and z tiles), forward, its variant on
    # the fixed scratch, a batch of three pixel ranges, and the adjoint
    torch, msft = env
    grid, det, pitch, lam = (97, 61, 75), 165, (7.0, 8.0, 6.0), 45.0
    print(f"[gpu] direct {precision} grid={grid} det={det}", flush=True)
    d, b = _fields(grid, 7)
    q = oracle.qmap(lam, 60.0, det)
    pix = inputs.random_pixels(det, 400, seed=8)
    d64, b64 = d.astype(np.float64), b.astype(np.float64)
    Ao = oracle.amplitude(q[pix], oracle.strength(oracle.MSFT, d64, b64, pitch, lam), pitch, 1)
    g = np.random.default_rng(9).normal(size=det * det).astype(np.float32)
    with msft.Plan(lam, 60.0, 0, grid, pitch, precision, q=q) as plan:
        assert msft.msft_plan_forms(plan.handle) == ("direct", "direct")
        dt, bt = torch.from_numpy(d).cuda(), torch.from_numpy(b).cuda()
        I, A = plan.simulate(dt, bt, amplitude=True)
        In = torch.full_like(I, float("nan"))
        msft.msft_simulate_noalloc(plan.handle, dt, bt, In, None)
        Ib = torch.full_like(I, float("nan"))
        nb = -(-plan.npix // msft.msft_pixel_block())
        cuts = [0, 5, nb - 1, nb]
        reqs = [(plan.handle, dt, bt, Ib, None, r) for r in zip(cuts, cuts[1:])]
        msft.msft_simulate_batch(reqs, msft.workspace_tensor(msft.msft_batch_query(reqs), "cuda"))
        assert torch.equal(I, In) and torch.equal(I, Ib)
        gd, gb = torch.full_like(dt, float("nan")), torch.full_like(bt, float("nan"))
        msft.msft_backward(plan.handle, dt, bt, torch.view_as_real(A).contiguous(),
                           torch.from_numpy(g).cuda(), gd, gb, plan.workspace())
        torch.cuda.synchronize()
        I, A = I.cpu().numpy().astype(np.float64), A.cpu().numpy().astype(np.complex128)
        gd, gb = (t.cpu().numpy().astype(np.float64).reshape(-1, grid[2]) for t in (gd, gb))
    cols = np.sort(np.random.default_rng(10).choice(grid[0] * grid[1], size=24, replace=False))
    od, ob = oracle.backward(oracle.MSFT, q, g.astype(np.float64), A, d64, b64, pitch, lam, cols=cols)
    errs = [_rel(A[pix], Ao), _rel(I[pix], np.abs(Ao) ** 2), _rel(gd[cols], od), _rel(gb[cols], ob)]
    print("  amplitude %.2e intensity %.2e gradients %.2e %.2e" % tuple(errs), flush=True)
    assert errs[0] <= TOL[precision] and errs[1] <= 2 * TOL[precision]
    assert max(errs[2:]) <= 2 * TOL["fp32"]


@pytest.mark.parametrize("n", [511, 383, 255])
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_uniform_column_groups_of_the_direct_form(env, n, precision):
    # detector sides whose second stage leaves a last, partial group of columns (the split: 2, 2
    # and 1 columns to a workgroup; the three products of FP32: 8, 4 and 2), on a grid small
    # enough for the direct form: seeded pixels, every row of column 0 and the last three
    torch, msft = env
    grid, pitch, lam = (8, 70, 5), (9.0, 7.0, 8.0), 45.0
    print(f"[gpu] direct uniform_q {precision} grid={grid} det={n}", flush=True)
    d, b = _fields(grid, n)
    q = oracle.qmap_uniform(lam, 60.0, n)
    rows = np.arange(n)
    pix = np.concatenate([inputs.random_pixels(n, 400, seed=n)] + [rows * n + i for i in (0, n - 3, n - 2, n - 1)])
    ok = ~np.isnan(q[pix, 2])
    w = oracle.strength(oracle.MSFT, d.astype(np.float64), b.astype(np.float64), pitch, lam)
    Io = np.abs(oracle.amplitude(q[pix][ok], w, pitch, 1)) ** 2
    with msft.Plan(lam, 60.0, n, grid, pitch, precision, detector="uniform_q") as plan:
        assert msft.msft_plan_forms(plan.handle) == ("direct", "direct")
        I = plan.simulate(torch.from_numpy(d).cuda(), torch.from_numpy(b).cuda())
        I = I.cpu().numpy().astype(np.float64)[pix]
    err = _rel(I[ok], Io)
    print(f"  intensity {err:.2e} on {int(ok.sum())} pixels", flush=True)
    assert err <= 2 * TOL[precision]
    assert np.all(I[~ok] == 0.0)


@pytest.mark.parametrize("grid,det,pitch,theta,detector,lam", [
    # more than 48 modes of a parity: the scan's products make a second pass
    ((20, 21, 230), 64, (4.0, 4.0, 5.0), 80.0, "flat", 13.5),
    # columns of more than 256 slices: rounds of 64
    ((33, 31, 300), 40, (9.0, 9.0, 9.0), 60.0, "flat", 45.0),
    ((12, 10, 1100), 61, (6.0, 6.0, 3.0), 60.0, "flat", 45.0),
    ((40, 40, 500), 200, (5.0, 5.0, 5.0), 60.0, "uniform_q", 45.0),
    # G of 32 of the 232 nodes at a time, the last part short
    ((130, 130, 130), 512, (6.1538,) * 3, 80.0, "uniform_q", 13.5),
])
def test_spherical_kernels_at_their_edges(env, grid, det, pitch, theta, detector, lam):
    _check(env, grid, det, pitch, theta, "fp32", detector, ("spherical", "spherical"), lam=lam, pixels=150)


@pytest.mark.parametrize("detector", ["flat", "uniform_q"])
def test_aliased_axes(env, detector):
    # MSFT_ALLOW_ALIAS: pitches past the sampling limit on every axis take the whole basis
    torch, msft = env
    grid, det, pitch, lam = (30, 28, 120), 150, (40.0, 41.0, 39.0), 45.0
    print(f"[gpu] aliased {detector} grid={grid} det={det}", flush=True)
    d, b = _fields(grid, 11, top=0.01)
    q = oracle.qmap(lam, 60.0, det) if detector == "flat" else oracle.qmap_uniform(lam, 60.0, det)
    pix = np.flatnonzero(~np.isnan(q[:, 2]))[::40]
    w = oracle.strength(oracle.MSFT, d.astype(np.float64), b.astype(np.float64), pitch, lam)
    Ao = oracle.amplitude(q[pix], w, pitch, 1)
    with pytest.raises(msft.MSFTError):
        msft.Plan(lam, 60.0, det, grid, pitch, detector=detector)
    with msft.Plan(lam, 60.0, det, grid, pitch, detector=detector, allow_alias=True) as plan:
        assert msft.msft_plan_forms(plan.handle)[0] == "spherical"
        _, A = plan.simulate(torch.from_numpy(d).cuda(), torch.from_numpy(b).cuda(), amplitude=True)
        A = A.cpu().numpy().astype(np.complex128)
    print(f"  amplitude {_rel(A[pix], Ao):.2e}", flush=True)
    assert _rel(A[pix], Ao) <= TOL["spherical"]


def test_batch_equals_each_request_alone(env):
    # bit for bit, where the batch takes other variants than a request alone: two tiles of b
    # to a workgroup (12 x 57 x 4 tiles, alone 228), four columns to a lane (9 rows' waves of
    # 128 past 2048, alone 256), nodes in parts beside whole plans, a direct plan beside them,
    # and a field of NaN in one request
    torch, msft = env
    lam = 45.0
    with msft.Plan(lam, 60.0, 512, (128, 128, 128), (5.18,) * 3) as star, \
         msft.Plan(13.5, 80.0, 256, (110, 60, 40), (5.4,) * 3) as wide, \
         msft.Plan(13.5, 80.0, 90, (116, 115, 114), (5.4,) * 3) as parts, \
         msft.Plan(lam, 60.0, 16, (8, 8, 8), (9.0,) * 3) as small:
        assert [msft.msft_plan_forms(p.handle)[0] for p in (star, wide, parts, small)] == \
            ["spherical"] * 3 + ["direct"]
        gen = torch.Generator(device="cuda").manual_seed(12)

        def field(p):
            return [torch.rand(p.grid, generator=gen, device="cuda") * 0.05 for _ in range(2)]

        for plans in ([star] * 12, [wide] * 9 + [parts, small, wide], [parts, star, parts]):
            print(f"[gpu] batch of {len(plans)}: {plans[0].grid} ...", flush=True)
            fields = [field(p) for p in plans]
            fields[1][0][3, 2, 1] = float("nan")
            out = [(torch.full((p.npix,), -1.0, device="cuda"), torch.full((p.npix, 2), -1.0, device="cuda"))
                   for p in plans]
            reqs = [(p.handle, *f, *o) for p, f, o in zip(plans, fields, out)]
            msft.msft_simulate_batch(reqs, msft.workspace_tensor(msft.msft_batch_query(reqs), "cuda"))
            for k, (p, f, o) in enumerate(zip(plans, fields, out)):
                I, A = p.simulate(*f, amplitude=True)
                if k == 1:
                    assert bool(o[0].isnan().all()) and bool(I.isnan().all())
                else:
                    assert torch.equal(I, o[0]) and torch.equal(torch.view_as_real(A), o[1])


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("detector", ["flat", "uniform_q"])
@pytest.mark.parametrize("nz", [70, 200, 500])
def test_a_voxel_that_is_not_finite_reaches_every_pixel(env, detector, nz, value):
    torch, msft = env
    with msft.Plan(45.0, 60.0, 200, (40, 40, nz), (5.0, 5.0, 5.0), detector=detector) as plan:
        assert msft.msft_plan_forms(plan.handle)[0] == "spherical"
        rim = torch.from_numpy(np.isnan(plan.qmap()[:, 2])).cuda()
        d = torch.rand(plan.grid, device="cuda") * 0.05
        for k in range(2):
            f = [d.clone(), d.clone()]
            f[k][17, 5, nz // 2] = value
            I = plan.simulate(*f)
            assert not bool(I[~rim].isfinite().any())
            assert bool((I[rim] == 0.0).all())


def test_buffers_off_a_16_byte_boundary(env):
    # the voxel arrays and gradients as views one float into their storage: the same bits
    torch, msft = env
    grid, det = (40, 33, 64), 160
    with msft.Plan(45.0, 60.0, det, grid, (6.0,) * 3) as plan:
        assert msft.msft_plan_forms(plan.handle) == ("spherical", "spherical")
        V = int(np.prod(grid))

        def off(t):
            v = torch.empty(V + 1, device="cuda")[1:].view(grid)
            v.copy_(t)
            return v
        d, b = torch.rand(grid, device="cuda") * 0.05, torch.rand(grid, device="cuda") * 0.05
        g = torch.randn(plan.npix, device="cuda")
        I, A = plan.simulate(d, b, amplitude=True)
        Ar = torch.view_as_real(A).contiguous()
        gd, gb = torch.empty_like(d), torch.empty_like(b)
        msft.msft_backward(plan.handle, d, b, Ar, g, gd, gb, plan.workspace())
        do, bo, god, gob = off(d), off(b), off(d), off(b)
        assert torch.equal(plan.simulate(do, bo), I)
        msft.msft_backward(plan.handle, do, bo, Ar, g, god, gob, plan.workspace())
        assert torch.equal(god, gd) and torch.equal(gob, gb)
