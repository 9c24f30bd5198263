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
        if plan.workspace_bytes <= msft.MSFT_NOALLOC_MAX_BYTES:
            In = torch.full_like(I, float("nan"))
            msft.msft_simulate_noalloc(plan.handle, dt, bt, In, None)
            assert torch.equal(I, In)
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
