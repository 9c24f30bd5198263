"""Which form a plan's sums take and what follows from it, on host-only plans."""
import numpy as np
import pytest

from paper_2202_03411_amd import msft, serving


def _forms(grid, det, pitch, theta=60.0, precision="fp32", detector="flat", lam=45.0):
    with msft.Plan(lam, theta, det, grid, pitch, precision, device=-1, detector=detector) as p:
        return msft.msft_plan_forms(p.handle)


def test_a_plan_tells_its_forms():
    pitch = (5.0, 5.0, 5.0)
    assert _forms((64, 64, 64), 128, pitch) == ("spherical", "spherical")
    assert _forms((64, 64, 64), 128, pitch, precision="bf16x3") == ("spherical", "spherical")
    assert _forms((64, 64, 64), 128, pitch, detector="uniform_q") == ("spherical", "spherical")
    assert _forms((64, 64, 64), 128, pitch, precision="bf16") == ("direct", "direct")
    assert _forms((8, 8, 8), 16, pitch) == ("direct", "direct")
    # over 400 angles
    assert _forms((512, 512, 64), 64, (20.0, 20.0, 20.0)) == ("direct", "direct")
    q = np.zeros((4096, 3))
    with msft.Plan(45.0, 60.0, 0, (64, 64, 64), pitch, device=-1, q=q) as p:
        assert msft.msft_plan_forms(p.handle) == ("direct", "direct")
    with pytest.raises(msft.MSFTError):
        msft.msft_plan_forms(None)


@pytest.mark.parametrize("grid,det,pitch,theta,precision,detector,forms", [
    # 64 pixels on 256^3 voxels: gradient 749 us in the spherical form, 390 direct; forward 356 / 29 286
    ((256, 256, 256), 8, (16.0, 16.0, 16.0), 60.0, "fp32", "flat", ("spherical", "direct")),
    # 28 columns of 1734 slices, split: forward 1102 / 242, gradient 578 / 929
    ((14, 2, 1734), 109, (3.78, 3.78, 4.567), 75.0, "bf16x3", "flat", ("direct", "spherical")),
    # many angles on the uniform detector: forward 127 / 103, gradient 278 / 53
    ((333, 87, 64), 78, (11.25, 11.25, 11.25), 60.0, "fp32", "uniform_q", ("spherical", "direct")),
    # long columns there: 375 / 58 and 481 / 110 at 171 x 13 x 285 on 126^2, split
    ((171, 13, 285), 126, (21.0, 21.0, 21.0), 60.0, "bf16x3", "uniform_q", ("direct", "direct")),
    # columns enough: 721 / 31 295
    ((76, 150, 1350), 40, (5.0, 5.0, 5.0), 60.0, "fp32", "flat", ("spherical", "spherical")),
])
def test_each_direction_takes_the_faster_form(grid, det, pitch, theta, precision, detector, forms):
    assert _forms(grid, det, pitch, theta, precision, detector) == forms


def test_the_fixed_scratch_binds_the_forward_alone():
    # 140^3 voxels at 13.5 nm: the direct form's tiles fit the 64 MiB of msft_simulate_noalloc,
    # the spherical form's sums do not; msft_backward has no such variant
    assert _forms((140, 140, 140), 512, (800 / 140,) * 3, 80.0, lam=13.5) == ("direct", "spherical")


def test_scratch_is_that_of_the_form_that_runs():
    # 192^3 voxels on 1024^2 pixels: the direct form's W tiles are 6 x chunks of 32 times 6 z
    # blocks of 32 times 192 y at 12 KiB (three planes of Re, Im at 64 bytes a row of 32)
    n, det = 192, 1024
    direct = 6 * 6 * n * 12288
    with msft.Plan(45.0, 60.0, det, (n, n, n), (700.0 / n,) * 3, device=-1) as p:
        assert msft.msft_plan_forms(p.handle) == ("spherical", "spherical")
        scratch = p.per_request_bytes - 2 * 4 * n ** 3 - 12 * det * det
        assert 0 < scratch < direct // 2
        assert scratch % 256 == 0 and p.workspace_bytes >= scratch
        # and the variant on the fixed scratch refuses what it did, by the direct form's
        assert direct > msft.MSFT_NOALLOC_MAX_BYTES
        assert msft._lib.msft_simulate_noalloc(p.handle, None, None, None, None, None) == msft.MSFT_ERR_UNSUPPORTED
        assert "direct form" in msft.msft_last_error()


@pytest.mark.parametrize("precision,slices", [("fp32", 1), ("bf16", 4)])
def test_a_request_is_sliced_only_where_its_work_divides_by_pixel_blocks(precision, slices):
    # the spherical form's scan and sums belong to the request, not to its pixel blocks:
    # cutting it into slices would repeat them; the direct form's blocks are the work
    plans = serving.PlanCache(msft, precision, device=-1, calibrate=False)
    ex = serving.GpuExecutor.__new__(serving.GpuExecutor)
    ex.plans, ex.msft, ex.batched, ex.wave_blocks = plans, msft, True, 256
    key = (45.0, 60.0, 360, (24, 24, 24), (9.0, 9.0, 9.0), "msft")
    launched = []
    ex.launch = lambda items: launched.extend(items)
    ex.poll = lambda handle: True
    ex.finish = lambda handle, items: None
    ex.complete = lambda req: None
    plans.get(key)
    plans.block_cost[key] = 1e-4     # 1013 blocks of 0.1 ms: some 20 quanta
    s = serving.Scheduler(ex, 1 << 40, max_inflight=2, quantum=0.005)
    s.submit(serving.Request(0, 0.0, key))
    while not s.idle():
        s.step()
    assert [b1 - b0 for _, b0, b1 in launched] == ([1013] if slices == 1 else [256, 256, 256, 245])
    plans.close()


def test_a_plan_the_form_cannot_serve_costs_no_more():
    # 512^3 voxels of 20 nm need more than 400 angles, which the phase's rate tells at once
    # (finding it from the series' coefficients took 16 ms); plain BF16 never asks
    import time

    def fastest(precision):
        best = 1.0
        for _ in range(7):
            t = time.perf_counter()
            with msft.Plan(45.0, 60.0, 64, (512, 512, 512), (20.0, 20.0, 20.0), precision, device=-1) as p:
                best = min(best, time.perf_counter() - t)
                assert msft.msft_plan_forms(p.handle) == ("direct", "direct")
        return best

    assert fastest("fp32") < fastest("bf16") + 4e-3
