"""Which form a plan's sums take and what follows from it, on host-only plans."""
import numpy as np
import pytest

from paper_2202_03411_amd import msft


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
