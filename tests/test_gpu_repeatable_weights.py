"""The weights after an ERWA update: equal check bits give the same bits in every run (the sums
of the normalization are taken in a fixed order), on both schedules."""
import numpy as np
import pytest

import workloads as W

from gpu_util import torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")
from paper_2603_22877_amd import solver as S  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("schedule", [1, 2])
def test_weights_repeat(schedule):
    """kappa = infinity, no steps: every run checks the same points, so only the weight update can
    differ. 11,475 constraints: 45 blocks a restart on the grid schedule."""
    p = W.make_workload("placement_150")
    h = fsmt.xbdd_compile(p)
    a, b = W.initial_points(p, 4, 99)
    w0 = np.random.default_rng(99).uniform(0.5, 2.0, (4, p.n_cons)).astype(np.float32)
    cfg = S.SolveConfig(kappas=[float("inf")] * 3, steps_per_level=0, eps=0.0, stop_on_sat=0, schedule=schedule)
    first = None
    for _ in range(12):
        st = S.BatchState(h, a, b, w0=w0)
        S.solve_batched([h], [st], cfg)
        torch.cuda.synchronize()
        w = st.w.cpu().numpy()
        if first is None:
            first = w
            np.testing.assert_allclose(w.sum(1, dtype=np.float64), p.n_cons, rtol=1e-4)
        np.testing.assert_array_equal(w.view(np.uint32), first.view(np.uint32))
    h.free()
