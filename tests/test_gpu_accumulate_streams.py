"""FSMT_ACCUMULATE from several streams into one set of outputs: every call's gradient and
objective are in the sum, on each path of cop_backward (one workgroup a restart, several slices,
gradient rows, Booleans in global memory, big diagrams)."""
import numpy as np
import pytest

import workloads as W

from gpu_util import T, dev, torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


CASES = {"wg": (lambda: W.make_workload("scheduling_200x10"), 32), "slices": (lambda: W.make_scheduling(400, 10, W.seed_seq(3)), 4),
         "rows": (lambda: W.make_placement(544, W.seed_seq(79)), 2), "mixed": (lambda: W.make_scheduling(520, 3, W.seed_seq(78)), 16),
         "big": (lambda: W.make_random_hybrid(100), 48)}


@pytest.mark.parametrize("name", list(CASES))
def test_streams_add_up(name):
    make, R = CASES[name]
    p = make()
    h = fsmt.xbdd_compile(p)
    a, b = (T(x) for x in W.initial_points(p, R, 100))
    w = T(np.ones(p.n_cons))
    one = [torch.zeros(R, device=dev()), torch.zeros_like(a), torch.zeros_like(b)]
    fsmt.cop_backward(h, a, b, 0.3, w, *one)
    total = [torch.zeros_like(x) for x in one]
    streams, calls = [torch.cuda.Stream() for _ in range(4)], 40
    torch.cuda.synchronize()
    for _ in range(calls):
        for s in streams:
            fsmt.cop_backward(h, a, b, 0.3, w, *total, flags=fsmt.FSMT_ACCUMULATE, stream=s)
    torch.cuda.synchronize()
    n = calls * len(streams)
    for got, x in zip(total, one):   # one lost call is 1/160 of the sum
        x = x.double().cpu().numpy()
        np.testing.assert_allclose(got.cpu().numpy(), n * x, rtol=1e-3, atol=1e-3 * np.abs(x).max())
    h.free()
