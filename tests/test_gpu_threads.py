"""Host threads that call into the library at once, each on a stream of its own, with instances
whose kernels take different amounts of LDS past the default 64 KB."""
import threading

import numpy as np
import pytest

import workloads as W
from workloads.format import KIND_CARD_LE, Builder, lit

from gpu_util import T, dev, torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _cards(n, length, count, seed):
    rng = np.random.default_rng([101, seed])
    b = Builder(n, 2, real_lo=np.full(2, -1.0), real_hi=np.full(2, 1.0))
    for _ in range(count):
        b.add(KIND_CARD_LE, [lit(int(v), bool(rng.integers(0, 2))) for v in rng.choice(n, length, replace=False)], length // 2)
    return b.build()


@pytest.mark.parametrize("R,messages", [(48, 0), (3, 2)])   # gradient sums in LDS / level by level
def test_different_lds_at_once(R, messages):
    """Four threads, diagrams and states of different sizes, 200 calls each."""
    cases = []
    for i, (n, length) in enumerate(((100, 40), (6000, 62), (2500, 50), (9000, 62))):
        p = _cards(n, length, 6, i)
        h = fsmt.xbdd_compile(p, messages=messages)
        a, b = (T(x) for x in W.initial_points(p, R, 102, i))
        w = T(np.ones(p.n_cons))
        out = [torch.zeros(R, device=dev()), torch.zeros_like(a), torch.zeros_like(b)]
        fsmt.cop_backward(h, a, b, 0.5, w, *out)
        cases.append((h, a, b, w, out, [x.clone() for x in out], torch.cuda.Stream()))
    torch.cuda.synchronize()
    errors, go = [], threading.Barrier(len(cases))

    def work(h, a, b, w, out, ref, stream):
        try:
            torch.cuda.set_device(0)
            go.wait()
            for _ in range(200):
                fsmt.cop_backward(h, a, b, 0.5, w, *out, stream=stream)
        except Exception as e:   # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=c) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for h, _, _, _, out, ref, _ in cases:
        for x, y in zip(out, ref):
            np.testing.assert_allclose(x.cpu().numpy(), y.cpu().numpy(), rtol=1e-5, atol=1e-6)
        h.free()
