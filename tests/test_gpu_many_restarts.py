"""Large restart counts (launches past 2^32 threads are split; workgroups shrink; nearly empty
buckets go to the lane kernel): every restart gets the answer of a small call at its point."""
import numpy as np
import pytest

import workloads as W
from workloads.format import KIND_CARD_LE, KIND_CLAUSE, KIND_XOR, Builder, lit

from gpu_util import T, dev, torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _clauses():
    """1,100 two-literal clauses over 40 Booleans: 16 waves a workgroup."""
    rng = np.random.default_rng(103)
    b = Builder(40, 1, real_lo=np.full(1, -1.0), real_hi=np.full(1, 1.0))
    for _ in range(1100):
        x, y = (int(v) for v in rng.choice(40, 2, replace=False))
        b.add(KIND_CLAUSE, [lit(x), lit(y)], 0)
    return b.build()


def _cards():
    rng = np.random.default_rng(104)
    b = Builder(64, 1, real_lo=np.full(1, -1.0), real_hi=np.full(1, 1.0))
    for _ in range(2):
        b.add(KIND_CARD_LE, [lit(int(v)) for v in rng.choice(64, 40, replace=False)], 20)
    return b.build()


def _shapes():
    """300 parities and cardinalities of nearly as many diagram shapes (node-by-node, LDS columns)."""
    rng = np.random.default_rng(107)
    b = Builder(40, 1, real_lo=np.full(1, -1.0), real_hi=np.full(1, 1.0))
    for i in range(300):
        n = int(rng.integers(4, 13))
        lits = [lit(int(v), bool(rng.integers(0, 2))) for v in rng.choice(40, n, replace=False)]
        b.add((KIND_XOR, KIND_CARD_LE)[i % 2], lits, n // 2 if i % 2 else 0)
    return b.build()


# past 2^32 threads; and where the workgroups get smaller, and shapes go to the lane kernel
@pytest.mark.parametrize("make,R,accumulate", [(_clauses, (1 << 22) + 70, False), (_clauses, (1 << 22) + 70, True),
                                               (_cards, 5_600_000, False), (_clauses, 1100, False),
                                               (_clauses, 8200, False), (_shapes, 1023, False), (_shapes, 1024, True)])
def test_every_restart(make, R, accumulate):
    p = make()
    h = fsmt.xbdd_compile(p)
    few = 512
    a0, b0 = (T(x) for x in W.initial_points(p, few, 105))
    w = T(np.ones(p.n_cons))
    ref = [torch.zeros(few, device=dev()), torch.zeros_like(a0), torch.zeros_like(b0)]
    fsmt.cop_backward(h, a0, b0, 0.5, w, *ref)
    reps = (R + few - 1) // few
    a, b = a0.repeat(reps, 1)[:R].contiguous(), b0.repeat(reps, 1)[:R].contiguous()
    out = [torch.ones(R, device=dev()), torch.ones_like(a), torch.ones_like(b)]
    print(f"{R} restarts of {p.n_cons} constraints, accumulate {accumulate}", flush=True)
    fsmt.cop_backward(h, a, b, 0.5, w, *out, flags=fsmt.FSMT_ACCUMULATE if accumulate else 0)
    fobj = torch.ones(R, device=dev())
    fsmt.cop_forward(h, a, b, 0.5, w, fobj)
    torch.cuda.synchronize()
    for got, x in zip(out + [fobj], ref + [ref[0]]):
        x = x + (1.0 if accumulate and got is not fobj else 0.0)
        scale = float(x.abs().max())
        for i in {0, R // few // 2, max(R // few - 1, 0)}:   # whole blocks of the small call's restarts
            assert float((got[i * few:(i + 1) * few] - x).abs().max()) <= 2e-6 * scale
        last = R % few
        assert last == 0 or float((got[R - last:] - x[:last]).abs().max()) <= 2e-6 * scale
    h.free()

