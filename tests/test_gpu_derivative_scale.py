"""The scale kappa / (sqrt(2 pi) |q|) of an atom's derivative, at points where every other factor
of the gradient is exact in float32: an atom at z = 0 (e^{-u^2} = 1) among literals whose
probabilities are 0 or 1. The gradient is then the scale itself, rounded once from 64 bits.
And at scales whose product with a weight exceeds float32, where e^{-u^2} is 0."""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads.format import KIND_EXPR, OP_LE, X_AND, X_OR, Builder, lit
from workloads.paper_suite import index_differs_program

from gpu_util import T, dev, torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")
from test_gpu_tiles import _clause_pairs, _index_pairs  # noqa: E402

KAPPAS = np.random.default_rng(96).uniform(0.05, 40.0, 64)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _scale(kappa):
    return np.float32(kappa * 0.5 * 0.5641895835477563)   # |q| = sqrt(2)


def _gradient_b(p, a, b, kappa):
    h = fsmt.xbdd_compile(p)
    ga, gb, obj = torch.zeros(1, p.n_bool, device=dev()), torch.zeros(1, p.n_real, device=dev()), torch.zeros(1, device=dev())
    fsmt.cop_backward(h, T(a), T(b), kappa, T(np.ones(p.n_cons)), obj, ga, gb)
    h.free()
    return gb.cpu().numpy()[0]


def test_index_pairs():
    """17 items (136 pairs: tiles): 0 and 1 agree in their bit and touch (y_0 - y_1 = the bound),
    every other pair differs in a bit."""
    n, L = 17, 5
    b = Builder(n * L, n, real_lo=np.full(n, -1e5), real_hi=np.full(n, 1e5))
    for j in range(n):
        for k in range(j + 1, n):
            at = [b.atom([u, v], [1.0, -1.0], OP_LE, -1.0) for u, v in ((j, k), (k, j))]
            bits = sum(([lit(i * n + j), lit(i * n + k)] for i in range(L)), [])
            b.add(KIND_EXPR, bits + [lit(x) for x in at], 0, index_differs_program(L, 2))
    p = b.build()
    code = np.maximum(np.arange(n), 1)   # items 0 and 1 share a code
    a = np.concatenate([np.where((code >> i) & 1, -1.0, 1.0) for i in range(L)]).astype(np.float32)[None]
    y = np.arange(n, dtype=np.float32)[None] * 1000.0
    y[0, 1] = y[0, 0] + 1.0              # y_0 - y_1 = -1: the atom's bound; the other is at +2
    for kappa in KAPPAS:
        if 2.0 * kappa * 0.5 < 6.0:      # the far atom must be False with probability 1 in float32
            continue
        gb = _gradient_b(p, a, y, kappa)
        assert gb[0] == _scale(kappa) and gb[1] == -_scale(kappa), (kappa, gb[:2], _scale(kappa))


def test_windows():
    """A window whose first bound is met exactly and whose second holds with probability 1."""
    b = Builder(3, 4, real_lo=np.full(4, -1e5), real_hi=np.full(4, 1e5))
    at = [b.atom([0, 1], [1.0, -1.0], OP_LE, 2.0), b.atom([2, 3], [1.0, -1.0], OP_LE, 0.0)]
    b.add(KIND_EXPR, [lit(0), lit(1), lit(2)] + [lit(x) for x in at], 0, [0, 1, X_OR, 2, X_OR, 3, 4, X_AND, X_OR])
    p = b.build()
    a = np.ones((1, 3), np.float32)
    y = np.array([[5.0, 3.0, 0.0, 4000.0]], np.float32)
    for kappa in KAPPAS:
        gb = _gradient_b(p, a, y, kappa)
        assert gb[0] == _scale(kappa) and gb[1] == -_scale(kappa), (kappa, gb, _scale(kappa))


@pytest.mark.parametrize("make", ["rect", "bits1", "bits2", "clauses"])
def test_weight_times_scale_beyond_float32(make):
    """kappa 1e30 and weights of 1e10: no atom is near its bound, so the gradient in b is 0 and the
    Booleans' is that of the indicator."""
    p = {"rect": lambda: W.make_placement(40, W.seed_seq(97), fill=0.3, max_side=5), "bits1": lambda: _index_pairs(33, 5, 1, 6),
         "bits2": lambda: _index_pairs(33, 9, 2, 7), "clauses": lambda: _clause_pairs(40, 3, 8)}[make]()
    a, b = W.initial_points(p, 3, 98)
    w = np.full((3, p.n_cons), 1e10, np.float32)
    h = fsmt.xbdd_compile(p)
    ga, gb, obj = torch.zeros(3, p.n_bool, device=dev()), torch.zeros(3, p.n_real, device=dev()), torch.zeros(3, device=dev())
    fsmt.cop_backward(h, T(a), T(b), 1e30, T(w), obj, ga, gb)
    h.free()
    o = oracle.objective(p, a, b, 1e30, w=w, per_constraint=False)
    np.testing.assert_array_equal(gb.cpu().numpy(), np.zeros_like(b))
    np.testing.assert_allclose(ga.cpu().numpy(), o["grad_a"], rtol=1e-5, atol=4e-7 * o["absg_a"].max())
    np.testing.assert_allclose(obj.cpu().numpy(), o["U"], rtol=1e-5)
