"""Instances that mix constraint families, against the oracle at the parity bar: window
disjunctions beside a long cardinality (a big diagram: the grid schedule's sweeps and the
level-synchronous pass), beside node-by-node templates, with the LDS message store, and where
the per-call passes keep the state or the message columns out of a workgroup's LDS; index pairs
with atoms that have no inline record."""
import numpy as np
import pytest

import oracle
import workloads as W
from workloads.format import KIND_CARD_LE, KIND_EXPR, KIND_XOR, OP_GE, OP_LE, X_AND, X_OR, Builder, lit
from workloads.paper_suite import index_differs_program

from gpu_util import T, assert_gradient, assert_objective, assert_unsat, dev, torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")
from test_gpu_solver import _assert_step, _one_step  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _windows_and(nb, beside, n_windows=200, extra=0, seed=0):
    """n_windows windows of nb Boolean literals, beside: "card60" one 60-literal cardinality,
    "xor3" three-literal parities, "card13" cardinalities whose node-by-node columns take 39 KB a
    wave, "" nothing; `extra` Booleans that no constraint names."""
    rng = np.random.default_rng([91, nb, n_windows, seed])
    n = 80
    b = Builder(n + extra, 6, real_lo=np.full(6, -3.0), real_hi=np.full(6, 3.0))
    for _ in range(n_windows):
        u = int(rng.integers(0, 6))
        at = [b.atom([u], [1.0], OP_GE, -1.0 + float(rng.integers(0, 8)) / 8),
              b.atom([u], [1.0], OP_LE, 1.0 + float(rng.integers(0, 8)) / 8)]
        lits = [lit(int(x), bool(rng.integers(0, 2))) for x in rng.choice(n, nb, replace=False)]
        prog = [0] + sum(([i, X_OR] for i in range(1, nb)), []) + [nb, nb + 1, X_AND, X_OR]
        b.add(KIND_EXPR, lits + [lit(a) for a in at], 0, prog)
    length, kind, count = {"card60": (60, KIND_CARD_LE, 1), "xor3": (3, KIND_XOR, 70), "card13": (13, KIND_CARD_LE, 9),
                           "": (0, 0, 0)}[beside]
    for _ in range(count):
        lits = [lit(int(x), bool(rng.integers(0, 2))) for x in rng.choice(n, length, replace=False)]
        b.add(kind, lits, length // 2 if kind == KIND_CARD_LE else 0)
    return b.build()


def _compare(p, R, kap, seed, messages=0):
    """cop_backward, cop_forward and round_and_check against the oracle."""
    rng = np.random.default_rng(seed)
    a, b = W.initial_points(p, R, 92, seed)
    w = rng.uniform(0.5, 2.0, (R, p.n_cons)).astype(np.float32)
    h = fsmt.xbdd_compile(p, messages=messages)
    ta, tb, tw = T(a), T(b), T(w)
    ga, gb = torch.full_like(ta, 7.0), torch.full_like(tb, 7.0)
    obj, fobj = (torch.full((R,), 7.0, device=dev()) for _ in range(2))
    unsat = torch.full((R, p.n_cons), -1.0, device=dev())
    fsmt.cop_backward(h, ta, tb, kap, tw, obj, ga, gb)
    fsmt.cop_forward(h, ta, tb, kap, tw, fobj, unsat)
    o = oracle.objective(p, a, b, kap, w=w)
    assert_objective(obj.cpu().numpy(), o["U"], w.sum(1))
    assert_objective(fobj.cpu().numpy(), o["U"], w.sum(1))
    assert_unsat(unsat.cpu().numpy(), o["unsat"])
    assert_gradient(ga.cpu().numpy(), o["grad_a"], o["absg_a"], "grad_a")
    assert_gradient(gb.cpu().numpy(), o["grad_b"], o["absg_b"], "grad_b")
    bits = torch.zeros(R, (p.n_cons + 31) // 32, dtype=torch.int32, device=dev())
    nu, ver = torch.zeros(R, dtype=torch.int32, device=dev()), torch.zeros(R, dtype=torch.int32, device=dev())
    fsmt.round_and_check(h, ta, tb, None, bits, nu, ver)
    ch = oracle.check(p, a, b)
    np.testing.assert_array_equal(bits.cpu().numpy().view(np.uint32), ch["sat_bits"])
    np.testing.assert_array_equal(nu.cpu().numpy(), ch["n_unsat"])
    info = fsmt.xbdd_info(h)
    h.free()
    return info


@pytest.mark.parametrize("nb", [1, 2, 4])
@pytest.mark.parametrize("beside,messages,schedule", [("card60", 0, 0), ("xor3", 0, 2), ("xor3", 0, 1), ("xor3", 1, 2),
                                                      ("", 1, 2), ("card60", 1, 2)])
def test_windows_beside_other_families(nb, beside, messages, schedule):
    p = _windows_and(nb, beside)
    print(f"windows of {nb} Booleans beside {beside or 'nothing'}, messages {messages}, schedule {schedule}", flush=True)
    info = _compare(p, 5, 0.9, nb, messages)
    assert (info["n_big"] > 0) == (beside == "card60")
    h, a0, b0, st = _one_step(p, 5, 0.9, 0.3, 0.3, 93 + nb, schedule=schedule, messages=messages)
    _assert_step(p, a0, b0, st, 0.9, 0.3, 0.3)
    h.free()


@pytest.mark.parametrize("nb", [1, 2, 4])
@pytest.mark.parametrize("beside,extra,R", [("", 45000, 3), ("", 45000, 70), ("xor3", 45000, 3), ("card13", 300, 5)])
def test_windows_out_of_workgroup_lds(nb, beside, extra, R):
    """States of 180 KB, and message columns that leave a workgroup fewer than four waves."""
    print(f"windows of {nb} Booleans beside {beside or 'nothing'}, {extra} more Booleans, R={R}", flush=True)
    _compare(_windows_and(nb, beside, 130, extra), R, 1.2, 10 + nb)


def _table_pairs(n, L, form):
    """Index pairs whose atoms have no inline record: right-hand sides that float32 does not hold
    (tenths), or three terms."""
    rng = np.random.default_rng([94, n, L])
    b = Builder(n * L, n + 1, real_lo=np.full(n + 1, -2.0), real_hi=np.full(n + 1, 2.0))
    for j in range(n):
        for k in range(j + 1, n):
            s = float(rng.integers(1, 9)) / (10.0 if form == "tenths" else 8.0)
            more = ([], []) if form == "tenths" else ([n], [0.5])
            at = [b.atom([u, v] + more[0], [1.0, -1.0] + more[1], OP_GE, s) for u, v in ((j, k), (k, j))]
            bits = sum(([lit(i * n + j), lit(i * n + k)] for i in range(L)), [])
            b.add(KIND_EXPR, bits + [lit(a) for a in at], 0, index_differs_program(L, 2))
    return b.build()


@pytest.mark.parametrize("form", ["tenths", "terms"])
@pytest.mark.parametrize("n,L,R,schedule", [(2, 1, 1, 2), (20, 3, 5, 2), (20, 3, 5, 1), (34, 10, 65, 2)])
def test_index_pairs_through_the_atom_table(form, n, L, R, schedule):
    p = _table_pairs(n, L, form)
    print(f"index pairs of {n} items, {L} bits, {form}, R={R}, schedule {schedule}", flush=True)
    info = _compare(p, R, 1.5, n + L)
    assert info["n_pair"] == p.n_cons
    h, a0, b0, st = _one_step(p, R, 1.5, 0.5, 0.1, 95, schedule=schedule)
    _assert_step(p, a0, b0, st, 1.5, 0.5, 0.1)
    h.free()
