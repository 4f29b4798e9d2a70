"""Tiles of index pairs and clause pairs, windows, and states beyond LDS at the parity bar itself,
coordinate by coordinate against the oracle, without the comparison with the general passes that
the rectangles' cancelling selectors need."""
import pytest

import workloads as W

from gpu_util import torch

pytestmark = pytest.mark.gpu
fsmt = pytest.importorskip("paper_2603_22877_amd")
from test_gpu_mixed_families import _compare  # noqa: E402
from test_gpu_tiles import _clause_pairs, _index_pairs, _with_extra_bools  # noqa: E402
from test_gpu_windows import _windows  # noqa: E402

INF = float("inf")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# two items (one constraint) are not here: at kappa 4 its false mass is near 1e-17, below the oracle's
# own resolution (it forms P[literal False] as 1 - p in 64 bits)
@pytest.mark.parametrize("n,L,D", [(9, 2, 2), (20, 7, 1), (20, 8, 2), (11, 9, 2), (26, 10, 1), (26, 10, 2)])
@pytest.mark.parametrize("R,kap", [(1, 1.5), (4, INF), (66, 4.0)])
def test_index_pairs(n, L, D, R, kap):
    print(f"index pairs: {n} items, {L} bits, {D} dimensions, R={R}, kappa={kap}", flush=True)
    _compare(_index_pairs(n, L, D, 0), R, kap, n)


@pytest.mark.parametrize("n,groups,drop,flip,shared", [(3, 1, 0.0, False, False), (9, 1, 0.0, True, False),
                                                       (40, 3, 0.3, False, False), (65, 4, 0.2, True, False),
                                                       (40, 3, 0.0, False, True)])
@pytest.mark.parametrize("R,kap", [(1, 0.3), (5, INF), (65, 0.0)])
def test_clause_pairs(n, groups, drop, flip, shared, R, kap):
    print(f"clause pairs: {n} jobs, {groups} machines, R={R}, kappa={kap}", flush=True)
    _compare(_clause_pairs(n, groups, 0, drop, flip, shared), R, kap, n)


@pytest.mark.parametrize("nb,n_cons", [(1, 5), (3, 64), (10, 130)])
@pytest.mark.parametrize("two_vars,neg_atoms", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("R,kap", [(1, 0.8), (5, INF), (70, 3.0)])
def test_windows(nb, n_cons, two_vars, neg_atoms, R, kap):
    print(f"windows: {nb} Booleans, {n_cons} constraints, R={R}, kappa={kap}", flush=True)
    _compare(_windows(nb, n_cons, 0, two_vars, neg_atoms), R, kap, nb)


@pytest.mark.parametrize("extra", [15000, 45000])
@pytest.mark.parametrize("make", ["bits1", "bits2", "rect"])
def test_states_beyond_lds(make, extra):
    p = {"rect": lambda: W.make_placement(40, W.seed_seq(74), fill=0.3, max_side=5),
         "bits1": lambda: _index_pairs(33, 5, 1, 2), "bits2": lambda: _index_pairs(33, 9, 2, 3)}[make]()
    print(f"{make} with {extra} more variables", flush=True)
    _compare(_with_extra_bools(p, extra), 3, 0.5, 6)


@pytest.mark.parametrize("R", [1, 6])
def test_clause_pairs_beyond_lds(R):
    _compare(W.make_scheduling(520, 3, W.seed_seq(78), n_prec=3), R, 0.1, 7)


@pytest.mark.parametrize("n_rect", [65, 131])
@pytest.mark.parametrize("R,kap", [(1, 0.15), (70, 0.6), (3, INF)])
def test_rectangle_pairs(n_rect, R, kap):
    """Enough constraints on every variable that no coordinate is one cancelling pair."""
    print(f"{n_rect} rectangles, R={R}, kappa={kap}", flush=True)
    _compare(W.make_placement(n_rect, W.seed_seq(72, n_rect, 20), fill=0.3, max_side=20), R, kap, n_rect)
