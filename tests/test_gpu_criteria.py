"""GPU parity of the stopping criteria of Section 3.1 beyond the LDS-sized
top-k test, through the C ABI: top-k with k > 4096 (device-wide sort of the
ranked list), the ranking criterion (k = n), the score criterion (u - l < eps
for every node, all nodes listed) and the pair criterion; and the separated
pairs of Table 1."""
import sys

import numpy as np
import pytest
import torch

import synthgraph as sg
from oracle import katz as OK
from tests.parity import assert_topk_parity

pytestmark = pytest.mark.gpu

TAU = 1e-12


def K():
    import paper_1807_03847_amd.katz as katz
    return katz


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def dev(rp, col):
    return (torch.from_numpy(np.asarray(rp, dtype=np.int64)).cuda(),
            torch.from_numpy(np.asarray(col, dtype=np.int32)).cuda())


CODES = {"topk": OK.TOPK, "ranking": OK.RANKING, "score": OK.SCORE, "pair": OK.PAIR}


def run_both(rp, col, criterion, k=1, eps=0.0, precision="fp64", pair=(0, 1), max_iter=0):
    a = 1.0 / (1 + sg.max_degree(rp))
    orc = OK.rank_static(rp, col, a, k, eps, max_iter=max_iter or 1000, criterion=CODES[criterion],
                         pair=pair if criterion == "pair" else None)
    rp_t, col_t = dev(rp, col)
    res = K().rank_static(rp_t, col_t, k, alpha=a, eps=eps, precision=precision, criterion=criterion, pair=pair,
                          max_iter=max_iter)
    torch.cuda.synchronize()
    return orc, res


def check(orc, res, fp32=False):
    ids = res.topk.cpu().numpy()
    lo = res.lower.cpu().numpy()
    up = res.upper.cpu().numpy()
    assert_topk_parity(ids, lo, up, orc, TAU, widened=fp32, check_status=True, gpu_status=res.status)
    assert np.all(lo[:-1] >= lo[1:]), "output not in lower-bound order"
    if not fp32:
        assert res.iterations == orc.iterations
    return ids, lo, up


@pytest.mark.parametrize("k", [4097, 5000, 12289])
def test_topk_beyond_lds_sort(k):
    """k past one workgroup's LDS sort: the ranked list is sorted device-wide
    (several tiles, global passes, a ragged last tile)."""
    say("topk large k", k)
    rp, col = sg.rmat(14, 16, seed=5)
    orc, res = run_both(rp, col, "topk", k=k, eps=1e-6)
    check(orc, res)
    assert res.active_final == orc.active_final


def test_topk_large_k_fp32():
    """FP32 form with k = 6000 on ER: eps = 1e-5 lies above twice the rounding
    margin of these scores, so the FP32 form certifies what the oracle does
    (at eps = 1e-6 neighbours of the ER top-6000 are closer than the margin
    can resolve and the run stops with W_PRECISION_LIMIT)."""
    say("topk large k fp32")
    rp, col = sg.erdos_renyi(16384, 131072, 2)
    orc, res = run_both(rp, col, "topk", k=6000, eps=1e-5, precision="fp32")
    check(orc, res, fp32=True)


@pytest.mark.parametrize("n,eps", [(3000, 1e-9), (16384, 1e-9)])
def test_ranking_er(n, eps):
    """Ranking criterion (k = n): one workgroup's sort while n <= 4096, the
    device-wide sort beyond."""
    say("ranking er", n)
    rp, col = sg.erdos_renyi(n, 8 * n, 3)
    orc, res = run_both(rp, col, "ranking", eps=eps, max_iter=300)
    ids, lo, up = check(orc, res)
    assert len(ids) == n and len(set(ids.tolist())) == n
    assert res.rest_upper_max == -np.inf
    # Separated pairs: the kernel's count on the returned bounds is exact; the
    # oracle's value on its own bounds agrees up to pairs that FP64 rounding
    # order can flip.
    assert res.separated_fraction == OK.separated_fraction(lo, up)
    assert abs(res.separated_fraction - OK.separated_fraction(orc.lower_all, orc.upper_all)) <= 1e-6


@pytest.mark.parametrize("n,m,eps", [(4097, 4, 1e-9), (6144, 8, 1e-9), (6145, 8, 1e-7), (8192, 3, 0.0), (10241, 5, 1e-8)])
def test_ranking_tile_edges(n, m, eps):
    """Lists that end just before, at and just past a 2048-record tile and a
    merged run: the tile test decides most iterations, the last ones go through
    the sort; r and the order equal the oracle's (sparse graphs with m = 3..5
    hold exact ties, which with eps = 0 run into the iteration limit)."""
    say("ranking tile edges", n)
    rp, col = sg.erdos_renyi(n, m * n, 11)
    orc, res = run_both(rp, col, "ranking", eps=eps, max_iter=60)
    ids, lo, up = check(orc, res)
    assert sorted(ids.tolist()) == list(range(n))


def test_ranking_rmat_ties_fp32():
    """R-MAT with isolated nodes (exact ties, separated only by eps) in the
    FP32 form: the widened intervals contain the oracle's."""
    say("ranking rmat fp32")
    rp, col = sg.rmat(13, 16, seed=2)
    orc, res = run_both(rp, col, "ranking", eps=1e-5, precision="fp32", max_iter=100)
    ids, lo, up = check(orc, res, fp32=True)
    assert res.separated_fraction == OK.separated_fraction(lo, up)


@pytest.mark.parametrize("precision,eps", [("fp64", 1e-6), ("fp64", 1e-9), ("fp32", 1e-5)])
def test_score_criterion(precision, eps):
    say("score", precision, eps)
    rp, col = sg.rmat(13, 16, seed=4)
    orc, res = run_both(rp, col, "score", eps=eps, precision=precision)
    ids, lo, up = check(orc, res, fp32=precision == "fp32")
    assert len(ids) == len(rp) - 1
    assert np.all(up - lo < eps) or res.status != K().OK
    assert res.active_final == len(rp) - 1
    assert res.separated_fraction == OK.separated_fraction(lo, up)


def test_pair_criterion():
    say("pair")
    rp, col = sg.erdos_renyi(16384, 131072, 1)
    full = OK.rank_static(rp, col, None, 40, 0.0)
    # Pairs: neighbours in the top list (close scores), a top node against the
    # last node, and two nodes given in reversed order.
    pairs = [(int(full.topk[0]), int(full.topk[1])), (int(full.topk[39]), int(full.topk[38])),
             (int(full.topk[5]), 16383), (7, 9)]
    for pair in pairs:
        for eps in (0.0, 1e-6):
            orc, res = run_both(rp, col, "pair", eps=eps, pair=pair)
            ids, lo, up = check(orc, res)
            assert sorted(ids.tolist()) == sorted(pair)
            assert res.active_final == 2
            assert abs(res.rest_upper_max - orc.rest_upper_max) <= 1e-12 * orc.rest_upper_max


def test_pair_exact_tie_stops_on_iteration_limit():
    """Two leaves of a star are true ties: eps = 0 cannot separate them."""
    say("pair tie")
    rp, col = sg.star_graph(50)
    orc, res = run_both(rp, col, "pair", eps=0.0, pair=(3, 4), max_iter=20)
    assert res.status == orc.status == K().W_ITER_LIMIT
    assert res.topk.cpu().tolist() == [3, 4] == orc.topk.tolist()


@pytest.mark.parametrize("n,k", [(20000, 16384), (20000, 16385), (16385, 16385), (45000, 40961)])
def test_long_lists_on_both_sides_of_the_gated_sort(n, k):
    """Up to 16384 entries the sort is launched in every iteration and returns at once
    where it is not needed, longer lists are sorted when the host has seen that they
    have to be: the list of every iteration limit, and the certified one, is the head of
    all nodes by lower bound, then id."""
    katz = K()
    rp, col = sg.erdos_renyi(n, 6 * n, 3)
    rp_t, col_t = dev(rp, col)
    for r in (1, 2, 5, 60):
        say("long lists", n, k, r)
        a = katz.rank_static(rp_t, col_t, k, eps=1e-3, max_iter=r)
        lo, up = katz.bounds(rp_t, col_t, a.iterations)
        ids = torch.argsort(lo, descending=True, stable=True)[:k]
        assert torch.equal(a.topk.long(), ids)
        assert torch.equal(a.lower, lo[ids]) and torch.equal(a.upper, up[ids])
        assert (a.status == katz.OK) == (a.iterations < r)


WAITS_CHILD = r"""
rp, col = sg.erdos_renyi(30000, 240000, 5)
rp, col = torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda()
waits = {}
for r in (4, 12):
    res, log = launches(lambda: katz.rank_static(rp, col, 5000, eps=1e-13, max_iter=r))
    assert res.iterations == r
    waits[r] = shim.log_syncs()
    print("[gpu-case] waits", r, waits[r], len(log), flush=True)
assert waits[4] == waits[12]
print("ok")
"""


def test_lists_past_the_lds_sort_do_not_stop_the_host_each_iteration(tmp_path):
    """k = 5000: the iterations' flags come back one behind, with no wait for the stream
    in any of them."""
    from tests.launch_log import run_child
    say("waits of long lists")
    assert run_child(tmp_path, WAITS_CHILD).rstrip().endswith("ok")
