"""GPU parity of dynamic updates (katz_rank_update, Algorithm 2).

Each update is checked three ways: against the oracle's delta-form Algorithm 2
(parity contract), bitwise against katz_bounds on the updated graph at the same
r (the re-walk computes exactly what a static run computes), and by the status.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
import synthgraph as sg
from tests.parity import assert_topk_parity

pytestmark = pytest.mark.gpu


def K():
    import paper_1807_03847_amd.katz as katz
    return katz


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def dev(rp, col):
    return torch.from_numpy(np.asarray(rp, dtype=np.int64)).cuda(), torch.from_numpy(np.asarray(col, np.int32)).cuda()


def random_batch(rng, rp, col, n, n_ins, n_del, hub_bias=0.0):
    src = np.repeat(np.arange(n), np.diff(rp))
    mask = src < col
    und = np.stack([src[mask], col[mask]], 1)
    existing = set(map(tuple, und.tolist()))
    dels = und[rng.choice(len(und), size=min(n_del, len(und)), replace=False)] if n_del else np.zeros((0, 2), int)
    ins = set()
    deg = np.diff(rp)
    hubs = np.argsort(-deg)[:8]
    while len(ins) < n_ins:
        a = int(rng.choice(hubs)) if rng.random() < hub_bias else int(rng.integers(0, n))
        b = int(rng.integers(0, n))
        a, b = min(a, b), max(a, b)
        if a != b and (a, b) not in existing:
            ins.add((a, b))
    return np.array(sorted(ins), dtype=np.int64).reshape(-1, 2), np.asarray(dels, dtype=np.int64).reshape(-1, 2)


def check_against_static(katz, dyn_res, rp_new, col_new, alpha):
    """Bitwise: the dynamic l_r, u_r of the returned nodes equal katz_bounds on the
    new graph at the same r."""
    lo, up = katz.bounds(*dev(rp_new, col_new), dyn_res.iterations, alpha=alpha)
    ids = dyn_res.topk.long()
    assert torch.equal(lo[ids], dyn_res.lower)
    assert torch.equal(up[ids], dyn_res.upper)


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_dynamic_er_batches(seed):
    katz = K()
    rng = np.random.default_rng(seed)
    rp, col = sg.erdos_renyi(3000, 15000, 40 + seed)
    dmax = sg.max_degree(rp)
    H = 30
    alpha = 1.0 / (1 + dmax + H)
    k, eps = 40, 1e-9
    say("dyn er create", seed)
    st, res0 = katz.create_state(*dev(rp, col), k, alpha=alpha, eps=eps, degree_cap=dmax + H)
    dyn = oracle.DynamicOracle(rp, col, alpha, k=k, eps=eps, degree_cap=dmax + H)
    assert_topk_parity(res0.topk.cpu().numpy(), res0.lower.cpu().numpy(), res0.upper.cpu().numpy(), dyn.result,
                       gpu_status=res0.status)
    for b, (ni, nd) in enumerate([(1, 0), (0, 1), (5, 3), (40, 20), (300, 100), (2000, 800)]):
        ins, dels = random_batch(rng, dyn.row_ptr, dyn.col, 3000, ni, nd)
        say("dyn er batch", seed, b, ni, nd)
        res = st.update(ins, dels)
        orc = dyn.update(ins, dels)
        assert res.iterations == orc.iterations
        assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                           gpu_status=res.status)
        check_against_static(katz, res, dyn.row_ptr, dyn.col, alpha)
    st.free()


def test_dynamic_rmat_hubs_and_relocation():
    """Skewed graph with segmented hub rows; insertions concentrated on hubs force
    row relocation in the slack pool; a large batch takes the dense re-walk."""
    katz = K()
    rng = np.random.default_rng(7)
    rp, col = sg.rmat(15, seed=3)
    n = len(rp) - 1
    dmax = sg.max_degree(rp)
    H = 5000
    alpha = 1.0 / (1 + dmax + H)
    k, eps = 200, 1e-7
    say("dyn rmat create")
    st, res0 = katz.create_state(*dev(rp, col), k, alpha=alpha, eps=eps, degree_cap=dmax + H)
    cur_rp, cur_col = rp, col
    for b, (ni, nd, bias) in enumerate([(10, 5, 0.9), (800, 10, 0.8), (3000, 3000, 0.2), (1, 1, 0.0)]):
        ins, dels = random_batch(rng, cur_rp, cur_col, n, ni, nd, hub_bias=bias)
        say("dyn rmat batch", b, ni, nd)
        res = st.update(ins, dels)
        # New graph on the host.
        src = np.repeat(np.arange(n), np.diff(cur_rp))
        keys = set(zip(src.tolist(), cur_col.tolist()))
        for a, c in dels:
            keys.discard((a, c))
            keys.discard((c, a))
        for a, c in ins:
            keys.add((a, c))
            keys.add((c, a))
        arr = np.array(sorted(keys), dtype=np.int64)
        cur_rp, cur_col = sg.from_edges(n, arr[:, 0], arr[:, 1], undirected=False)
        check_against_static(katz, res, cur_rp, cur_col, alpha)
        orc = oracle.rank_static(cur_rp, cur_col, alpha, k, eps)
        # The dynamic r never shrinks (it may exceed the static one); compare the
        # certified rankings through the oracle's tie groups at its own r.
        assert res.status == orc.status == oracle.OK
        assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                           check_status=False)
    st.free()


def rmat_batch(pool, rng, rp, col, n, size):
    """One serving-shaped batch: 70% insertions whose endpoints come from the
    graph's own R-MAT distribution (``pool``, consumed from the front;
    self-loops, present edges and repeats rejected), 30% deletions of present
    edges, uniform."""
    n_del = int(round(0.3 * size))
    n_ins = size - n_del
    src = np.repeat(np.arange(n, dtype=np.int64), np.diff(rp))
    keys = src * n + col
    und = np.nonzero(src < col)[0]
    di = rng.choice(und, size=n_del, replace=False) if n_del else np.zeros(0, np.int64)
    dels = np.stack([src[di], col[di].astype(np.int64)], 1)
    ins, seen, used = [], set(), 0
    while len(ins) < n_ins:
        a, b = (int(v) for v in pool[used])
        used += 1
        a, b = min(a, b), max(a, b)
        key = a * n + b
        pos = np.searchsorted(keys, key)
        if a != b and (a, b) not in seen and not (pos < keys.size and keys[pos] == key):
            seen.add((a, b))
            ins.append((a, b))
    return np.array(ins, dtype=np.int64).reshape(-1, 2), dels, pool[used:]


def test_dynamic_rmat18_serving_batches():
    """R-MAT scale 18 with the serving workload's batches: sizes up to 10^4
    edges, R-MAT-distributed insertions (hub-heavy), deletions of present
    edges; each result against the oracle's Algorithm 2 (and its r), and
    bitwise against katz_bounds on the updated graph.  The large batches take
    the dense re-walk and relocate hub rows in the slack pool."""
    katz = K()
    rng = np.random.default_rng(18)
    rp, col = sg.rmat(18, seed=5)
    n = len(rp) - 1
    dmax = sg.max_degree(rp)
    H = 20000
    alpha = 1.0 / (1 + dmax + H)
    k, eps = 100, 1e-6
    pool = sg.rmat_pairs(18, 60000, seed=5, stream=11)
    say("dyn rmat18 create", n, int(rp[-1]))
    st, res0 = katz.create_state(*dev(rp, col), k, alpha=alpha, eps=eps, degree_cap=dmax + H)
    dyn = oracle.DynamicOracle(rp, col, alpha, k=k, eps=eps, degree_cap=dmax + H)
    assert_topk_parity(res0.topk.cpu().numpy(), res0.lower.cpu().numpy(), res0.upper.cpu().numpy(), dyn.result,
                       gpu_status=res0.status)
    for b, size in enumerate([1, 3, 40, 700, 10000, 2500]):
        ins, dels, pool = rmat_batch(pool, rng, dyn.row_ptr, dyn.col, n, size)
        say("dyn rmat18 batch", b, len(ins), len(dels))
        res = st.update(ins, dels)
        orc = dyn.update(ins, dels)
        assert res.iterations == orc.iterations
        assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                           gpu_status=res.status)
        check_against_static(katz, res, dyn.row_ptr, dyn.col, alpha)
    st.free()


def test_node_insertion_and_deletion_through_isolated_padding():
    """Node insertions and deletions through isolated padding nodes (Section 4:
    the initial graph carries enough isolated nodes): inserting a node is
    inserting edges at a padding node, deleting a node is deleting all of its
    edges.  Each step against the oracle's Algorithm 2, and a deleted node ends
    with exact zero bounds."""
    katz = K()
    rng = np.random.default_rng(4)
    base_rp, base_col = sg.erdos_renyi(2000, 8000, 12)
    rp, col = sg.with_isolated(base_rp, base_col, 64)          # nodes 2000..2063: padding
    n = len(rp) - 1
    dmax = sg.max_degree(rp)
    H = 60
    alpha = 1.0 / (1 + dmax + H)
    k, eps = 30, 1e-9
    say("padding create")
    st, _ = katz.create_state(*dev(rp, col), k, alpha=alpha, eps=eps, degree_cap=dmax + H)
    dyn = oracle.DynamicOracle(rp, col, alpha, k=k, eps=eps, degree_cap=dmax + H)
    hub = int(np.argmax(np.diff(rp)))
    # New nodes 2000 and 2001: 2000 joins ten existing nodes and the hub, 2001
    # joins 2000 and forty existing nodes (it becomes a high-degree node).
    nb0 = [int(v) for v in rng.choice(np.setdiff1d(np.arange(2000), [hub]), 10, replace=False)] + [hub]
    nb1 = [int(v) for v in rng.choice(2000, 40, replace=False)]
    steps = [(np.array([[min(2000, v), max(2000, v)] for v in nb0]), None),
             (np.array([[2000, 2001]] + [[v, 2001] for v in nb1]), None)]
    # Delete node 17: all of its current edges.
    for ins, dels in steps:
        say("padding insert", len(ins))
        res = st.update(ins, dels)
        orc = dyn.update(ins, dels)
        assert res.iterations == orc.iterations
        assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                           gpu_status=res.status)
    v = 17
    nbrs = dyn.col[dyn.row_ptr[v]:dyn.row_ptr[v + 1]].astype(np.int64)
    dels = np.stack([np.minimum(v, nbrs), np.maximum(v, nbrs)], 1)
    say("padding delete node", v, len(dels))
    res = st.update(None, dels)
    orc = dyn.update(None, dels)
    assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                       gpu_status=res.status)
    # The isolated node's bounds: zero in a static run on the new graph; the
    # oracle's delta form keeps only the rounding residue of its updates.
    assert abs(orc.lower_all[v]) < 1e-15 and abs(orc.upper_all[v]) < 1e-15
    lo, up = katz.bounds(*dev(dyn.row_ptr, dyn.col), res.iterations, alpha=alpha)
    assert lo[v].item() == up[v].item() == 0.0
    st.free()


@pytest.mark.parametrize("tuning", [None, (65536, 1, 4), (16384, 4, 0)])
def test_state_renumbering_is_invisible(tuning):
    """A state renumbered by degree class (the default) and one in caller order
    (KATZ_FLAG_NO_REORDER) give bitwise the same results through updates,
    also under tuned launch shapes whose LDS copy of the hottest entries serves
    the dense re-walk levels and the resumed iterations."""
    katz = K()
    saved = katz.tuning_get()
    try:
        if tuning:
            katz.tuning_set(tuning[0], tuning[1], walk_groups=tuning[2])
        rng = np.random.default_rng(21)
        rp, col = sg.rmat(14, seed=8)
        n = len(rp) - 1
        dmax = sg.max_degree(rp)
        H = 3000
        alpha = 1.0 / (1 + dmax + H)
        say("state renumbering", tuning)
        st_a, ra = katz.create_state(*dev(rp, col), 50, alpha=alpha, eps=1e-8, degree_cap=dmax + H)
        st_b, rb = katz.create_state(*dev(rp, col), 50, alpha=alpha, eps=1e-8, degree_cap=dmax + H,
                                     flags=katz.FLAG_NO_REORDER)
        dyn = oracle.DynamicOracle(rp, col, alpha, k=50, eps=1e-8, degree_cap=dmax + H)
        results = [(ra, rb, dyn.result)]
        for ni, nd, bias in [(3, 1, 0.5), (200, 50, 0.6), (6000, 2000, 0.3), (1, 0, 0.0)]:
            ins, dels = random_batch(rng, dyn.row_ptr, dyn.col, n, ni, nd, hub_bias=bias)
            results.append((st_a.update(ins, dels), st_b.update(ins, dels), dyn.update(ins, dels)))
        for a, b, orc in results:
            assert torch.equal(a.topk.cpu(), b.topk.cpu())
            assert torch.equal(a.lower.cpu(), b.lower.cpu()) and torch.equal(a.upper.cpu(), b.upper.cpu())
            assert (a.iterations, a.status) == (b.iterations, b.status)
            assert_topk_parity(a.topk.cpu().numpy(), a.lower.cpu().numpy(), a.upper.cpu().numpy(), orc,
                               gpu_status=a.status)
        st_a.free()
        st_b.free()
    finally:
        katz.tuning_set(**saved)


def test_dynamic_rejections_leave_state_unchanged():
    katz = K()
    rp, col = sg.erdos_renyi(500, 2000, 9)
    dmax = sg.max_degree(rp)
    alpha = 1.0 / (2 + dmax)
    say("dyn reject create")
    st, _ = katz.create_state(*dev(rp, col), 10, alpha=alpha, eps=1e-9, degree_cap=dmax + 1)
    src = np.repeat(np.arange(500), np.diff(rp))
    e0 = (int(src[0]), int(col[0]))
    absent = next((a, b) for a in range(500) for b in range(a + 1, 500)
                  if b not in set(col[rp[a]:rp[a + 1]].tolist()))
    bad = [([e0], []), ([], [absent]), ([(3, 3)], []), ([(0, 600)], []), ([absent, absent[::-1]], []),
           ([absent], [absent])]
    for ins, dels in bad:
        with pytest.raises(katz.KatzError) as e:
            st.update(np.array(ins).reshape(-1, 2), np.array(dels).reshape(-1, 2))
        assert e.value.code == katz.E_UPDATE
    hub = int(np.argmax(np.diff(rp)))
    nbrs = set(col[rp[hub]:rp[hub + 1]].tolist())
    extra = [(min(hub, v), max(hub, v)) for v in range(500) if v != hub and v not in nbrs][:2]
    with pytest.raises(katz.KatzError) as e:
        st.update(np.array(extra), None)
    assert e.value.code == katz.E_DEGREE_CAP
    # A valid batch still gives the static answer on the updated graph.
    res = st.update(np.array([absent]), None)
    dyn = oracle.DynamicOracle(rp, col, alpha, k=10, eps=1e-9, degree_cap=dmax + 1)
    orc = dyn.update(np.array([absent]), None)
    assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                       gpu_status=res.status)
    st.free()


def test_empty_batch_is_a_noop():
    katz = K()
    rp, col = sg.erdos_renyi(800, 3000, 2)
    st, r0 = katz.create_state(*dev(rp, col), 15, eps=1e-9)
    say("dyn empty batch")
    r1 = st.update(None, None)
    assert torch.equal(r0.topk, r1.topk) and torch.equal(r0.lower, r1.lower)
    assert r1.iterations == r0.iterations
    st.free()


def test_host_outputs_match_device_outputs():
    """States created from host buffers write their results into host memory
    (creation and every update) through device staging; results equal the
    device-memory path bitwise."""
    katz = K()
    rng = np.random.default_rng(11)
    rp, col = sg.erdos_renyi(1500, 6000, 21)
    n = len(rp) - 1
    dmax = sg.max_degree(rp)
    alpha, cap, k = 1.0 / (dmax + 40), dmax + 39, 20
    say("host outputs", n)
    st_h, r_h = katz.create_state(torch.from_numpy(rp), torch.from_numpy(col), k, alpha=alpha, eps=1e-9,
                                  degree_cap=cap)
    st_d, r_d = katz.create_state(*dev(rp, col), k, alpha=alpha, eps=1e-9, degree_cap=cap)
    assert r_h.topk.device.type == "cpu"
    assert np.array_equal(r_h.topk.numpy(), r_d.topk.cpu().numpy())
    assert np.array_equal(r_h.lower.numpy(), r_d.lower.cpu().numpy())
    for _ in range(3):
        ins, dels = random_batch(rng, rp, col, n, 12, 4)
        a = st_h.update(ins, dels)
        b = st_d.update(ins, dels)
        assert a.topk.device.type == "cpu"
        assert np.array_equal(a.topk.numpy(), b.topk.cpu().numpy())
        assert np.array_equal(a.lower.numpy(), b.lower.cpu().numpy())
        assert np.array_equal(a.upper.numpy(), b.upper.cpu().numpy())
        assert (a.iterations, a.status) == (b.iterations, b.status)
        e = np.concatenate([ins, ins[:, ::-1]]) if len(ins) else np.zeros((0, 2), np.int64)
        d = np.concatenate([dels, dels[:, ::-1]]) if len(dels) else np.zeros((0, 2), np.int64)
        src = np.repeat(np.arange(n), np.diff(rp))
        keep = np.ones(len(src), bool)
        dset = set(map(tuple, d.tolist()))
        for j, (u, v) in enumerate(zip(src.tolist(), col.tolist())):
            if (u, v) in dset:
                keep[j] = False
        rp, col = sg.from_edges(n, np.concatenate([src[keep], e[:, 0]]), np.concatenate([col[keep], e[:, 1]]),
                                undirected=False)
    st_h.free()
    st_d.free()


@pytest.mark.parametrize("undirected", [True, False])
def test_state_save_and_load_resume_bitwise(tmp_path, undirected):
    """A state saved after two batches and loaded again answers the next batches
    bitwise as the original state does, and as the oracle's Algorithm 2 does;
    a truncated or foreign file is refused."""
    katz = K()
    rng = np.random.default_rng(4)
    if undirected:
        rp, col = sg.rmat(13, seed=5)
    else:
        rp, col = sg.rmat_directed(12, 8, seed=6)
    n = len(rp) - 1
    dmax = sg.max_degree(rp)
    alpha = 1.0 / (1 + dmax + 100)
    say("state save create", undirected)
    st, _ = katz.create_state(*dev(rp, col), 25, alpha=alpha, eps=1e-9, degree_cap=dmax + 100, undirected=undirected)
    dyn = oracle.DynamicOracle(rp, col, alpha, k=25, eps=1e-9, undirected=undirected, degree_cap=dmax + 100)

    def batch(size):
        src = np.repeat(np.arange(n), np.diff(dyn.row_ptr))
        arcs = np.stack([src, dyn.col], 1)
        if undirected:
            arcs = arcs[arcs[:, 0] < arcs[:, 1]]
        present = set(map(tuple, arcs.tolist()))
        dels = arcs[rng.choice(len(arcs), size // 3, replace=False)]
        ins = set()
        while len(ins) < size:
            a, b = (int(v) for v in rng.integers(0, n, 2))
            if undirected:
                a, b = min(a, b), max(a, b)
            if a != b and (a, b) not in present:
                ins.add((a, b))
        return np.array(sorted(ins)), dels

    for size in (30, 300):
        ins, dels = batch(size)
        st.update(ins, dels)
        dyn.update(ins, dels)
    path = tmp_path / "state.bin"
    st.save(path)
    st2 = katz.load_state(path)
    for size in (5, 500, 1):
        ins, dels = batch(size)
        say("state save batch", undirected, size)
        a = st.update(ins, dels)
        b = st2.update(ins, dels)
        orc = dyn.update(ins, dels)
        assert torch.equal(a.topk, b.topk) and torch.equal(a.lower, b.lower) and torch.equal(a.upper, b.upper)
        assert (a.iterations, a.status) == (b.iterations, b.status)
        assert_topk_parity(b.topk.cpu().numpy(), b.lower.cpu().numpy(), b.upper.cpu().numpy(), orc,
                           gpu_status=b.status)
    st.free()
    st2.free()
    data = path.read_bytes()
    (tmp_path / "short.bin").write_bytes(data[:len(data) // 2])
    (tmp_path / "junk.bin").write_bytes(b"not a state" * 20)
    for bad in ("short.bin", "junk.bin", "missing.bin"):
        with pytest.raises(katz.KatzError) as e:
            katz.load_state(tmp_path / bad)
        assert e.value.code == katz.E_INVALID_ARG


def _apply(n, rp, col, ins, dels, undirected=True):
    src = np.repeat(np.arange(n, dtype=np.int64), np.diff(rp))
    key = src * n + col
    both = lambda p: np.concatenate([p[:, 0] * n + p[:, 1]] + ([p[:, 1] * n + p[:, 0]] if undirected else []))
    key = np.concatenate([key[~np.isin(key, both(dels))], both(ins)])
    return sg.from_edges(n, key // n, key % n, undirected=False)


@pytest.mark.parametrize("hub_len", [4095, 4096, 4097, 8192, 12289])
@pytest.mark.parametrize("flags", [0, 1])
def test_merge_chunk_edges(hub_len, flags):
    """Updates of a hub whose row ends just before, at and past a 4096-entry merge
    chunk: entries deleted and inserted at both ends of the row and on both sides
    of every chunk boundary, a row emptied, an empty row filled; then undone."""
    katz = K()
    say("merge chunks", hub_len, flags)
    n = 3 * hub_len + 50
    nbr = 10 + 3 * np.arange(hub_len)                  # gaps of two ids between the hub's neighbours
    extra = np.stack([nbr[:-1:7], nbr[1::7][:nbr[:-1:7].size]], 1)
    extra = np.concatenate([extra, [[0, 2]]])
    src = np.concatenate([np.full(hub_len, 1), extra[:, 0]])
    rp, col = sg.from_edges(n, src, np.concatenate([nbr, extra[:, 1]]))
    alpha = 1.0 / (1 + sg.max_degree(rp) + 3000)
    st, _ = katz.create_state(*dev(rp, col), 20, alpha=alpha, eps=1e-9, degree_cap=sg.max_degree(rp) + 3000, flags=flags)
    edge = sorted({p for b in range(0, hub_len + 1, 4096) for p in (b - 2, b - 1, b, b + 1) if 0 <= p < hub_len} |
                  {0, 1, hub_len - 2, hub_len - 1})
    dels = np.array([[1, nbr[p]] for p in edge] + [[0, 2]], dtype=np.int64)        # node 0's row becomes empty
    ins = [[1, nbr[p] + 1] for p in edge] + [[1, nbr[p] - 1] for p in edge] + [[3, 4], [1, 5], [1, n - 1]]
    ins += [[1, v] for v in nbr[hub_len // 2:hub_len // 2 + 600] + 2 if [1, v] not in ins]   # outgrows its capacity or not
    ins = np.unique(np.array(ins, dtype=np.int64), axis=0)
    for add, drop in ((ins, dels), (dels, ins), (ins, dels)):
        res = st.update(add, drop)
        rp, col = _apply(n, rp, col, add, drop)
        check_against_static(katz, res, rp, col, alpha)
    st.free()


def test_state_with_more_hubs_than_a_binning_workgroup_holds():
    """1100 rows of several segments side by side (a renumbered state puts them
    first): their segment tables come from one 1024-row binning workgroup and the
    next.  Updates re-bin them; results stay bitwise a static run's."""
    katz = K()
    say("many hubs")
    hubs, leaves = 1100, 4200
    n = hubs + leaves
    a, b = np.meshgrid(np.arange(hubs), hubs + np.arange(leaves), indexing="ij")
    rp, col = sg.from_edges(n, a.ravel(), b.ravel())
    alpha = 1.0 / (1 + sg.max_degree(rp) + 10)
    st, _ = katz.create_state(*dev(rp, col), 10, alpha=alpha, eps=1e-9, degree_cap=sg.max_degree(rp) + 10, max_iter=6)
    ins = np.array([[0, 1], [2, 7], [1098, 1099]], dtype=np.int64)
    dels = np.array([[5, hubs], [1099, n - 1]], dtype=np.int64)
    res = st.update(ins, dels)
    rp, col = _apply(n, rp, col, ins, dels)
    check_against_static(katz, res, rp, col, alpha)
    st.free()


BINS_CHILD = r"""
side = 260
n = side * side
i = np.arange(n).reshape(side, side)
a = np.concatenate([i[:, :-1].ravel(), i[:-1].ravel()])
b = np.concatenate([i[:, 1:].ravel(), i[1:].ravel()])
rng = np.random.default_rng(2)
keep = rng.random(len(a)) >= 0.2
rp, col = sg.from_edges(n, a[keep], b[keep])
dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=t))).cuda()
state, res = katz.create_state(dev(rp, np.int64), dev(col, np.int32), 20, alpha=0.1, eps=1e-6, degree_cap=6)
whole = lambda log: sum("prep_place" in name and "SlackRows" in name for name, _ in log)
gone = np.stack([a[~keep], b[~keep]], 1)[:64].astype(np.int32)
for step, batch in enumerate(gone.reshape(8, 8, 2)):
    print("[gpu-case] update", step, flush=True)
    before = res.iterations
    res, log = launches(lambda: state.update(batch))
    assert res.status == katz.OK
    print("iterations", before, res.iterations, "binned", whole(log), "launches", len(log), flush=True)
    # The creation walked the whole graph, so the first update may bin it ahead of a walk.
    if step > 0 and last == before == res.iterations:
        assert whole(log) == 0
        print("small", flush=True)
    last = before
"""


def test_small_updates_leave_the_whole_graph_unbinned(tmp_path):
    """Updates whose affected set stays small, as on a grid, do not bin the whole graph:
    they walk it only where the ranking takes further iterations."""
    from tests.launch_log import run_child
    say("bins of small updates")
    out = run_child(tmp_path, BINS_CHILD)
    assert out.count("small") >= 3


RECHECK_CHILD = r"""
for n, wide in ((16384, 0), (16390, 1), (60000, 1)):
    rp, col = sg.erdos_renyi(n, 3 * n, 1)
    rp, col = torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda()
    # eps = 1 keeps every node, so the re-check is over all of them.
    state, res = katz.create_state(rp, col, 50, eps=1.0, max_iter=2, precision=sys.argv[2])
    again, log = launches(lambda: state.update())
    names = [name for name, _ in log]
    print("[gpu-case] re-check", n, sum("sel_hist0" in m for m in names), sum("select_wg" in m for m in names), flush=True)
    assert sum("sel_hist0" in m for m in names) == wide and sum("select_wg" in m for m in names) == 1 - wide
    assert torch.equal(res.topk, again.topk) and torch.equal(res.lower, again.lower)
    assert (res.active_final, res.status) == (again.active_final, again.status)
    state.free()
print("ok")
"""


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_large_active_sets_are_rechecked_by_the_whole_device(tmp_path, precision):
    """The selection of an update's re-check: one workgroup up to 16384 active nodes,
    the device-wide one above, with the same result."""
    from tests.launch_log import run_child
    say("re-check of large sets", precision)
    assert run_child(tmp_path, RECHECK_CHILD, precision).rstrip().endswith("ok")
