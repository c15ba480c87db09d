"""GPU parity under other row-length classes of the degree binning
(katz_tuning.bin_bounds, searched by katz_autotune).  The classes decide how
many lanes sum a row, so they change the order of additions: results must
still equal the oracle's within the parity contract, batches must still be
bitwise their single-graph calls, and a state must keep the classes of its
creation so that its re-walks stay bitwise a static run's."""
import sys

import numpy as np
import pytest
import torch

import oracle
import synthgraph as sg
from tests.parity import assert_topk_parity

pytestmark = pytest.mark.gpu

TABLES = [[4, 8, 16, 64, 256, 2048], [2, 4, 8, 16, 64, 512], [4, 8, 24, 48, 192, 1536], [1, 2, 3, 5, 9, 17]]


def K():
    import paper_1807_03847_amd.katz as katz
    return katz


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def dev(rp, col):
    return torch.from_numpy(np.asarray(rp, dtype=np.int64)).cuda(), torch.from_numpy(np.asarray(col, np.int32)).cuda()


@pytest.fixture
def katz():
    k = K()
    saved = k.tuning_get()
    yield k
    k.tuning_set(**saved)


@pytest.mark.parametrize("table", TABLES)
def test_bin_tables_static_parity(katz, table):
    graphs = [("rmat14", sg.rmat(14, seed=6), True), ("ba", sg.barabasi_albert(20000, 6, 3), True),
              ("rmatd12", sg.rmat_directed(12, 8, seed=7), False)]
    for hub, bpc, groups in ((0, 0, 0), (159744, 1, 4)):
        katz.tuning_set(hub, bpc, walk_groups=groups, bin_bounds=table)
        for name, (rp, col), und in graphs:
            say("bins static", table, hub, name)
            alpha = 1.0 / (1 + sg.max_degree(rp))
            orc = oracle.rank_static(rp, col, alpha, 60, 1e-9, undirected=und)
            for precision in ("fp64", "fp32"):
                res = katz.rank_static(*dev(rp, col), 60, alpha=alpha, eps=1e-9 if precision == "fp64" else 1e-6,
                                       precision=precision, undirected=und)
                if precision == "fp32":
                    orc32 = oracle.rank_static(rp, col, alpha, 60, 1e-6, undirected=und)
                    if res.status == katz.W_PRECISION_LIMIT:
                        continue
                    assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(),
                                       orc32, widened=True, gpu_status=res.status)
                else:
                    assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(),
                                       orc, gpu_status=res.status)
            lo, up = katz.bounds(*dev(rp, col), 5, alpha=alpha, undirected=und)
            olo, oup = oracle.bounds(rp, col, alpha, 5, undirected=und)
            np.testing.assert_allclose(lo.cpu().numpy(), olo, rtol=1e-12, atol=0)
            np.testing.assert_allclose(up.cpu().numpy(), oup, rtol=1e-12, atol=0)


@pytest.mark.parametrize("table", TABLES[:2])
def test_bin_tables_batch_is_bitwise_single(katz, table):
    katz.tuning_set(bin_bounds=table)
    rng = np.random.default_rng(3)
    graphs, params = [], []
    for i in range(8):
        rp, col = sg.barabasi_albert(int(rng.integers(1000, 30000)), int(rng.integers(3, 20)), 40 + i)
        graphs.append((*dev(rp, col), True))
        params.append(dict(k=int(rng.integers(10, 80)), eps=1e-7, precision="fp32"))
    say("bins batch", table)
    outs = katz.rank_static_batch(graphs, params)
    for (rp_t, col_t, _), pp, res in zip(graphs, params, outs):
        one = katz.rank_static(rp_t, col_t, pp["k"], eps=pp["eps"], precision="fp32")
        assert torch.equal(res.topk, one.topk)
        assert torch.equal(res.lower, one.lower) and torch.equal(res.upper, one.upper)
        assert res.iterations == one.iterations


def test_state_keeps_the_classes_of_its_creation(katz):
    """A state created under one table and updated under another re-walks with
    its own: its results equal katz_bounds on the new graph under the
    creation table, bit for bit."""
    rp, col = sg.rmat(13, seed=9)
    n = len(rp) - 1
    dmax = sg.max_degree(rp)
    alpha = 1.0 / (1 + dmax + 50)
    table = TABLES[1]
    katz.tuning_set(bin_bounds=table)
    say("bins state create")
    st, _ = katz.create_state(*dev(rp, col), 30, alpha=alpha, eps=1e-9, degree_cap=dmax + 50)
    dyn = oracle.DynamicOracle(rp, col, alpha, k=30, eps=1e-9, degree_cap=dmax + 50)
    katz.tuning_set()                                   # default classes from here on
    rng = np.random.default_rng(1)
    for b in range(3):
        src = np.repeat(np.arange(n), np.diff(dyn.row_ptr))
        und = np.stack([src, dyn.col], 1)
        und = und[und[:, 0] < und[:, 1]]
        dels = und[rng.choice(len(und), 20, replace=False)]
        present = set(map(tuple, und.tolist()))
        ins = set()
        while len(ins) < 40:
            a, c = sorted(int(v) for v in rng.integers(0, n, 2))
            if a != c and (a, c) not in present:
                ins.add((a, c))
        ins = np.array(sorted(ins))
        say("bins state batch", b)
        res = st.update(ins, dels)
        orc = dyn.update(ins, dels)
        assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                           gpu_status=res.status)
        katz.tuning_set(bin_bounds=table)
        lo, up = katz.bounds(*dev(dyn.row_ptr, dyn.col), res.iterations, alpha=alpha)
        katz.tuning_set()
        ids = res.topk.long()
        assert torch.equal(lo[ids], res.lower) and torch.equal(up[ids], res.upper)
    st.free()


def test_autotune_chooses_among_the_tables(katz):
    rp, col = sg.rmat(14, seed=2)
    say("bins autotune")
    t = katz.autotune(*dev(rp, col), 50, eps=1e-6, precision="fp32")
    assert t["bin_bounds"] in [[0] * 6] + TABLES[:3]
    assert katz.tuning_get() == t
    orc = oracle.rank_static(rp, col, None, 50, 1e-6)
    res = katz.rank_static(*dev(rp, col), 50, eps=1e-6, precision="fp32")
    assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc, widened=True,
                       gpu_status=res.status)


def test_state_creation_checks_symmetry_loops_and_repeats(katz):
    """States check their graph strictly: an asymmetric graph (against its
    device transpose), a self-loop and a repeated neighbour are E_CSR."""
    say("state strict checks")
    asym = sg.from_edges(6, [0, 1, 2], [1, 2, 3], undirected=False)
    rp, col = sg.cycle_graph(6)
    loop_rp = rp.copy()
    loop_rp[1:] += 1
    loop_col = np.insert(col, 0, 0)                     # 0 -> 0 before row 0's arcs
    dup_col = col.copy()
    dup_col[1] = dup_col[0]                             # row 0 lists a neighbour twice
    for g in (asym, (loop_rp, loop_col), (rp, dup_col)):
        with pytest.raises(katz.KatzError) as e:
            katz.create_state(*dev(*g), 2, alpha=0.2)
        assert e.value.code == katz.E_CSR
    st, res = katz.create_state(*dev(rp, col), 2, alpha=0.2)
    assert res.status in (katz.OK, katz.W_EXACT_TIES, katz.W_ITER_LIMIT)
    st.free()


def test_autotune_cache(katz, tmp_path):
    """With a cache file set, the first autotune of a workload times the
    candidates and appends one line; a second call installs the stored setting
    without timing (the file is unchanged); another workload misses; a line
    holding an invalid setting is ignored."""
    path = tmp_path / "tune.txt"
    katz.autotune_cache(path)
    try:
        rp, col = sg.rmat(12, seed=4)
        say("autotune cache miss")
        t1 = katz.autotune(*dev(rp, col), 20, eps=1e-6, precision="fp32")
        lines = path.read_text().splitlines()
        assert len(lines) == 1 and lines[0].count("\t") == 1
        katz.tuning_set()
        say("autotune cache hit")
        t2 = katz.autotune(*dev(rp, col), 20, eps=1e-6, precision="fp32")
        assert t2 == t1 and katz.tuning_get() == t1
        assert path.read_text().splitlines() == lines
        rp2, col2 = sg.rmat(11, seed=4)
        katz.autotune(*dev(rp2, col2), 20, eps=1e-6, precision="fp32")
        assert len(path.read_text().splitlines()) == 2
        key = lines[0].split("\t")[0]
        path.write_text(key + "\t1 2 3\n" + key + "\t0 0 0 0 0 7 0 0 0 0 0 0 0\n")
        katz.autotune(*dev(rp, col), 20, eps=1e-6, precision="fp32")
        assert len(path.read_text().splitlines()) == 3          # both lines skipped: tuned again
    finally:
        katz.autotune_cache(None)


@pytest.mark.parametrize("undirected", [True, False])
def test_state_strict_checks_across_runs_of_empty_rows(katz, undirected):
    """Arcs only on every 40th node, so a 4096-arc chunk of the strict row check
    crosses more than 2048 rows (runs of empty rows) and follows them forward:
    the graph is accepted and the state ranks as the oracle does; a self-loop
    or a repeated neighbour in it is E_CSR (a directed graph has no symmetry
    check to catch them first)."""
    n = 40 * 3000
    act = np.arange(0, n, 40)
    m = len(act)
    src, dst = [], []
    for i in range(m):
        for d in (1, 2, 3) + ((7,) if i % 5 == 0 else ()):
            src.append(int(act[i]))
            dst.append(int(act[(i + d) % m]))
    rp, col = sg.from_edges(n, src, dst, undirected=undirected)
    rp, col = np.asarray(rp, np.int64), np.asarray(col, np.int32)
    assert int(rp[-1]) > 4096
    alpha = 1.0 / (2 + sg.max_degree(rp))
    say("strict checks empty-row runs", undirected)
    st, res = katz.create_state(*dev(rp, col), 16, alpha=alpha, eps=1e-9, undirected=undirected, max_iter=200)
    orc = oracle.rank_static(rp, col, alpha, 16, 1e-9, undirected=undirected, max_iter=200)
    assert_topk_parity(res.topk.cpu().numpy(), res.lower.cpu().numpy(), res.upper.cpu().numpy(), orc,
                       gpu_status=res.status)
    st.free()
    row = int(act[m // 2])
    j = int(rp[row]) + 1
    loop = col.copy()
    loop[j] = row
    dup = col.copy()
    dup[j] = dup[j - 1]
    for bad in (loop, dup):
        with pytest.raises(katz.KatzError) as e:
            katz.create_state(*dev(rp, bad), 16, alpha=alpha, undirected=undirected)
        assert e.value.code == katz.E_CSR


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2049, 13000])
@pytest.mark.parametrize("table", [None, [1, 2, 3, 5, 9, 17]])
@pytest.mark.parametrize("rp64", [True, False])
def test_binning_block_edges(katz, n, table, rp64):
    """Rows around the 1024-row share of a binning workgroup, in every length
    class: hubs of several segments (n = 13000: in different workgroups), equal
    lengths, empty rows.  Bounds equal the oracle's, and the renumbered run is
    bitwise the run in caller order."""
    say("binning edges", n, table, rp64)
    rng = np.random.default_rng(n)
    src, dst = [], []
    for hub in {0, n // 2, n - 1}:                        # up to n - 1 arcs each
        leaves = rng.choice(n, size=(n * 3) // 4, replace=False)
        src.append(np.full(leaves.size, hub))
        dst.append(leaves)
    body = rng.integers(0, n, size=(2, 3 * n))
    keep = (body % 5 != 4).all(axis=0)                    # every fifth node stays near-empty
    rp, col = sg.from_edges(n, np.concatenate(src + [body[0][keep]]), np.concatenate(dst + [body[1][keep]]))
    alpha = 1.0 / (1 + sg.max_degree(rp))
    katz.tuning_set(bin_bounds=table)
    rp_t = torch.from_numpy(np.asarray(rp, dtype=np.int64 if rp64 else np.int32)).cuda()
    col_t = torch.from_numpy(np.asarray(col, dtype=np.int32)).cuda()
    for precision in ("fp64", "fp32"):
        lo, up = katz.bounds(rp_t, col_t, 4, alpha=alpha, precision=precision)
        lo2, up2 = katz.bounds(rp_t, col_t, 4, alpha=alpha, precision=precision, flags=katz.FLAG_NO_REORDER)
        assert torch.equal(lo, lo2) and torch.equal(up, up2)
        if precision == "fp64":
            olo, oup = oracle.bounds(rp, col, alpha, 4)
            np.testing.assert_allclose(lo.cpu().numpy(), olo, rtol=1e-12, atol=0)
            np.testing.assert_allclose(up.cpu().numpy(), oup, rtol=1e-12, atol=0)


def test_autotune_keeps_the_shape_of_one_workgroup_per_item(katz, tmp_path):
    """One workgroup per work item, which unset launch fields mean on small graphs
    only: the autotuner names it (walk_groups = 1), a stored entry that leaves the
    fields unset installs it, and on a graph whose walk vector outgrows an L2 it gives
    the bits of the library's own choice."""
    path = tmp_path / "tune.txt"
    katz.autotune_cache(path)
    try:
        rp, col = sg.rmat(11, seed=6)
        say("autotune shapes")
        best = katz.autotune(*dev(rp, col), 20, eps=1e-6, precision="fp32")
        assert any(best[f] for f in ("hub_bytes", "blocks_per_cu", "walk_groups", "split_hot_bytes"))
        key = path.read_text().split("\t")[0]
        path.write_text(key + "\t0 0 4 2 0 0 0 0 0 0 0 0 0\n")
        hit = katz.autotune(*dev(rp, col), 20, eps=1e-6, precision="fp32")
        assert hit == katz.tuning_get()
        assert (hit["hub_bytes"], hit["blocks_per_cu"], hit["walk_groups"]) == (0, 0, 1)
        assert (hit["batch_blocks_per_cu"], hit["batch_tile"]) == (4, 2)
    finally:
        katz.autotune_cache(None)
    rp_t, col_t = sg.rmat_device(20, 8, seed=3)
    say("shapes above an L2")
    katz.tuning_set()
    a = katz.rank_static(rp_t, col_t, 100, eps=1e-6)
    katz.tuning_set(walk_groups=1)
    b = katz.rank_static(rp_t, col_t, 100, eps=1e-6)
    assert torch.equal(a.topk, b.topk) and torch.equal(a.lower, b.lower) and torch.equal(a.upper, b.upper)
    assert (a.iterations, a.status, a.rest_upper_max) == (b.iterations, b.status, b.rest_upper_max)
