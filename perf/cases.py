"""The calls that a user of this library times: certified Katz rankings through
the public binding (``paper_1807_03847_amd.katz``), from graphs of a few hundred
nodes, where a call is launches and latency, to a billion arcs, where it is
memory traffic.

A case is a dict: ``call`` names the entry point, the other keys are its sizes
and options.  Graphs are drawn on the GPU from the seed:

* ``er``   Erdos-Renyi, ``ef`` * n edge draws (flat degrees),
* ``rmat`` R-MAT (.57, .19, .19, .05), ``ef`` * n edge draws, labels permuted
           (skewed degrees; the stand-in for social and web graphs),
* ``ba``   Barabasi-Albert, ``m`` targets per node (the batched workload).

Undirected graphs hold both arcs of every edge; rows are sorted, without
repeats or loops.  ``tuned`` cases run with the launch shape and row-length
classes that ``katz.autotune`` finds for graphs of this kind (installed from a
stored result, as a long-lived program does); the others with the defaults, as
a program that only calls the ranking does.
"""
import math

import torch

from paper_1807_03847_amd import katz

# katz.autotune's answer on R-MAT graphs of 2^22 nodes and up.
TUNED = dict(hub_bytes=159744, blocks_per_cu=1, walk_groups=4, bin_bounds=(4, 8, 16, 64, 256, 2048))


def listed():
    return [
        # A program that may not allocate ranks a tiny graph: all latency.
        dict(name="noalloc_er2k_fp64", call="noalloc", graph="er", n=2000, ef=8, k=10, eps=0.0, precision="fp64"),
        # The plain method's workload: exact top-100 (plain separation, eps = 0).
        dict(name="static_er16k_fp64", call="static", graph="er", n=16384, ef=8, k=100, eps=0.0, precision="fp64",
             tuned=False),
        # An ordinary social graph of no round size.
        dict(name="static_rmat150k_fp32", call="static", graph="rmat", n=150001, ef=12, k=50, eps=1e-6,
             precision="fp32", tuned=False),
        # R-MAT 22, top-1000: the call as it comes, and the FP64 form with the autotuned launch shape.
        dict(name="static_rmat22_fp32", call="static", graph="rmat", n=1 << 22, ef=16, k=1000, eps=1e-6,
             precision="fp32", tuned=False),
        dict(name="static_rmat22_fp64_tuned", call="static", graph="rmat", n=1 << 22, ef=16, k=1000, eps=1e-6,
             precision="fp64", tuned=True),
        # The largest: about 1e9 arcs, int64 row offsets, the walk vector far beyond the caches.
        dict(name="static_rmat25_fp32_tuned", call="static", graph="rmat", n=1 << 25, ef=16, k=100, eps=1e-6,
             precision="fp32", tuned=True, rp64=True),
        # Inbound Katz of a directed graph (the call reverses the graph first).
        dict(name="inbound_rmat1m_fp64", call="inbound", graph="rmat", n=1000003, ef=16, k=1000, eps=1e-6,
             precision="fp64"),
        # Every node ranked (k = n): the device-wide sort.
        dict(name="ranking_rmat500k_fp64", call="ranking", graph="rmat", n=500009, ef=16, eps=1e-6,
             precision="fp64"),
        # Many graphs of very different sizes in one call.
        dict(name="batch48_ba_fp32", call="batch", graph="ba", count=48, n_lo=1024, n_hi=131072, eps=1e-6,
             precision="fp32"),
        # Edge updates of a served graph, each batch applied and then undone: a trickle on a graph of half a
        # million nodes, and a bulk change on four million (FP32 state).
        dict(name="update16_rmat500k_fp64", call="update", graph="rmat", n=524288, ef=16, k=100, eps=1e-6,
             precision="fp64", batch=16),
        dict(name="update4000_rmat22_fp32", call="update", graph="rmat", n=1 << 22, ef=16, k=100, eps=1e-6,
             precision="fp32", batch=4000),
        # Katz scores of every node by conjugate gradients.
        dict(name="solve_cg_rmat2m", call="solve", graph="rmat", n=2000003, ef=16, method="cg", tol=1e-12),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(["noalloc", "static", "static", "static", "inbound", "ranking", "batch", "update", "update",
                       "solve"])
    precision = rng.choice(["fp64", "fp32"])
    if call == "batch":
        n_lo = size(300, 4000)
        return dict(call=call, graph="ba", count=size(3, 64), n_lo=n_lo, n_hi=n_lo * size(2, 40), eps=1e-6,
                    precision=precision)
    n = {"noalloc": lambda: size(300, 20000), "static": lambda: size(3000, 1 << 24),
         "inbound": lambda: size(5000, 1 << 21), "ranking": lambda: size(2000, 1 << 20),
         "update": lambda: size(20000, 1 << 22), "solve": lambda: size(5000, 1 << 21)}[call]()
    case = dict(call=call, graph="er" if call == "noalloc" or rng.random() < 0.2 and n < 200000 else "rmat", n=n,
                ef=rng.randint(4, 16))
    if call == "solve":
        return dict(case, method=rng.choice(["cg", "foster"]), tol=rng.choice([1e-9, 1e-12]))
    case.update(precision=precision, eps=1e-6)
    if call != "ranking":
        case["k"] = min(size(5, 2000), n // 20)
    if call == "static":
        case["tuned"] = n > 1000000 and rng.random() < 0.5
        case["rp64"] = rng.random() < 0.3
    if call == "update":
        case["batch"] = min(size(1, 10000), n // 10)
    return case


# ---------------------------------------------------------------------------
# Graphs, drawn on the GPU.
# ---------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rmat_pairs(n, count, perm, g):
    """``count`` endpoint pairs of the R-MAT recursion over the smallest power of
    two that holds n, labels permuted; pairs with an end at or past n are dropped."""
    bits = max(1, (n - 1).bit_length())
    us, vs = [], []
    for first in range(0, count, 1 << 26):
        m = min(1 << 26, count - first)
        u = torch.zeros(m, dtype=torch.int32, device="cuda")
        v = torch.zeros(m, dtype=torch.int32, device="cuda")
        for _ in range(bits):
            q = torch.rand(m, device="cuda", generator=g)
            down = q >= 0.76
            u.mul_(2).add_(down)
            v.mul_(2).add_(torch.where(down, q >= 0.95, q >= 0.57))
        u, v = perm[u.long()], perm[v.long()]
        keep = (u < n) & (v < n)
        us.append(u[keep])
        vs.append(v[keep])
    return torch.cat(us), torch.cat(vs)


def _csr(n, u, v, undirected, rp64):
    """Sorted rows without repeats or loops from endpoint pairs."""
    key = torch.cat([u.long() * n + v, v.long() * n + u]) if undirected else u.long() * n + v
    loops = torch.cat([u == v, u == v]) if undirected else u == v
    key = key[~loops]
    del u, v, loops
    key = torch.sort(key).values
    fresh = torch.ones_like(key, dtype=torch.bool)
    fresh[1:] = key[1:] != key[:-1]
    key = key[fresh]
    row_ptr = torch.searchsorted(key, torch.arange(n + 1, dtype=torch.int64, device="cuda") * n)
    col = (key % n).to(torch.int32)
    return (row_ptr if rp64 else row_ptr.to(torch.int32)), col


def _graph(case, g):
    """(row_ptr, col, label permutation or None)."""
    n, count = case["n"], case["ef"] * case["n"]
    undirected = case["call"] != "inbound"
    if case["graph"] == "er":
        u = torch.randint(0, n, (count,), device="cuda", generator=g)
        v = torch.randint(0, n, (count,), device="cuda", generator=g)
        return _csr(n, u, v, undirected, case.get("rp64", False)) + (None,)
    full = 1 << max(1, (n - 1).bit_length())
    perm = torch.randperm(full, device="cuda", generator=g).to(torch.int32)
    u, v = _rmat_pairs(n, count, perm, g)
    return _csr(n, u, v, undirected, case.get("rp64", False)) + (perm,)


def _ba_graph(n, m, g):
    """Preferential attachment by the endpoint list: edge e = (e // m, the endpoint
    at a uniform earlier position of the list); odd positions are targets, which
    are followed to the edge that holds them until a source is reached."""
    e = torch.arange(n * m, dtype=torch.int64, device="cuda")
    pos = (torch.rand(n * m, device="cuda", generator=g, dtype=torch.float64) * (2 * e + 1).double()).long()
    while True:
        odd = (pos & 1) == 1
        if not bool(odd.any()):
            break
        pos = torch.where(odd, pos[pos >> 1], pos)
    return _csr(n, e // m, (pos >> 1) // m, True, False)


def _batch_sizes(case):
    """(nodes, targets per node, f, k) of each graph of a batch: nodes spread over
    the logarithm of the range, alpha = f / (1 + deg_max)."""
    out, count = [], case["count"]
    for i in range(count):
        t = ((i * 37) % count + 0.5) / count
        n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** t))
        out.append((n, 4 + (i * 11) % 29, 10.0 ** (-3.0 * ((i * 17) % count) / count), 10 + (i * 53) % 200))
    return out


def _edges(case, row_ptr, col, perm, g):
    """A batch of edge updates of the graph: 70% insertions of absent pairs from
    its own distribution, 30% deletions of its edges (numpy arrays)."""
    n, want = case["n"], case["batch"]
    rp = row_ptr.long()
    n_ins = max(1, (want * 7) // 10)
    if case["graph"] == "rmat":
        u, v = _rmat_pairs(n, 8 * n_ins + 64, perm, g)
    else:
        u = torch.randint(0, n, (4 * n_ins + 64,), device="cuda", generator=g)
        v = torch.randint(0, n, (4 * n_ins + 64,), device="cuda", generator=g)
    lo, hi = torch.minimum(u, v).long(), torch.maximum(u, v).long()
    key = torch.unique((lo * n + hi)[lo != hi])
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), rp[1:] - rp[:-1])
    have = src * n + col
    at = torch.searchsorted(have, key).clamp(max=max(have.numel() - 1, 0))
    key = key[have[at] != key]
    key = key[torch.randperm(key.numel(), device="cuda", generator=g)[:n_ins]]
    ins = torch.stack([key // n, key % n], 1).to(torch.int32).cpu().numpy()
    arcs = torch.randint(0, col.numel(), (want - n_ins,), device="cuda", generator=g)
    a, b = src[arcs], col[arcs].long()
    gone = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    dels = torch.stack([gone // n, gone % n], 1).to(torch.int32).cpu().numpy()
    return ins, dels


def _update_inputs(case, seed):
    g = _generator(seed)
    row_ptr, col, perm = _graph(case, g)
    ins, dels = _edges(case, row_ptr, col, perm, g)
    dmax = int((row_ptr[1:] - row_ptr[:-1]).max())
    cap = dmax + dmax // 8 + 2 * case["batch"] + 16   # room for the insertions (Theorem 1: alpha * deg_max < 1)
    return row_ptr, col, ins, dels, cap


def prepare(case, seed):
    katz.tuning_set(**(TUNED if case.get("tuned") else {}))
    call = case["call"]
    if call == "batch":
        g = _generator(seed)
        graphs, params = [], []
        for n, m, f, k in _batch_sizes(case):
            row_ptr, col = _ba_graph(n, m, g)
            dmax = int((row_ptr[1:] - row_ptr[:-1]).max())
            graphs.append((row_ptr, col, True))
            params.append(dict(k=min(k, n), alpha=f / (1.0 + dmax), eps=case["eps"] * f, precision=case["precision"]))
        return dict(case=case, graphs=graphs, params=params)
    if call == "update":
        row_ptr, col, ins, dels, cap = _update_inputs(case, seed)
        state, _ = katz.create_state(row_ptr, col, case["k"], alpha=1.0 / (1.0 + cap), eps=case["eps"],
                                     degree_cap=cap, precision=case["precision"])
        # A served state has seen updates: its level count has reached what these batches need.
        state.update(ins, dels)
        state.update(dels, ins)
        return dict(case=case, state=state, ins=ins, dels=dels)
    row_ptr, col, _ = _graph(case, _generator(seed))
    out = None
    if call == "noalloc":
        out = (torch.empty(case["k"], dtype=torch.int32, device="cuda"),
               torch.empty(case["k"], dtype=torch.float64, device="cuda"),
               torch.empty(case["k"], dtype=torch.float64, device="cuda"))
    return dict(case=case, row_ptr=row_ptr, col=col, out=out)


def _answer(r):
    return dict(ids=r.topk, lower=r.lower, upper=r.upper, iterations=r.iterations, status=r.status)


def run(state):
    case = state["case"]
    call = case["call"]
    if call == "batch":
        res = katz.rank_static_batch(state["graphs"], state["params"])
        return dict(ids=torch.cat([r.topk for r in res]), lower=torch.cat([r.lower for r in res]),
                    upper=torch.cat([r.upper for r in res]),
                    iterations=torch.tensor([r.iterations for r in res]),
                    status=torch.tensor([r.status for r in res]))
    if call == "update":
        there = state["state"].update(state["ins"], state["dels"])
        back = state["state"].update(state["dels"], state["ins"])
        return dict(there=_answer(there), back=_answer(back))
    rp, col = state["row_ptr"], state["col"]
    if call == "solve":
        scores, info, status = katz.solve(rp, col, case["method"], case["tol"])
        return dict(scores=scores, iterations=info["iterations"], status=status)
    if call == "noalloc":
        r = katz.rank_static_noalloc(rp, col, case["k"], eps=case["eps"], precision=case["precision"],
                                     out=state["out"])
    elif call == "inbound":
        r = katz.rank_static(rp, col, case["k"], eps=case["eps"], precision=case["precision"], undirected=False,
                             flags=katz.FLAG_INBOUND)
    elif call == "ranking":
        r = katz.rank_static(rp, col, case["n"], eps=case["eps"], precision=case["precision"], criterion="ranking")
    else:
        r = katz.rank_static(rp, col, case["k"], eps=case["eps"], precision=case["precision"])
    return _answer(r)


def work(case):
    """The graph read once and the results written once; an addition per arc and
    walk step, over the five steps that a ranking takes at the least."""
    call = case["call"]
    if call == "batch":
        sizes = _batch_sizes(case)
        arcs = sum(2 * n * m for n, m, _, _ in sizes)
        return {"bytes": 4 * arcs + 4 * sum(n for n, _, _, _ in sizes) + 20 * sum(k for _, _, _, k in sizes),
                "flops": 5 * arcs}
    n = case["n"]
    arcs = case["ef"] * n * (1 if call == "inbound" else 2)
    if call == "update":
        # Two updates: every node's bound is tested again (c, the top walk level, FP32: the margin).
        return {"bytes": 2 * (16 * n + 16 * case["batch"] + 20 * case["k"]), "flops": 2 * 5 * 32 * case["batch"]}
    listing = 8 * n if call == "solve" else 20 * (n if call == "ranking" else case["k"])
    return {"bytes": 4 * arcs + (8 if case.get("rp64") else 4) * n + listing, "flops": 5 * arcs}


# ---------------------------------------------------------------------------
# The same answers in plain 64-bit torch.
# ---------------------------------------------------------------------------
class _Plain:
    """Walk sums of one graph (row offsets and columns): c_r and alpha^r omega_r, level by level."""

    def __init__(self, row_ptr, col, alpha, undirected):
        self.row_ptr, self.col, self.alpha, self.undirected = row_ptr.long(), col, alpha, undirected
        n = row_ptr.numel() - 1
        dmax = int((self.row_ptr[1:] - self.row_ptr[:-1]).max())
        self.gamma = dmax / (1.0 - alpha * dmax)
        self.s = torch.ones(n, dtype=torch.float64, device="cuda")
        self.c = torch.zeros(n, dtype=torch.float64, device="cuda")
        self.n, self.r = n, 0

    def step(self):
        t = torch.empty_like(self.s)
        for first in range(0, self.n, 1 << 21):
            ptr = self.row_ptr[first:first + (1 << 21) + 1]
            x = self.s[self.col[int(ptr[0]):int(ptr[-1])].long()]
            t[first:first + (1 << 21)] = torch.segment_reduce(x, "sum", offsets=ptr - ptr[0], initial=0.0)
        self.s = self.alpha * t
        self.c = self.c + self.s
        self.r += 1

    def bounds(self):
        lower = self.c + self.alpha * self.s if self.undirected else self.c
        return lower, self.c + self.alpha * self.gamma * self.s

    def certify(self, k, eps, r_min=1, r_max=400):
        """Steps until the k first nodes by lower bound are eps-separated from
        each other and from the rest; (lower, upper) of the k nodes in order."""
        while True:
            if self.r < r_min:
                self.step()
                continue
            lower, upper = self.bounds()
            order = torch.sort(lower, descending=True, stable=True).indices
            top = order[:k]
            lo, up = lower[top], upper[top]
            apart = bool((up[1:] - eps < lo[:-1]).all()) and (
                k == self.n or bool((upper[order[k:]] - eps < lo[-1]).all()))
            if apart or self.r >= r_max or not bool(self.s.any()):
                return lo, up
            self.step()


def _sources(row_ptr):
    rp = row_ptr.long()
    return torch.repeat_interleave(torch.arange(rp.numel() - 1, device="cuda"), rp[1:] - rp[:-1])


def _exact_answer(lower, upper):
    return dict(ids=None, lower=lower, upper=upper, iterations=None, status=None)


def exact(case, seed):
    call = case["call"]
    if call == "batch":
        lo, up, g = [], [], _generator(seed)
        for n, m, f, k in _batch_sizes(case):
            row_ptr, col = _ba_graph(n, m, g)
            dmax = int((row_ptr[1:] - row_ptr[:-1]).max())
            a, b = _Plain(row_ptr, col, f / (1.0 + dmax), True).certify(min(k, n), case["eps"] * f)
            lo.append(a)
            up.append(b)
        return _exact_answer(torch.cat(lo), torch.cat(up))
    if call == "update":
        row_ptr, col, ins, dels, cap = _update_inputs(case, seed)
        n, i, d = case["n"], torch.from_numpy(ins).long().cuda(), torch.from_numpy(dels).long().cuda()
        key = _sources(row_ptr) * n + col
        key = key[~torch.isin(key, torch.cat([d[:, 0] * n + d[:, 1], d[:, 1] * n + d[:, 0]]))]
        key = torch.cat([key, i[:, 0] * n + i[:, 1], i[:, 1] * n + i[:, 0]])
        graphs = [(row_ptr, col), _csr(n, key // n, key % n, False, True)]
        answers, r = {}, 1
        # As prepare() and run() do: the graph, then there and back twice; levels reached are kept.
        for which in (0, 1, 0, 1, 0):
            p = _Plain(*graphs[which], 1.0 / (1.0 + cap), True)
            answers[which] = p.certify(case["k"], case["eps"], r)
            r = p.r
        return dict(there=_exact_answer(*answers[1]), back=_exact_answer(*answers[0]))
    row_ptr, col, _ = _graph(case, _generator(seed))
    n = case["n"]
    alpha = 1.0 / (1.0 + int((row_ptr[1:] - row_ptr[:-1]).max()))
    if call == "inbound":
        row_ptr, col = _csr(n, col, _sources(row_ptr), False, True)
        alpha = 1.0 / (1.0 + int((row_ptr[1:] - row_ptr[:-1]).max()))
    plain = _Plain(row_ptr, col, alpha, call != "inbound")
    if call == "solve":
        for _ in range(400):
            plain.step()
            if float(plain.s.max()) < 1e-18:
                break
        return dict(scores=plain.c, iterations=None, status=None)
    return _exact_answer(*plain.certify(n if call == "ranking" else case["k"], case["eps"]))
