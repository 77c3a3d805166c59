"""Performance cases of the exact-reliability library.

Each case is one call (or one training step) that a user's program makes
through the public entry points, on a seeded random network of the sizes the
benchmark, the tests and the README use.  A case names its network by `net`
(a generator seed), so that a run's seed only changes the probabilities: a
program keeps its network and asks for many probability vectors.

  call      kind
  forward   bat_reliability_ex: R and the count, host buffers
  async     bat_reliability_async: device buffers, the current stream
  grad      bat_reliability_grad: R, the count and every dR/dp, T1, T0
  step      torch_fn.reliability and its backward, device tensors
  range     bat_reliability_range: one equal division of the counter
  batched   bat_reliability_batched: graphs x probability vectors
  ms        bat_ms_reliability: arcs with three capacity levels
"""
import functools

import numpy as np
import torch


def listed():
    return [
        # the smallest call: the 5-arc bridge, all latency
        {"name": "forward bridge m5", "kind": "forward", "net": 0, "n": 4, "m": 5, "directed": False},
        # an optimiser's step on a small network: R, then its gradient
        {"name": "step n10 m18", "kind": "step", "net": 11, "n": 10, "m": 18},
        # a digraph of everyday size
        {"name": "forward directed n13 m24", "kind": "forward", "net": 12, "n": 13, "m": 24, "directed": True},
        # the random 30-arc network of the benchmark's second workload
        {"name": "forward n20 m30", "kind": "forward", "net": 13, "n": 20, "m": 30, "directed": False},
        # one of 64 equal divisions of a 36-arc network, as a shard runs it
        {"name": "range n18 m36 1/64", "kind": "range", "net": 14, "n": 18, "m": 36, "parts": 64, "part": 41},
        # the headline workload: 5x5 grid, 2^40 vectors, device buffers
        {"name": "async grid5x5 m40", "kind": "async", "net": -5, "n": 25, "m": 40},
        # all importances of an odd-sized middle network
        {"name": "grad n14 m27", "kind": "grad", "net": 15, "n": 14, "m": 27},
        # all importances of the benchmark's 36-arc workload
        {"name": "grad n18 m36", "kind": "grad", "net": 16, "n": 18, "m": 36},
        # a small untuned batch: few small graphs, few probability vectors
        {"name": "batched 16x3", "kind": "batched", "net": 17, "graphs": 16, "pvec": 3, "n_lo": 5, "n_hi": 12,
         "m_lo": 8, "m_hi": 20, "tuned": False},
        # the benchmark's batch, tuned once as its program does
        {"name": "batched 256x32 tuned", "kind": "batched", "net": 18, "graphs": 256, "pvec": 32, "n_lo": 8,
         "n_hi": 16, "m_lo": 16, "m_hi": 28, "tuned": True},
        # the multi-state workload: flow 2 over 18 three-level arcs
        {"name": "ms n10 m18 demand 2", "kind": "ms", "net": 19, "n": 10, "m": 18, "demand": 2},
        # a demand above the bit-sliced kernel's: augmenting paths
        {"name": "ms n9 m15 demand 4", "kind": "ms", "net": 20, "n": 9, "m": 15, "demand": 4},
    ]


def draw(rng):
    kind = rng.choice(["forward", "forward", "async", "grad", "step", "range", "batched", "ms"])
    net = rng.randrange(1000, 1 << 30)
    if kind in ("forward", "async", "grad", "step", "range"):
        m = rng.randrange(*{"forward": (5, 37), "async": (12, 39), "grad": (6, 35), "step": (8, 27),
                            "range": (18, 37)}[kind])
        n = rng.randrange(max(4, m // 3), min(m, 2 + m * 2 // 3 + 1) + 1)
        while n * (n - 1) // 2 < m:
            n += 1
        c = {"kind": kind, "net": net, "n": n, "m": m}
        if kind == "forward":
            c["directed"] = rng.random() < 0.3
        if kind == "range":
            c["parts"] = rng.choice([8, 64, 48, 100])
            c["part"] = rng.randrange(c["parts"])
        return c
    if kind == "batched":
        m_hi = rng.randrange(14, 27)
        return {"kind": "batched", "net": net, "graphs": int(round(2 ** rng.uniform(1, 7))),
                "pvec": int(round(2 ** rng.uniform(0, 6))), "n_lo": 6, "n_hi": rng.randrange(9, 17), "m_lo": 9,
                "m_hi": m_hi, "tuned": False}
    d = rng.randrange(1, 6)
    m = rng.randrange(7, 18 if d <= 3 else 16)
    n = rng.randrange(max(5, m // 2), min(10, m) + 1)
    while n * (n - 1) // 2 < m:
        n += 1
    return {"kind": "ms", "net": net, "n": n, "m": m, "demand": d}


# ---------------------------------------------------------------- networks

def random_arcs(n, m, rng):
    """A random spanning tree, then distinct further node pairs."""
    perm = rng.permutation(n)
    arcs, have = [], set()
    for i in range(1, n):
        a, b = int(perm[i]), int(perm[int(rng.integers(0, i))])
        arcs.append((min(a, b), max(a, b)))
        have.add(arcs[-1])
    rest = [(i, j) for i in range(n) for j in range(i + 1, n) if (i, j) not in have]
    arcs += [rest[int(k)] for k in rng.choice(len(rest), size=m - (n - 1), replace=False)] if m > n - 1 else []
    return arcs


def grid_arcs(k):
    across = [(k * r + c, k * r + c + 1) for r in range(k) for c in range(k - 1)]
    return across + [(k * r + c, k * r + c + k) for r in range(k - 1) for c in range(k)]


def network(case):
    """(n, arcs, s, t) of a single-network case."""
    n, m, net = case["n"], case["m"], case["net"]
    if net == 0:
        return 4, [(0, 1), (0, 2), (1, 2), (1, 3), (2, 3)], 0, 3
    if net < 0:
        return n, grid_arcs(-net), 0, n - 1
    rng = np.random.default_rng([220909711, net])
    arcs = random_arcs(n, m, rng)
    if case.get("directed"):
        # most arcs along the node order, and one whole path from s to t
        arcs = [(b, a) if rng.random() < 0.3 else (a, b) for a, b in arcs]
        came, todo = {0: None}, [0]
        for x in todo:
            for i, e in enumerate(arcs):
                y = e[0] + e[1] - x
                if x in e and y not in came:
                    came[y] = (x, i)
                    todo.append(y)
        x = n - 1
        while came[x] is not None:
            u, i = came[x]
            arcs[i] = (u, x)
            x = u
    return n, arcs, 0, n - 1


@functools.lru_cache(maxsize=4)
def batch_graphs(net, graphs, n_lo, n_hi, m_lo, m_hi):
    rng = np.random.default_rng([220909711, net])
    out = []
    for _ in range(graphs):
        n, m = int(rng.integers(n_lo, n_hi + 1)), int(rng.integers(m_lo, m_hi + 1))
        m = max(n - 1, min(m, n * (n - 1) // 2))
        arcs = random_arcs(n, m, rng)
        s, t = (int(x) for x in rng.choice(n, size=2, replace=False))
        out.append((n, arcs, s, t))
    return out


def batch_of(case):
    return batch_graphs(*(case[k] for k in ("net", "graphs", "n_lo", "n_hi", "m_lo", "m_hi")))


def probabilities(seed, shape):
    return np.random.default_rng([3, seed]).uniform(0.6, 0.99, size=shape)


def state_weights(seed, m):
    """Three levels per arc: failed, degraded, the rest at full capacity."""
    rng = np.random.default_rng([4, seed])
    w0, w1 = rng.uniform(0.02, 0.10, size=m), rng.uniform(0.10, 0.30, size=m)
    return np.stack([w0, w1, 1.0 - w0 - w1], axis=1)


def division(case):
    """Division `part` of `parts` equal ones (the last takes the remainder)."""
    total, k = 1 << case["m"], case["part"]
    return total * k // case["parts"], total * (k + 1) // case["parts"]


# ------------------------------------------------------------ the measured

_tuned = set()


def prepare(case, seed):
    import paper_2209_09711_amd as B
    kind, st = case["kind"], {"B": B, "kind": case["kind"]}
    if kind == "batched":
        graphs = batch_of(case)
        rng = np.random.default_rng([5, seed])
        st["graphs"] = graphs
        st["p"] = [rng.uniform(0.5, 0.99, size=(case["pvec"], len(g[1]))) for g in graphs]
        if case["tuned"] and case["net"] not in _tuned:
            B.bat_autotune_batched(graphs, st["p"])  # once per batch structure
            _tuned.add(case["net"])
        return st
    n, arcs, s, t = network(case)
    st.update(n=n, arcs=np.asarray(arcs, dtype=np.int32), s=s, t=t)
    if kind == "ms":
        st.update(states=[3] * len(arcs), cap=np.tile(np.arange(3, dtype=np.int32), len(arcs)),
                  w=state_weights(seed, len(arcs)).reshape(-1), demand=case["demand"])
        return st
    st["p"] = probabilities(seed, len(arcs))
    if kind == "forward":
        st["directed"] = case["directed"]
    elif kind == "range":
        st["lo"], st["hi"] = division(case)
    elif kind in ("async", "step"):
        st["p"] = torch.tensor(st["p"], dtype=torch.float64, device="cuda")
        if kind == "step":
            st["p"].requires_grad_(True)
        else:
            st["R"] = torch.zeros((), dtype=torch.float64, device="cuda")
            st["count"] = torch.zeros((), dtype=torch.int64, device="cuda")
    return st


def run(st):
    B, kind = st["B"], st["kind"]
    if kind == "batched":
        R, count = B.bat_reliability_batched(st["graphs"], st["p"])
        return {"R": R, "count": count.astype(np.int64)}
    if kind == "ms":
        R, count = B.bat_ms_reliability(st["n"], st["arcs"], st["states"], st["cap"], st["w"], st["s"], st["t"],
                                        st["demand"])
        return {"R": np.float64(R), "count": count}
    net = (st["n"], st["arcs"], st["p"], st["s"], st["t"])
    if kind == "forward":
        R, count = B.bat_reliability_ex(*net, directed=st["directed"])
        return {"R": np.float64(R), "count": count}
    if kind == "grad":
        g = B.bat_reliability_grad(*net)
        return {"R": np.float64(g.R), "count": g.count, "dRdp": g.dRdp, "T1": g.T1, "T0": g.T0}
    if kind == "range":
        r = B.bat_reliability_range(*net, st["lo"], st["hi"])
        return {"R": np.float64(r.R), "count": r.count}
    if kind == "step":
        from paper_2209_09711_amd.torch_fn import reliability
        R, count = reliability(st["p"], st["n"], st["arcs"], st["s"], st["t"])
        (grad,) = torch.autograd.grad(R, st["p"])
        return {"R": R, "count": count, "dRdp": grad}
    B.bat_reliability_async(st["n"], st["arcs"], st["p"].data_ptr(), st["s"], st["t"], st["R"].data_ptr(),
                            st["count"].data_ptr(), None, torch.cuda.current_stream().cuda_stream)
    return {"R": st["R"], "count": st["count"]}


def work(case):
    """Bytes: the probabilities in, the results out.  Operations: one
    connectivity verdict and one addition per state vector (and probability
    vector), which is what the method is about, however they are decided."""
    if case["kind"] == "batched":
        ms = [len(g[1]) for g in batch_of(case)]
        return {"bytes": 8 * case["pvec"] * (sum(ms) + len(ms)) + 8 * len(ms),
                "flops": float(sum(1 << m for m in ms)) * (1 + case["pvec"])}
    m = case["m"]
    if case["kind"] == "ms":
        return {"bytes": 36 * m + 16, "flops": 2.0 * 3.0 ** m}
    if case["kind"] == "range":
        lo, hi = division(case)
        return {"bytes": 16 * m + 16, "flops": 2.0 * (hi - lo)}
    adds = 1 + (m if case["kind"] in ("grad", "step") else 0)
    return {"bytes": 16 * m + 16 + (24 * m if adds > 1 else 0), "flops": float(1 << m) * (1 + adds)}


# ------------------------------------------------------- values in 64 bits
# A dynamic programme over the arcs: a state is what the arcs so far make of
# the nodes that later arcs still touch (which reach which).  Sums in
# extended precision; a column with every probability 1/2 counts vectors
# exactly.

L = np.longdouble


def programme(n, arcs, s, t, directed):
    """(moves, dead): for each arc in an order that keeps few nodes open, the
    pair (arc, [(state if it fails, state if it works), one per state]),
    where state -1 is a connected end and -2 one that cannot connect; dead:
    no arc touches s or t.  A state is the reach mask of each open node."""
    left, at, seen = set(range(len(arcs))), {}, {s}
    touch = [[i for i, e in enumerate(arcs) if x in e] for x in range(n)]
    order = []
    while left:
        def cost(i):
            a, b = arcs[i]
            opened = (a not in seen) + (b not in seen)
            closes = sum(all(j == i or j not in left for j in touch[x]) for x in (a, b))
            near = sum(min((at[j] for j in touch[x] if j in at), default=len(arcs)) for x in (a, b))
            return opened - closes, near, i
        i = min(left, key=cost)
        at[i] = len(order)
        order.append(i)
        left.discard(i)
        seen.update(arcs[i])
    if not touch[s] or not touch[t]:
        return [], True
    last = [max((at[i] for i in touch[x]), default=-1) for x in range(n)]
    first = [min((at[i] for i in touch[x]), default=-1) for x in range(n)]

    def join(reach, a, b):
        return [r | reach[b] if (r >> a) & 1 else r for r in reach]

    steps, states = [], {tuple(1 << x for x in range(n)): 0}
    for k, i in enumerate(order):
        a, b = arcs[i]
        live = sum(1 << x for x in range(n) if first[x] <= k < last[x] or x in (s, t))
        ahead = sum(1 << x for x in range(n) if last[x] > k)
        nxt, moves = {}, []

        def settle(reach):
            if (reach[s] >> t) & 1:
                return -1
            # an end's open nodes: with none left nothing can connect any more
            if not reach[s] & ahead or not any((reach[x] >> t) & 1 for x in range(n) if (ahead >> x) & 1):
                return -2
            key = tuple(reach[x] & live if (live >> x) & 1 else 1 << x for x in range(n))
            return nxt.setdefault(key, len(nxt))
        for st in states:
            up = st
            if a != b:
                up = join(st, a, b)
                up = up if directed else join(up, b, a)
            moves.append((settle(st), settle(up)))
        steps.append((i, moves))
        states = nxt
    return steps, False


def solve(n, arcs, s, t, p, directed=False, grad=False):
    """R for each row of p (and T1, T0 per arc) in extended precision."""
    p = np.asarray(p, dtype=L)
    P, m = p.shape
    T1, T0 = np.zeros((P, m), L), np.zeros((P, m), L)
    steps, dead = programme(n, arcs, s, t, directed)
    if dead:
        return np.zeros(P, L), T1, T0
    # the value of each state before arc k, then rows for -2 and -1
    ends = np.stack([np.zeros(P, L), np.ones(P, L)])
    rest = [None] * (len(steps) + 1)
    rest[len(steps)] = ends
    move = [np.array(moves, dtype=np.int64).reshape(-1, 2) for _, moves in steps]
    for k in range(len(steps) - 1, -1, -1):
        q = p[:, steps[k][0]]
        rest[k] = np.concatenate([q * rest[k + 1][move[k][:, 1]] + (1 - q) * rest[k + 1][move[k][:, 0]], ends])
    if grad:
        mass = np.ones((1, P), L)
        ended = np.zeros(P, L)  # mass that connected before this arc
        for k, (i, _) in enumerate(steps):
            f, w, nxt = move[k][:, 0], move[k][:, 1], np.zeros_like(rest[k + 1])
            T1[:, i] = ended + (mass * rest[k + 1][w]).sum(axis=0)
            T0[:, i] = ended + (mass * rest[k + 1][f]).sum(axis=0)
            np.add.at(nxt, w, mass * p[:, i])
            np.add.at(nxt, f, mass * (1 - p[:, i]))
            ended = ended + nxt[-1]
            mass = nxt[:-2]
    return rest[0][0], T1, T0


def with_half(p):
    p = np.atleast_2d(p)
    return np.concatenate([p, np.full((1, p.shape[1]), 0.5)])


def exact_range(n, arcs, s, t, p, lo, hi):
    """[lo, hi) as whole sub-cubes of the counter: in each, the leading arcs
    are fixed."""
    m, R, count = len(arcs), L(0), 0
    while lo < hi:
        k = min((lo & -lo).bit_length() - 1 if lo else m, (hi - lo).bit_length() - 1)
        fixed = [(lo >> (m - 1 - i)) & 1 for i in range(m - k)]
        q = with_half(p).astype(L)
        scale = np.ones(2, L)
        for i, x in enumerate(fixed):
            scale *= q[:, i] if x else 1 - q[:, i]
            q[:, i] = x
        r = solve(n, arcs, s, t, q)[0] * scale
        R += r[0]
        count += int(r[1] * L(2) ** m)
        lo += 1 << k
    return R, count


def exact_ms(n, arcs, s, t, w, demand):
    """Max-flow min-cut over every cut, the arcs in two halves: each half's
    state vectors are merged by their (clipped) capacities across the cuts."""
    others = [x for x in range(n) if x not in (s, t)]
    sides = [{s} | {x for k, x in enumerate(others) if (c >> k) & 1} for c in range(1 << len(others))]

    def half(ids):
        caps = np.zeros((1, len(sides)), np.uint8)
        weight, number = np.ones(1, L), np.ones(1, np.int64)
        for i in ids:
            across = np.array([(arcs[i][0] in c) != (arcs[i][1] in c) for c in sides], np.uint8)
            rows = np.concatenate([np.minimum(caps + k * across, demand).astype(np.uint8) for k in range(3)])
            wk, nk = np.concatenate([weight * L(w[i][k]) for k in range(3)]), np.concatenate([number] * 3)
            keys, at = np.unique(rows.view([("", rows.dtype)] * rows.shape[1]).ravel(), return_inverse=True)
            caps = keys.view(np.uint8).reshape(len(keys), -1)
            weight, number = np.zeros(len(keys), L), np.zeros(len(keys), np.int64)
            np.add.at(weight, at, wk)
            np.add.at(number, at, nk)
        return caps, weight, number
    dist = {s: 0}
    todo = [s]
    for x in todo:
        for a, b in arcs:
            for u, v in ((a, b), (b, a)):
                if u == x and v not in dist:
                    dist[v] = dist[x] + 1
                    todo.append(v)
    ids = sorted(range(len(arcs)), key=lambda i: (dist.get(arcs[i][0], n) + dist.get(arcs[i][1], n), i))
    A, B = half(ids[:len(ids) // 2]), half(ids[len(ids) // 2:])
    if len(A[1]) * len(B[1]) * len(sides) > 3e10:
        return None
    R, count = L(0), 0
    for row, wa, na in zip(*A):
        ok = ((B[0] + row) >= demand).all(axis=1)
        R += wa * B[1][ok].sum()
        count += int(na) * int(B[2][ok].sum())
    return R, count


def exact(case, seed):
    kind = case["kind"]
    if kind == "batched":
        graphs = batch_of(case)
        rng = np.random.default_rng([5, seed])
        R, count = [], []
        for n, arcs, s, t in graphs:
            r = solve(n, arcs, s, t, with_half(rng.uniform(0.5, 0.99, size=(case["pvec"], len(arcs)))))[0]
            R.append(r[:-1].astype(np.float64))
            count.append(int(r[-1] * L(2) ** len(arcs)))
        return {"R": np.array(R), "count": np.array(count, np.int64)}
    n, arcs, s, t = network(case)
    if kind == "ms":
        got = exact_ms(n, arcs, s, t, state_weights(seed, len(arcs)), case["demand"])
        return None if got is None else {"R": np.float64(got[0]), "count": got[1]}
    p = probabilities(seed, len(arcs))
    if kind == "range":
        R, count = exact_range(n, arcs, s, t, p, *division(case))
        return {"R": np.float64(R), "count": count}
    want_grad = kind in ("grad", "step")
    R, T1, T0 = solve(n, arcs, s, t, with_half(p), case.get("directed", False), want_grad)
    out = {"R": np.float64(R[0]), "count": int(R[1] * L(2) ** len(arcs))}
    if want_grad:
        out["dRdp"] = (T1[0] - T0[0]).astype(np.float64)
        if kind == "grad":
            out.update(T1=T1[0].astype(np.float64), T0=T0[0].astype(np.float64))
    return out
