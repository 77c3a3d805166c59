"""Sub-cube sweeps at the edges of their launches: batches whose launches
follow each other at once on a busy device, spaces of many work items,
checkpoints and reports under other settings than they began with."""
import numpy as np
import pytest

import bat_workloads as W
import oracle

pytestmark = pytest.mark.gpu

# sums of terms of one sign by plain additions, at most some 2^9 in a chain
# between the compensated ones: 2^9 roundings of 1.1e-16 at worst
REL_SUMS = 6e-14


def _B():
    import paper_2209_09711_amd as B
    return B


@pytest.mark.parametrize("n_graphs,n_pvec", [(3, 1024), (2, 1023), (40, 100)])
def test_batches_of_many_entries_per_graph(n_graphs, n_pvec):
    """More than 64 entries, several to a graph, so that the second launch
    follows the first without planning in between; with other work of the
    process in front of them."""
    import torch
    B = _B()
    rng = np.random.default_rng(2400 + n_pvec)
    nets = [W.random_connected(8 + k % 3, 14 + k % 5, seed=500 + k) for k in range(n_graphs)]
    p = [rng.uniform(0.2, 0.99, (n_pvec, x.m)) for x in nets]
    a = torch.ones(4096, 4096, device="cuda")
    for _ in range(8):
        a = (a @ a).clamp_(0.0, 1.0)
    print("cube batch", n_graphs, n_pvec, flush=True)
    R, cnt = B.bat_reliability_batched([(x.n, x.arcs, x.s, x.t) for x in nets], p)
    assert B.bat_last_launch().perm == 5
    torch.cuda.synchronize()
    for g in range(n_graphs):
        for j in (0, 31, 32, n_pvec // 2, n_pvec - 1) if n_graphs < 10 else (g % n_pvec,):
            o = oracle.reliability(nets[g].n, nets[g].arcs, p[g][j], nets[g].s, nets[g].t)
            assert cnt[g] == o.count and abs(R[g, j] - o.sum) <= REL_SUMS * o.sum, (g, j)


def _ms(B, net, demand, seed=0):
    """A three-level network's arguments."""
    w = np.random.default_rng(seed).uniform(0.1, 1.0, (net.m, 3))
    w /= w.sum(axis=1, keepdims=True)
    return net.n, net.arcs, [3] * net.m, [0, 1, 2] * net.m, list(w.ravel()), net.s, net.t, demand


@pytest.mark.parametrize("m,demand", [(21, 1), (22, 2), (21, 3)])
def test_multi_state_spaces_of_many_items(m, demand):
    """More work items than wavefronts, against the sweep of every word."""
    B = _B()
    args = _ms(B, W.random_connected(12, m, seed=m), demand)
    print("multi-state cubes", m, demand, flush=True)
    R, cnt = B.bat_ms_reliability(*args)
    li = B.bat_last_launch()
    assert li.perm == 5 and li.n_chunks > 65536
    old = B.bat_get_option("BAT_CUBES")
    try:
        B.bat_set_option("BAT_CUBES", 0)
        want, wcnt = B.bat_ms_reliability(*args)
    finally:
        B.bat_set_option("BAT_CUBES", old)
    assert cnt == wcnt and abs(R - want) <= REL_SUMS * want


@pytest.mark.parametrize("states,m,demand", [(3, 15, 4), (2, 23, 2), (5, 10, 7)])
def test_multi_state_flow_in_several_launches(states, m, demand):
    """More cubes than one launch of the flow kernel takes (of one vector
    each): the whole space, and a range with ends inside two launches."""
    B = _B()
    net = W.random_connected(9, m, seed=m + demand)
    w = np.random.default_rng(m).uniform(0.1, 1.0, (m, states))
    w /= w.sum(axis=1, keepdims=True)
    args = (net.n, net.arcs, [states] * m, list(range(states)) * m, list(w.ravel()), net.s, net.t, demand)
    N = states ** m
    lo, hi = N // 10 + 3, N - N // 7
    print("multi-state flow", states, m, demand, flush=True)
    got = {}
    old = {k: B.bat_get_option(k) for k in ("BAT_MS_RUN", "BAT_MS_BITS")}
    try:
        B.bat_set_option("BAT_MS_BITS", 0)
        for run in (0, 1):
            B.bat_set_option("BAT_MS_RUN", run)
            got[run] = [B.bat_ms_reliability(*args)]
            li = B.bat_last_launch()
            assert li.vectors == N and 0.0 < li.kernel_ms <= li.total_ms and (run == 0 or li.n_chunks > 65536)
            r = B.bat_ms_reliability_range(*args, lo, hi)
            got[run].append((r.R, r.count))
    finally:
        for k, v in old.items():
            B.bat_set_option(k, v)
    for (R, cnt), (want, wcnt) in zip(got[1], got[0]):
        assert cnt == wcnt and abs(R - want) <= REL_SUMS * want


def test_sweep_of_chunked_units():
    """2^24 work items and more: units in chunks; whole and in parts."""
    from oracle import frontier_dp
    B = _B()
    net = W.random_connected(24, 46, seed=1, p_lo=0.6, p_hi=0.99)
    Rd, cd = frontier_dp.reliability(net.n, net.arcs, net.p, net.s, net.t)
    args = (net.n, net.arcs, net.p, net.s, net.t)
    print("chunked", net.name, flush=True)
    R, cnt = B.bat_reliability(*args)
    li = B.bat_last_launch()
    assert li.perm == 5 and li.specialised == 1 and li.n_chunks == 1 << 24
    assert cnt == cd and abs(R - Rd) <= REL_SUMS * Rd
    R, cnt = B.bat_reliability_checkpointed(*args, net.m - 2, None)
    assert cnt == cd and abs(R - Rd) <= REL_SUMS * Rd


def _exact_gradient(net):
    """T1, T0 in extended precision, every vector by itself."""
    m, L = net.m, np.longdouble
    x = (np.arange(1 << m)[:, None] >> np.arange(m)) & 1 == 1
    reach = np.zeros((1 << m, net.n), bool)
    reach[:, net.s] = True
    for _ in range(net.n):
        for i, (a, b) in enumerate(net.arcs):
            both = (reach[:, a] | reach[:, b]) & x[:, i]
            reach[:, a] |= both
            reach[:, b] |= both
    up = np.asarray(net.p, L)
    q = np.where(x, up, 1 - up)
    T1, T0 = np.zeros(m, L), np.zeros(m, L)
    for i in range(m):
        w = np.prod(np.delete(q, i, axis=1), axis=1) * reach[:, net.t]
        T1[i], T0[i] = w[x[:, i]].sum(), w[~x[:, i]].sum()
    return T1, T0


def test_gradients_as_accurate_as_the_plain_sweep():
    """Root mean square errors of T1, T0 and dR/dp over 32 networks of 12 arcs,
    where the fold of a wavefront's columns weighs most: no more than those of
    the plain sweep, which folds in double-double (the two scatter by some 5%
    over samples of 380 values; a plain fold gave three times the error of
    dR/dp)."""
    B = _B()
    err = {0: [], -1: []}
    old = B.bat_get_option("BAT_CUBES")
    try:
        for k in range(32):
            net = W.random_connected(8, 12, seed=900 + k, p_lo=0.6, p_hi=0.99)
            T1, T0 = _exact_gradient(net)
            for v in err:
                B.bat_set_option("BAT_CUBES", v)
                g = B.bat_reliability_grad(net.n, net.arcs, net.p, net.s, net.t)
                assert (B.bat_last_launch().perm == 5) == (v != 0)
                err[v].append([np.abs(a - e) / T1 for a, e in ((g.T1, T1), (g.T0, T0), (g.dRdp, T1 - T0))])
    finally:
        B.bat_set_option("BAT_CUBES", old)
    rms = {v: np.sqrt((np.array(e, float) ** 2).mean(axis=(0, 2))) for v, e in err.items()}
    print("rms errors of T1, T0, dR/dp: plain", rms[0], "cubes", rms[-1], flush=True)
    assert np.all(rms[-1] <= 1.15 * rms[0])


def test_autotune_reports_the_sweep_that_runs():
    """The tuner's time per vector is that of the launch a whole call takes
    (the plain launch it also tunes is several times slower here)."""
    B = _B()
    net = W.random_connected(16, 33, seed=77, p_lo=0.6, p_hi=0.99)
    print("autotune", net.name, flush=True)
    ns = B.bat_autotune(net.n, net.arcs, net.p, net.s, net.t)
    ks = []
    for _ in range(5):
        B.bat_reliability(net.n, net.arcs, net.p, net.s, net.t)
        assert B.bat_last_launch().perm == 5
        ks.append(B.bat_last_launch().kernel_ms)
    got = min(ks) * 1e6 / 2.0 ** net.m
    assert 0.5 * got <= ns <= 2.0 * got, (ns, got)


def test_reports_while_a_stream_is_captured():
    """bat_last_launch after an asynchronous sweep, called while the thread
    captures another stream, waits and leaves the capture whole; a captured
    launch has no times, and its replays none to spoil."""
    import torch
    B = _B()
    long, short = W.random_connected(24, 46, seed=1, p_lo=0.6, p_hi=0.99), W.random_connected(9, 16, seed=72)
    side = torch.cuda.Stream()
    pl, ps = (torch.tensor(x.p, dtype=torch.float64, device="cuda") for x in (long, short))
    out = [(torch.zeros((), dtype=torch.float64, device="cuda"), torch.zeros((), dtype=torch.int64, device="cuda"))
           for _ in range(2)]

    def launch(x, p, o, stream):
        B.bat_reliability_async(x.n, x.arcs, p.data_ptr(), x.s, x.t, o[0].data_ptr(), o[1].data_ptr(), None,
                                stream.cuda_stream)
    launch(long, pl, out[0], side)
    launch(short, ps, out[1], side)
    torch.cuda.synchronize()
    print("capture and report", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(torch.cuda.Stream()):
        launch(long, pl, out[0], side)
        g.capture_begin()
        li = B.bat_last_launch()
        launch(short, ps, out[1], torch.cuda.current_stream())
        with pytest.raises(B.BatError) as e:
            B.bat_last_launch()
        g.capture_end()
    assert li.vectors == 1 << long.m and 1.0 < li.kernel_ms <= li.total_ms
    assert e.value.code == B.BAT_EDEVICE
    want = B.bat_reliability(short.n, short.arcs, short.p, short.s, short.t)
    for k in range(20):
        out[1][0].zero_()
        out[1][1].zero_()
        launch(long, pl, out[0], side) if k == 3 else launch(short, ps, out[1], side)
        g.replay()
        li = B.bat_last_launch()
        assert 0.0 < li.kernel_ms <= li.total_ms < 1e4, k
        torch.cuda.synchronize()
        assert (float(out[1][0]), int(out[1][1])) == want, k


def test_noalloc_on_a_new_thread():
    """Its first call there, reported through events or the thread's slots."""
    import threading

    import torch
    B = _B()
    net = W.random_connected(12, 24, seed=73)
    p = torch.tensor(net.p, dtype=torch.float64, device="cuda")
    R, cnt = torch.zeros((), dtype=torch.float64, device="cuda"), torch.zeros((), dtype=torch.int64, device="cuda")
    got = []

    def work():
        for _ in range(2):
            B.bat_reliability_noalloc(net.n, net.arcs, p.data_ptr(), net.s, net.t, R.data_ptr(), cnt.data_ptr(), None,
                                      torch.cuda.current_stream().cuda_stream)
            got.append(B.bat_last_launch())
    print("noalloc on a thread", flush=True)
    th = threading.Thread(target=work)
    th.start()
    th.join()
    torch.cuda.synchronize()
    assert (float(R), int(cnt)) == B.bat_reliability(net.n, net.arcs, net.p, net.s, net.t)
    assert len(got) == 2 and all(0.0 < li.kernel_ms <= li.total_ms and li.perm == 5 for li in got)


@pytest.mark.parametrize("n,m", [(4, 5), (10, 18), (13, 25), (16, 34)])
def test_outputs_in_the_place_of_p(n, m):
    """The device forms check p before any output is written: each output in
    turn overwrites p, with the results of separate buffers; an invalid p is
    found all the same."""
    import torch
    B = _B()
    net = W.random_connected(n, m, seed=m, p_lo=0.5, p_hi=0.99)
    st = torch.zeros((), dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream

    def sweep(bad, place):
        """place: which output lies where p does."""
        p = torch.tensor(net.p, dtype=torch.float64, device="cuda")
        if bad:
            p[m - 1] = 1.5
        out = {k: torch.zeros(m, dtype=torch.float64, device="cuda") for k in ("R", "d", "T1", "T0")}
        cnt = torch.zeros((), dtype=torch.int64, device="cuda")
        if place:
            out[place] = p
        B.bat_reliability_grad_async(n, net.arcs, p.data_ptr(), net.s, net.t, out["R"].data_ptr(), cnt.data_ptr(),
                                     out["d"].data_ptr(), out["T1"].data_ptr(), out["T0"].data_ptr(), st.data_ptr(), stream)
        assert B.bat_last_launch().perm == 5
        got = {k: (v[:1] if k == "R" else v).cpu().numpy() for k, v in out.items()}
        return got, int(cnt), int(st)
    print("outputs over p", n, m, flush=True)
    want = sweep(False, None)
    assert want[2] == 0
    for place in ("d", "T1", "T0", "R"):
        got = sweep(False, place)
        assert got[1:] == want[1:] and all(np.array_equal(got[0][k], want[0][k]) for k in want[0]), place
        got = sweep(True, place)
        assert got[2] == B.BAT_EINVAL and all(np.isnan(v).all() for v in got[0].values()), place


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("levels,m", [(2, 26), (3, 25)])
def test_checkpoint_resumed_under_another_split(tmp_path, levels, m, grad):
    """The file keeps how the items are cut, so that the parts after an
    interruption are summed as those before it: the same file, bit for bit,
    whatever the split then set; a cut that the library does not make is
    refused."""
    B = _B()
    net = W.random_connected(13, m, seed=23, p_lo=0.4, p_hi=0.99)
    args = (net.n, net.arcs, net.p, net.s, net.t, m - 2)
    whole, cut = str(tmp_path / "whole.ckpt"), str(tmp_path / "cut.ckpt")
    old = {k: B.bat_get_option(k) for k in ("BAT_CUBES", "BAT_CUBE_LEVELS", "BAT_CUBE_SPLIT")}
    try:
        for k, v in {"BAT_CUBES": 1, "BAT_CUBE_LEVELS": levels, "BAT_CUBE_SPLIT": 1}.items():
            B.bat_set_option(k, v)
        print("checkpoint split", levels, m, grad, flush=True)
        B.bat_reliability_checkpointed(*args, whole, grad=grad)
        assert B.bat_reliability_checkpointed(*args, cut, grad=grad, max_chunks=2) is None
        B.bat_set_option("BAT_CUBE_SPLIT", 3)
        lines = open(cut).read().splitlines()
        for a, b in (("split=1 ", "split=65 "), ("units=", "units=1000"), ("chunk=1 ", "chunk=0 "), ("split=1 ", "")):
            assert a in lines[3]
            bad = str(tmp_path / "bad.ckpt")
            open(bad, "w").write("\n".join(lines[:3] + [lines[3].replace(a, b)] + lines[4:]) + "\n")
            with pytest.raises(B.BatError) as e:
                B.bat_reliability_checkpointed(*args, bad, grad=grad)
            assert e.value.code == B.BAT_EIO
        B.bat_reliability_checkpointed(*args, cut, grad=grad)
    finally:
        for k, v in old.items():
            B.bat_set_option(k, v)
    assert open(cut).read() == open(whole).read()


@pytest.mark.parametrize("option,value", [("BAT_JIT", 0), ("BAT_JIT", 1), ("BAT_CUBES", 0), ("BAT_CHUNK_LOG2", 7)])
def test_checkpoint_resumed_under_other_options(tmp_path, option, value):
    """A sweep begun by sub-cubes goes on so, whatever is set since."""
    B = _B()
    net = W.random_connected(16, 34, seed=24, p_lo=0.6, p_hi=0.99)
    args = (net.n, net.arcs, net.p, net.s, net.t, net.m - 1)
    want = B.bat_reliability_checkpointed(*args, None)
    f = str(tmp_path / "c.ckpt")
    assert B.bat_reliability_checkpointed(*args, f, max_chunks=1) is None
    old = B.bat_get_option(option)
    print("checkpoint", option, value, flush=True)
    try:
        B.bat_set_option(option, value)
        assert B.bat_reliability_checkpointed(*args, f) == want
    finally:
        B.bat_set_option(option, old)


@pytest.mark.parametrize("run", [0, 1, 40, 1 << 20])
@pytest.mark.parametrize("states", [2, 3, 5, 9, 12, 32])
def test_multi_state_flow_of_many_states(states, run):
    """The flow kernel's cubes over arcs of many states, their capacities in
    order, in no order, equal for several states: whole spaces and ranges
    against the oracle.  R: compensated sums of products of at most 13
    factors, one a sum of up to 32 terms, some 45 roundings of 1.1e-16."""
    B = _B()
    rng = np.random.default_rng(2500 + states)
    m = {2: 13, 3: 9, 5: 6, 9: 4, 12: 4, 32: 3}[states]
    old = {k: B.bat_get_option(k) for k in ("BAT_MS_RUN", "BAT_MS_BITS")}
    try:
        B.bat_set_option("BAT_MS_BITS", 0)
        B.bat_set_option("BAT_MS_RUN", run)
        for k in range(6):
            n = int(rng.integers(3, 7))
            net = W.random_multigraph(n, m, seed=int(rng.integers(1 << 30)))
            cap = rng.integers(0, 2 * states if k % 2 else 4, (m, states))
            if k < 4:
                cap = np.sort(cap, axis=1)
            w = rng.uniform(0.0, 1.0, (m, states))
            args = (net.n, net.arcs, [states] * m, cap, w / w.sum(axis=1, keepdims=True), 0, net.n - 1,
                    int(rng.integers(1, 3 * states)))
            N = states ** m
            lo, hi = sorted(int(x) for x in rng.integers(0, N + 1, 2))
            print("multi-state flow", states, run, k, net.n, m, args[-1], lo, hi, flush=True)
            R, cnt = B.bat_ms_reliability(*args, directed=k == 3)
            r = B.bat_ms_reliability_range(*args, lo, hi, directed=k == 3)
            o = oracle.ms_reliability(*args, directed=k == 3)
            p = oracle.ms_reliability_range(*args, lo, hi, directed=k == 3)
            assert (cnt, r.count) == (o.count, p.count)
            assert abs(R - o.sum) <= 5e-15 * o.sum and abs(r.R - p.sum) <= 5e-15 * p.sum
    finally:
        for k, v in old.items():
            B.bat_set_option(k, v)


@pytest.mark.parametrize("n_pvec", [1, 0])
def test_ranges_and_single_vectors_to_rounding(n_pvec):
    """One probability vector per graph, and ranges (n_pvec 0): products of at
    most 30 factors and compensated sums, as whole sweeps: some 30 roundings
    of 1.1e-16."""
    B = _B()
    rng = np.random.default_rng(2600)
    nets = [W.random_connected(n, m, seed=m + 7, p_lo=0.2, p_hi=0.99)
            for n, m in ((4, 5), (6, 9), (7, 11), (8, 13), (9, 16), (11, 18), (12, 20))]
    print("to rounding", n_pvec, flush=True)
    if n_pvec:
        R, cnt = B.bat_reliability_batched([(x.n, x.arcs, x.s, x.t) for x in nets], [x.p[None, :] for x in nets])
        assert B.bat_last_launch().perm == 5
    for k, x in enumerate(nets):
        if n_pvec:
            got, c, o = R[k, 0], cnt[k], oracle.reliability(x.n, x.arcs, x.p, x.s, x.t)
        else:
            lo, hi = sorted(int(v) for v in rng.integers(0, (1 << x.m) + 1, 2))
            r = B.bat_reliability_range(x.n, x.arcs, x.p, x.s, x.t, lo, hi)
            assert B.bat_last_launch().perm == 5 or lo == hi
            got, c, o = r.R, r.count, oracle.reliability_range(x.n, x.arcs, x.p, x.s, x.t, lo, hi)
        assert c == o.count and abs(got - o.sum) <= 4e-15 * o.sum, (k, got, o.sum)


@pytest.mark.parametrize("demand", [1, 2])
def test_multi_state_cubes_as_accurate_as_every_word(demand):
    """Root mean square error of R over 4 networks of 9 arcs with 40 sets of
    weights each, against every vector in extended precision (max-flow
    min-cut): no more than that of the sweep of every word (two such values
    over 160 samples scatter by some 6% each).  Tables rounded at each factor
    gave 1.5 and 1.6 times its error."""
    B = _B()
    L = np.longdouble
    x = np.stack([np.arange(3 ** 9) // 3 ** k % 3 for k in range(9)], axis=1)
    err = {0: [], 1: []}
    old = B.bat_get_option("BAT_CUBES")
    try:
        for k in range(4):
            net = W.random_connected(6, 9, seed=40 + k)
            sides = [{net.s} | {v for j, v in enumerate(v for v in range(6) if v not in (net.s, net.t)) if c >> j & 1}
                     for c in range(16)]
            across = np.array([[(a in s) != (b in s) for s in sides] for a, b in net.arcs], int)
            ok = (x @ across).min(axis=1) >= demand
            for j in range(40):
                rng = np.random.default_rng([k, j])
                w = rng.uniform(0.02, 0.3, (9, 3))
                w[:, 2] = 1.0 - w[:, 0] - w[:, 1]
                want = np.prod(w.astype(L)[np.arange(9), x], axis=1)[ok].sum()
                for v in err:
                    B.bat_set_option("BAT_CUBES", v)
                    R, cnt = B.bat_ms_reliability(6, net.arcs, [3] * 9, [0, 1, 2] * 9, list(w.ravel()), net.s, net.t,
                                                  demand)
                    assert cnt == ok.sum() and (B.bat_last_launch().perm == 5) == (v == 1)
                    err[v].append(float((R - want) / want))
    finally:
        B.bat_set_option("BAT_CUBES", old)
    rms = {v: float(np.sqrt((np.array(e) ** 2).mean())) for v, e in err.items()}
    print("rms errors: every word", rms[0], "cubes", rms[1], flush=True)
    assert rms[1] <= 1.2 * rms[0]
