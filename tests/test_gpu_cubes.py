"""The sub-cube sweep (whole sweeps that decide and add connected cubes of
vectors as one) against the oracle and the frontier DP, at the sizes where
its split changes: fewer arcs than a word, one lane, one and several work
items, each number of levels, items shared by several wavefronts.  Counts
are exact; R within 2e-15 relative (products of at most 30 factors and
compensated sums: about 30 roundings of 1.1e-16, met by the frontier DP's
own plain sums).
"""
import contextlib

import numpy as np
import pytest

import bat_workloads as W
import oracle
from oracle import frontier_dp

pytestmark = pytest.mark.gpu

REL = 4e-15


def _B():
    import paper_2209_09711_amd as B
    return B


@contextlib.contextmanager
def options(**kw):
    B = _B()
    old = {k: B.bat_get_option(k) for k in kw}
    try:
        for k, v in kw.items():
            B.bat_set_option(k, v)
        yield
    finally:
        for k, v in old.items():
            B.bat_set_option(k, v)


def _digraph(n, m, seed):
    rng = np.random.default_rng(seed)
    arcs = [tuple(int(x) for x in rng.choice(n, 2, replace=False)) for _ in range(m)]
    return W.Network(f"di{n}_{m}", n, arcs, 0, n - 1, rng.uniform(0.3, 0.95, m))


def _nets():
    out = [(W.bridge(0.9), False), (W.figure1(), False), (W.parallel(3, [0.2, 0.5, 0.7]), False),
           (W.grid(2, 4, p=np.linspace(0.5, 0.95, 10)), False), (W.grid(3, 4, p=np.linspace(0.4, 0.98, 17)), False)]
    for n, m in [(2, 1), (4, 4), (6, 10), (7, 11), (7, 12), (8, 15), (9, 16), (10, 17), (11, 21), (12, 22)]:
        out.append((W.random_connected(n, m, seed=40 + m, p_lo=0.2, p_hi=0.99), False))
    for k in range(3):
        out.append((W.random_multigraph(5, 11 + k, seed=60 + k), False))
        out.append((_digraph(8, 14 + 2 * k, 70 + k), True))
    return out


@pytest.mark.parametrize("levels", [1, 2, 3])
@pytest.mark.parametrize("split", [1, 3, 16])
def test_cubes_vs_oracle(levels, split):
    B = _B()
    with options(BAT_CUBES=1, BAT_CUBE_LEVELS=levels, BAT_CUBE_SPLIT=split):
        for net, directed in _nets():
            print("cubes", levels, split, net.name, net.n, net.m, flush=True)
            R, cnt = B.bat_reliability_ex(net.n, net.arcs, net.p, net.s, net.t, directed=directed)
            li = B.bat_last_launch()
            o = oracle.reliability(net.n, net.arcs, net.p, net.s, net.t, directed=directed)
            assert li.perm == 5 and 0.0 < li.kernel_ms <= li.total_ms
            assert cnt == o.count, net.name
            assert abs(R - o.sum) <= REL * o.sum, (net.name, R, o.sum)


@pytest.mark.parametrize("n,m,seed", [(13, 26, 3), (14, 27, 4), (16, 29, 5), (11, 30, 6), (18, 31, 7)])
def test_cubes_larger_vs_frontier_dp(n, m, seed):
    """The default launch (two levels from 24 relevant arcs on, several work
    items per block), twice with the same bits."""
    B = _B()
    net = W.random_connected(n, m, seed=seed, p_lo=0.5, p_hi=0.99)
    print("cubes", net.name, flush=True)
    R, cnt = B.bat_reliability(net.n, net.arcs, net.p, net.s, net.t)
    assert B.bat_last_launch().perm == 5
    assert (R, cnt) == B.bat_reliability(net.n, net.arcs, net.p, net.s, net.t)
    Rd, cd = frontier_dp.reliability(net.n, net.arcs, net.p, net.s, net.t)
    assert cnt == cd and abs(R - Rd) <= REL * Rd


@pytest.mark.parametrize("levels", [1, 2, 3])
def test_cubes_specialised(levels):
    """The graph-specialised build against the oracle, and as every other
    launch: the same count, R within rounding."""
    B = _B()
    nets = [_nets()[k] for k in (0, 3, 4, 9, 12, 14, 16, 18)]
    for net, directed in nets:
        print("specialised cubes", levels, net.name, flush=True)
        with options(BAT_CUBES=1, BAT_JIT=1, BAT_CUBE_LEVELS=levels):
            R, cnt = B.bat_reliability_ex(net.n, net.arcs, net.p, net.s, net.t, directed=directed)
            assert B.bat_last_launch().specialised == 1
        o = oracle.reliability(net.n, net.arcs, net.p, net.s, net.t, directed=directed)
        assert cnt == o.count and abs(R - o.sum) <= REL * o.sum, net.name


@pytest.mark.parametrize("n,m", [(12, 32), (16, 33), (26, 38), (40, 44)])
def test_cubes_specialised_larger(n, m):
    """2^32 vectors and more (three levels from 33 relevant arcs on; more
    than 32 counter bits; more nodes than a 32-bit node set)."""
    B = _B()
    net = W.random_connected(n, m, seed=m, p_lo=0.6, p_hi=0.99)
    print("specialised cubes", net.name, flush=True)
    R, cnt = B.bat_reliability(net.n, net.arcs, net.p, net.s, net.t)
    li = B.bat_last_launch()
    assert li.specialised == 1 and li.perm == 5
    Rd, cd = frontier_dp.reliability(net.n, net.arcs, net.p, net.s, net.t)
    assert cnt == cd and abs(R - Rd) <= REL * Rd


def test_cubes_exact_probabilities():
    """p = 1/2 gives count 2^-m to the bit; p of 0 and 1 stay exact."""
    B = _B()
    net = W.random_connected(13, 25, seed=9)
    with options(BAT_CUBES=1, BAT_CUBE_LEVELS=3):
        R, cnt = B.bat_reliability(net.n, net.arcs, np.full(net.m, 0.5), net.s, net.t)
        assert R == cnt * 2.0 ** -net.m
        assert B.bat_reliability(net.n, net.arcs, np.ones(net.m), net.s, net.t) == (1.0, cnt)
        assert B.bat_reliability(net.n, net.arcs, np.zeros(net.m), net.s, net.t) == (0.0, cnt)


def test_cubes_checkpointed(tmp_path):
    """A sub-cube sweep in parts: resumed bitwise the uninterrupted one, and
    a file whose work items this library does not cut is refused."""
    B = _B()
    net = W.random_connected(12, 24, seed=21, p_lo=0.4, p_hi=0.99)
    o = oracle.net_reliability(net)
    with options(BAT_CUBES=1, BAT_CUBE_LEVELS=2):
        args = (net.n, net.arcs, net.p, net.s, net.t, net.m - 3)
        whole = B.bat_reliability_checkpointed(*args, None)
        f = str(tmp_path / "c.ckpt")
        assert B.bat_reliability_checkpointed(*args, f, max_chunks=3) is None
        lines = open(f).read().splitlines()
        assert lines[2] == "parts 8" and lines[3].startswith("launch order=5 ") and lines[4] == "done 3"
        bad = str(tmp_path / "bad.ckpt")
        for launch in (lines[3][:-1] + ("0" if lines[3][-1] != "0" else "1"), "launch order=5 items=80 chain=0",
                       "launch order=5 items=7 chain=0 bits=0"):
            open(bad, "w").write("\n".join(lines[:3] + [launch] + lines[4:]) + "\n")
            with pytest.raises(B.BatError) as e:
                B.bat_reliability_checkpointed(*args, bad)
            assert e.value.code == B.BAT_EIO
    # the file's launch holds when the options have changed since
    assert B.bat_reliability_checkpointed(*args, f) == whole
    assert whole[1] == o.count and abs(whole[0] - o.sum) <= REL * o.sum


# T1 and T0: a lane adds its words' terms, all of one sign, by plain fused
# additions, at most some 2^9 of them between folds at these sizes: 2^9
# roundings of 1.1e-16 at worst.
REL_GRAD = 6e-14


def _rel(a, b):
    a, b = np.asarray(a), np.asarray(b)
    assert np.all(a[b == 0.0] == 0.0)
    return float(np.max(np.abs(a - b)[b != 0.0] / b[b != 0.0], initial=0.0))


@pytest.mark.parametrize("levels", [1, 2, 3])
@pytest.mark.parametrize("split,jit", [(1, 0), (3, 0), (16, 0), (2, 1)])
def test_cube_gradients_vs_oracle(levels, split, jit):
    B = _B()
    nets = _nets()
    nets.append((W.bridge(0.9).with_p([1.0, 0.0, 0.7, 1.0, 0.0]), False))
    nets.append((W.Network("loops", 4, [(0, 1), (1, 1), (1, 3), (2, 2), (0, 2)], 0, 3,
                           np.array([.9, .5, .8, .3, .7])), False))
    if jit:
        nets = [nets[k] for k in (0, 4, 9, 12, 14, 16, 18, len(nets) - 2)]
    with options(BAT_CUBES=1, BAT_JIT=jit, BAT_CUBE_LEVELS=levels, BAT_CUBE_SPLIT=split):
        for net, directed in nets:
            print("cube gradients", levels, split, jit, net.name, net.n, net.m, flush=True)
            g = B.bat_reliability_ex(net.n, net.arcs, net.p, net.s, net.t, directed=directed, grad=True)
            li = B.bat_last_launch()
            assert li.perm == 5 and li.specialised == jit
            o = oracle.reliability(net.n, net.arcs, net.p, net.s, net.t, grad=True, directed=directed)
            assert g.count == o.count, net.name
            assert abs(g.R - o.sum) <= REL * o.sum, net.name
            assert _rel(g.T1, o.T1) <= REL_GRAD and _rel(g.T0, o.T0) <= REL_GRAD, net.name


@pytest.mark.parametrize("n,m", [(13, 25), (14, 27), (20, 30), (12, 32), (16, 34)])
def test_cube_gradients_larger(n, m):
    """The default launch at the sizes where levels, splits and the
    specialised build begin; the same bits twice and through device
    pointers."""
    import torch
    from paper_2209_09711_amd.torch_fn import reliability
    B = _B()
    net = W.random_connected(n, m, seed=m, p_lo=0.5, p_hi=0.99)
    print("cube gradients", net.name, flush=True)
    g = B.bat_reliability_grad(net.n, net.arcs, net.p, net.s, net.t)
    assert B.bat_last_launch().perm == 5
    h = B.bat_reliability_grad(net.n, net.arcs, net.p, net.s, net.t)
    assert (g.R, g.count) == (h.R, h.count) and np.array_equal(g.T1, h.T1) and np.array_equal(g.T0, h.T0)
    Rd, cd = frontier_dp.reliability(net.n, net.arcs, net.p, net.s, net.t)
    T1, T0 = frontier_dp.gradient(net.n, net.arcs, net.p, net.s, net.t)
    assert g.count == cd and abs(g.R - Rd) <= REL * Rd
    assert _rel(g.T1, T1) <= REL_GRAD and _rel(g.T0, T0) <= REL_GRAD
    p = torch.tensor(net.p, dtype=torch.float64, device="cuda", requires_grad=True)
    R, cnt = reliability(p, net.n, net.arcs, net.s, net.t)
    assert int(cnt) == g.count
    R.backward()
    assert abs(R.item() - g.R) <= 2.3e-16 * g.R
    np.testing.assert_allclose(p.grad.cpu().numpy(), g.T1 - g.T0, rtol=0, atol=REL_GRAD)


def test_cube_gradients_checkpointed(tmp_path):
    B = _B()
    net = W.random_connected(12, 24, seed=22, p_lo=0.4, p_hi=0.99)
    args = (net.n, net.arcs, net.p, net.s, net.t, net.m - 2)
    whole = B.bat_reliability_checkpointed(*args, None, grad=True)
    f = str(tmp_path / "g.ckpt")
    assert B.bat_reliability_checkpointed(*args, f, grad=True, max_chunks=1) is None
    assert open(f).read().splitlines()[3].startswith("launch order=5 ")
    got = B.bat_reliability_checkpointed(*args, f, grad=True)
    assert (got.R, got.count) == (whole.R, whole.count) and np.array_equal(got.dRdp, whole.dRdp)
    o = oracle.net_reliability(net, grad=True)
    assert got.count == o.count and _rel(got.T1, o.T1) <= REL_GRAD and _rel(got.T0, o.T0) <= REL_GRAD


@pytest.mark.parametrize("levels", [0, 1, 2])
@pytest.mark.parametrize("n_pvec", [1, 2, 5, 12, 32, 33])
def test_cube_batches_vs_oracle(n_pvec, levels):
    """Batches by sub-cubes: one kernel for each number of vectors a word's
    sum is spread over, graphs of no arc, fewer arcs than a word, one and
    several work items, probabilities of 1; the same bits twice."""
    B = _B()
    rng = np.random.default_rng(2000 + n_pvec)
    graphs, pblocks = [], []
    for k in range(13):
        if k % 5 == 4:
            net = W.random_multigraph(int(rng.integers(2, 7)), int(rng.integers(0, 12)), seed=int(rng.integers(1 << 30)))
        else:
            n = int(rng.integers(3, 12))
            net = W.random_connected(n, int(rng.integers(n - 1, min(17, n * (n - 1) // 2) + 1)),
                                     seed=int(rng.integers(1 << 30)))
        s, t = (int(x) for x in rng.choice(net.n, 2, replace=False))
        graphs.append((net.n, net.arcs, s, t))
        pblocks.append(np.where(rng.random((n_pvec, len(net.arcs))) < 0.05, 1.0,
                                rng.uniform(0.0, 1.0, (n_pvec, len(net.arcs)))))
    with options(BAT_CUBE_LEVELS=levels):
        print("cube batch", levels, n_pvec, flush=True)
        R, cnt = B.bat_reliability_batched(graphs, pblocks)
        assert B.bat_last_launch().perm == 5
        R2, cnt2 = B.bat_reliability_batched(graphs, pblocks)
    assert np.array_equal(R, R2) and np.array_equal(cnt, cnt2)
    for g, (n, arcs, s, t) in enumerate(graphs):
        for j in sorted({g % n_pvec, n_pvec - 1}):
            o = oracle.reliability(n, arcs, pblocks[g][j], s, t)
            assert cnt[g] == o.count and abs(R[g, j] - o.sum) <= REL_GRAD * o.sum, (g, j)


@pytest.mark.parametrize("n_pvec", [1, 20])
def test_cube_batch_two_launches(n_pvec):
    """More graphs than one launch takes, up to 27 arcs, against single
    sweeps; a graph of more arcs than the kernels hold sends the whole batch
    to the plain launch."""
    B = _B()
    rng = np.random.default_rng(2100)
    graphs, pblocks = [], []
    for k in range(70):
        m = 27 if k == 33 else 9 + k % 16
        net = W.random_connected(max(6, m // 2), m, seed=3000 + k)
        graphs.append((net.n, net.arcs, net.s, net.t))
        pblocks.append(rng.uniform(0.4, 0.99, (n_pvec, m)))
    print("cube batch of 70", n_pvec, flush=True)
    R, cnt = B.bat_reliability_batched(graphs, pblocks)
    assert B.bat_last_launch().perm == 5
    for g in range(0, 70, 3):
        n, arcs, s, t = graphs[g]
        Rg, cg = B.bat_reliability(n, arcs, pblocks[g][g % n_pvec], s, t)
        assert cnt[g] == cg and abs(R[g, g % n_pvec] - Rg) <= REL_GRAD * Rg
    ring = (34, [(i, (i + 1) % 34) for i in range(34)], 0, 17)
    p = rng.uniform(0.9, 0.999, (n_pvec, 34))
    R, cnt = B.bat_reliability_batched(graphs[:2] + [ring], pblocks[:2] + [p])
    assert B.bat_last_launch().perm != 5
    want = 1.0 - (1.0 - np.prod(p[:, :17], axis=1)) * (1.0 - np.prod(p[:, 17:], axis=1))
    assert np.allclose(R[2], want, rtol=1e-13, atol=0) and cnt[2] == (1 << 34) - ((1 << 17) - 1) ** 2


def test_cube_batch_of_many_entries():
    """More entries than one sweep takes."""
    B = _B()
    rng = np.random.default_rng(2200)
    nets = [W.random_connected(6 + k % 4, 9 + k % 5, seed=4000 + k) for k in range(23)]
    graphs = [(nets[k % 23].n, nets[k % 23].arcs, 0, nets[k % 23].n - 1) for k in range(1100)]
    pblocks = [rng.uniform(0.1, 0.99, (2, len(g[1]))) for g in graphs]
    print("cube batch of 1100", flush=True)
    R, cnt = B.bat_reliability_batched(graphs, pblocks)
    li = B.bat_last_launch()
    assert li.perm == 5 and 0.0 < li.kernel_ms <= li.total_ms
    for g in list(range(0, 1100, 37)) + [1023, 1024, 1099]:
        o = oracle.reliability(graphs[g][0], graphs[g][1], pblocks[g][1], graphs[g][2], graphs[g][3])
        assert cnt[g] == o.count and abs(R[g, 1] - o.sum) <= REL_GRAD * o.sum, g


@pytest.mark.parametrize("forward", [False, True])
def test_cube_ranges_vs_oracle(forward):
    """Ranges of the paper's counters as aligned cubes and windowed ends:
    from 0, to the end, aligned, inside one block, of one vector; graphs whose
    leading arcs join or separate the terminals."""
    B = _B()
    rng = np.random.default_rng(2300 + forward)
    nets = [W.parallel(3, [0.2, 0.5, 0.7]), W.series(6, np.full(6, 0.9)), W.bridge(0.9),
            W.Network("apart", 4, [(0, 1), (2, 3)], 0, 3, np.full(2, 0.5)), W.random_multigraph(5, 12, seed=3)]
    nets += [W.random_connected(n, m, seed=80 + m, p_lo=0.0, p_hi=1.0) for n, m in ((6, 11), (8, 15), (9, 17), (11, 18))]
    for net in nets:
        end = 1 << net.m
        lo, hi = sorted(int(x) for x in rng.integers(0, end + 1, 2))
        part = max(1, end >> 3)
        for a, b in {(0, hi), (lo, end), (lo, hi), (lo // part * part, min(end, lo // part * part + part)), (lo, lo + 1)}:
            if a == b or b > end:
                continue
            print("cube range", net.name, net.m, a, b, forward, flush=True)
            r = B.bat_reliability_range(net.n, net.arcs, net.p, net.s, net.t, a, b, forward=forward)
            assert B.bat_last_launch().perm == 5
            o = oracle.reliability_range(net.n, net.arcs, net.p, net.s, net.t, a, b, forward=forward)
            assert r.count == o.count and abs(r.R - o.sum) <= REL_GRAD * o.sum


@pytest.mark.parametrize("n,m,lo,hi", [(12, 24, 12345, 7654321), (13, 25, 1 << 20, 3 << 20), (14, 27, 1 << 26, 1 << 27),
                                       (15, 30, (1 << 30) // 100 * 17, (1 << 30) // 100 * 18), (13, 33, 0, 1 << 33)])
def test_cube_ranges_larger(n, m, lo, hi):
    """Several cubes of both numbers of levels, against the plain sweep of
    the range: the same count, R within rounding."""
    B = _B()
    net = W.random_connected(n, m, seed=m, p_lo=0.5, p_hi=0.99)
    for forward in (False, True):
        print("cube range", net.name, lo, hi, forward, flush=True)
        r = B.bat_reliability_range(net.n, net.arcs, net.p, net.s, net.t, lo, hi, forward=forward)
        assert B.bat_last_launch().perm == 5
        with options(BAT_CUBES=0):
            q = B.bat_reliability_range(net.n, net.arcs, net.p, net.s, net.t, lo, hi, forward=forward)
            assert B.bat_last_launch().perm != 5
        assert r.count == q.count and abs(r.R - q.R) <= REL_GRAD * q.R


def test_cube_reports_of_overlapping_launches():
    """Synchronous calls while asynchronous launches, more than there are
    report slots, and a replayed graph still write their reports."""
    import torch
    B = _B()
    long, short = W.random_connected(16, 34, seed=71, p_lo=0.6, p_hi=0.99), W.random_connected(9, 16, seed=72)
    want = [B.bat_reliability(x.n, x.arcs, x.p, x.s, x.t) for x in (long, short)]
    side = torch.cuda.Stream()
    pl, ps = (torch.tensor(x.p, dtype=torch.float64, device="cuda") for x in (long, short))
    out = [(torch.zeros((), dtype=torch.float64, device="cuda"), torch.zeros((), dtype=torch.int64, device="cuda"))
           for _ in range(3)]

    def launch(x, p, o, stream):
        B.bat_reliability_async(x.n, x.arcs, p.data_ptr(), x.s, x.t, o[0].data_ptr(), o[1].data_ptr(), None,
                                stream.cuda_stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.bat_reliability_noalloc(short.n, short.arcs, ps.data_ptr(), short.s, short.t, out[2][0].data_ptr(),
                                  out[2][1].data_ptr(), None, torch.cuda.current_stream().cuda_stream)
    for k in range(40):
        launch(long, pl, out[0], side)
        launch(short, ps, out[1], torch.cuda.current_stream())
        g.replay()
        assert B.bat_reliability(short.n, short.arcs, short.p, short.s, short.t) == want[1], k
        li = B.bat_last_launch()
        assert 0.0 < li.kernel_ms <= li.total_ms
    launch(short, ps, out[1], torch.cuda.current_stream())
    B.bat_last_launch()
    torch.cuda.synchronize()
    for o, w in zip(out, (want[0], want[1], want[1])):
        assert int(o[1]) == w[1] and abs(float(o[0]) - w[0]) <= REL * w[0]
