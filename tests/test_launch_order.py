"""The order in which the library's work reaches the device, on a recording
HIP runtime (no GPU is needed)."""
import pytest

import recorder


def _batch(graphs, pvec, arcs=12):
    return f"""
nets = [W.random_connected(8, {arcs}, seed=50 + k) for k in range({graphs})]
g = [(x.n, x.arcs, x.s, x.t) for x in nets]
p = [np.full(({pvec}, {arcs}), 0.5) for _ in g]
try:
    B.bat_reliability_batched(g, p)
except B.BatError as e:
    result = e.code
"""


_RANGE = """
x = W.random_connected(16, 40, seed=9)
try:
    B.bat_reliability_range(x.n, x.arcs, x.p, x.s, x.t, 0, 70 << 32)
except B.BatError as e:
    result = e.code
"""

BATCHES = [_batch(16, 3), _batch(70, 3), _batch(3, 1024), _batch(40, 100), _batch(70, 1), _batch(1100, 2), _RANGE]


@pytest.mark.parametrize("code", BATCHES, ids=["16x3", "70x3", "3x1024", "40x100", "70x1", "1100x2", "range"])
def test_batch_launches_follow_their_copies(code):
    """Every launch of a sub-cube batch, also the one on the side stream,
    starts after all that was copied for it: the table of its blocks goes up
    with the first copy."""
    code, ops = recorder.run(code, fail="finish")
    assert code == -3
    sweeps = [i for i, o in enumerate(ops) if o.kind == "launch" and "k_cube_batch" in o.args[1] and not o.failed]
    copies = [i for i, o in enumerate(ops) if o.kind == "copy"]
    assert sweeps and copies
    for i in sweeps:
        assert {c for c in copies if c < i} <= ops[i].after
    # and the reduction after them all
    (end,) = [i for i, o in enumerate(ops) if o.kind == "launch" and o.failed]
    last = max(i for i in range(end) if ops[i].kind != "sync" and ops[i].stream == ops[end].stream)
    assert set(sweeps) <= ops[last].after | {last}


@pytest.mark.parametrize("code", [BATCHES[1], BATCHES[6]], ids=["70x3", "range"])
def test_failed_batch_leaves_nothing_in_flight(code):
    """Whichever call fails, both streams are waited for before the batch
    returns: the thread's next call uses the same buffers."""
    for k in range(40):
        rc, ops = recorder.run(code, fail=f"#{k},k_cube_batch_finish")
        assert rc == -3, k
        queued = {o.stream for o in ops if o.kind in ("copy", "launch") and not o.failed}
        for s in queued:
            last = max(i for i, o in enumerate(ops) if o.kind in ("copy", "launch") and o.stream == s and not o.failed)
            assert any(o.kind == "sync" and o.stream == s for o in ops[last:]), (k, s)
        if any(o.failed and o.kind == "launch" and "finish" in o.args[1] for o in ops):
            break
    assert 6 < k < 39


@pytest.mark.parametrize("states,arcs,demand", [(3, 27, 1), (3, 27, 2), (3, 32, 1), (4, 31, 1), (2, 32, 3),
                                                  (3, 30, 4), (3, 32, 7), (4, 31, 5)])
def test_large_multi_state_spaces_are_launched(states, arcs, demand):
    """Whole multi-state spaces of any accepted size: the launch stays under
    2^32 threads (which the recorder refuses, as HIP does) and its partials
    under a few MiB."""
    rc, ops = recorder.run(f"""
x = W.random_connected(14, {arcs}, seed=5)
try:
    B.bat_ms_reliability(x.n, x.arcs, [{states}] * {arcs}, list(range({states})) * {arcs},
                         [1.0 / {states}] * {states * arcs}, x.s, x.t, {demand})
except B.BatError as e:
    result = e.code
""", fail="finish")
    assert rc == -3
    sweeps = [o for o in ops if o.kind == "launch" and "finish" not in o.args[1]]
    assert sweeps and not any(o.failed for o in sweeps)
    assert sum(int(o.args[1]) for o in ops if o.kind == "alloc") < 16 << 20


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("m", [44, 45, 51, 56, 62])
def test_large_sweeps_are_launched(m, grad):
    """Whole sweeps by sub-cubes up to the most arcs: the launch stays under
    2^32 threads and its partials under a few MiB, at the default split and
    at the largest."""
    for split in (0, 64):
        rc, ops = recorder.run(f"""
x = W.random_connected(30, {m}, seed=4)
B.bat_set_option("BAT_CUBE_SPLIT", {split})
try:
    (B.bat_reliability_grad if {grad} else B.bat_reliability)(x.n, x.arcs, x.p, x.s, x.t)
except B.BatError as e:
    result = e.code
""", fail="finish")
        assert rc == -3
        sweeps = [o for o in ops if o.kind == "launch" and "finish" not in o.args[1]]
        assert len(sweeps) == 1 and not sweeps[0].failed, (m, split, sweeps)
        assert split or sum(int(o.args[1]) for o in ops if o.kind == "alloc") < 32 << 20


_ASYNC = """
import ctypes
rec = ctypes.CDLL(os.environ["HIP_RECORDER"])
x = W.random_connected(8, 14, seed=3)
buf = np.zeros(64)
at = buf.ctypes.data
stream = ctypes.c_void_p()
rec.hipStreamCreateWithFlags(ctypes.byref(stream), 0)
"""


def test_last_launch_waits_for_its_own_stream():
    """The report of an asynchronous launch is waited for on its stream, not
    on the device, which other streams may keep busy or be capturing.  (The
    recorder runs nothing, so there are no times.)"""
    times, ops = recorder.run(_ASYNC + """
B.bat_reliability_async(x.n, x.arcs, at, x.s, x.t, at + 256, at + 264, None, stream.value)
li = B.bat_last_launch()
result = [li.kernel_ms, li.total_ms, li.perm]
""")
    assert times == [0.0, 0.0, 5]
    launch = next(i for i, o in enumerate(ops) if o.kind == "launch")
    assert [o.kind for o in ops[launch + 1:] if o.kind != "launch"] == ["sync"]
    assert ops[-1].stream == ops[launch].stream != 0


@pytest.mark.parametrize("m", [8, 14, 30])
def test_noalloc_allocates_nothing_on_a_threads_first_call(m):
    """Neither device memory nor pinned host memory; the launch is reported
    through events then."""
    times, ops = recorder.run(_ASYNC + f"""
x = W.random_connected(max(6, {m} // 2), {m}, seed=3)
B.bat_reliability_noalloc(x.n, x.arcs, at, x.s, x.t, at + 256, at + 264, None, stream.value)
li = B.bat_last_launch()
result = [li.kernel_ms, li.perm]
""")
    assert times == [1.0, 5]
    assert [o.kind for o in ops].count("launch") >= 1 and not any(o.kind == "alloc" for o in ops)


@pytest.mark.parametrize("graphs", [512, 1100])
def test_batch_with_one_level_forced_is_launched(graphs):
    """Hundreds of graphs of 32 arcs with one level, 2^21 work items each:
    under 2^32 threads in a launch."""
    rc, ops = recorder.run(f"""
x = W.random_connected(12, 32, seed=8)
B.bat_set_option("BAT_CUBES", 1)
B.bat_set_option("BAT_CUBE_LEVELS", 1)
try:
    B.bat_reliability_batched([(x.n, x.arcs, x.s, x.t)] * {graphs}, [np.full((2, 32), 0.5)] * {graphs})
except B.BatError as e:
    result = e.code
""", fail="finish")
    sweeps = [o for o in ops if o.kind == "launch" and "finish" not in o.args[1]]
    assert rc == -3 and len(sweeps) == 2 and not any(o.failed for o in sweeps)


def test_workspace_of_a_large_batch():
    """1024 entries of 32 arcs and 32 vectors: the partials that the thread
    keeps stay within some tens of MiB."""
    rc, ops = recorder.run("""
x = W.random_connected(14, 32, seed=8)
try:
    B.bat_reliability_batched([(x.n, x.arcs, x.s, x.t)] * 32, [np.full((1024, 32), 0.5)] * 32)
except B.BatError as e:
    result = e.code
""", fail="finish")
    assert rc == -3 and not any(o.failed for o in ops if o.kind == "launch" and "finish" not in o.args[1])
    assert sum(int(o.args[1]) for o in ops if o.kind == "alloc" and o.args[0] == "device") < 48 << 20
