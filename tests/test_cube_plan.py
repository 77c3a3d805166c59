"""The sub-cube sweep's plan, checked on the CPU.

The closures the library hands to hiprtc (bat_jit_source, perm 5) are
straight-line steps that remove the nodes one by one.  These tests parse
them out of the source text and run them on bits, one vector at a time:
closure 0 must give the verdict of a breadth-first search for every vector,
and the closures of the higher levels the verdicts with the arcs below
their word all up and all down.  With those, replaying the sweep's levels
(cubes that connect for certain added whole, cubes that cannot dropped, the
rest split) must count exactly the connected vectors.  No GPU is needed.
"""
import re

import numpy as np
import pytest

import bat_workloads as W


def _B():
    import paper_2209_09711_amd as B
    return B


def _plan(net, directed, levels):
    B = _B()
    old = B.bat_get_option("BAT_CUBE_LEVELS")
    try:
        B.bat_set_option("BAT_CUBE_LEVELS", levels)
        src = B.bat_jit_source(net.n, net.arcs, net.s, net.t, perm=5, directed=directed)
    finally:
        B.bat_set_option("BAT_CUBE_LEVELS", old)
    g = src[src.index("struct JitCube"):]
    P = {k: int(re.search(r"static constexpr int %s = (\d+);" % k, g).group(1)) for k in ("M", "REL", "SLOTS")}
    P["LEVELS"] = int(re.search(r"LEVELS = (\d+)u", g).group(1))
    P["ARCS"] = [int(x) for x in re.search(r"counter bits 0, 1, \.\.\.:([ \d]*)\n", g).group(1).split()]
    P["RESULT"] = [int(x) for x in re.search(r"RESULT\[5\] = \{([^}]*)\}", g).group(1).replace("u", "").split(",")]
    P["STEPS"] = []
    for k in range(2 * P["LEVELS"] - 1):
        body = re.search(r"if constexpr \(K == %du\) \{\n(.*?)    \}\n" % k, g, re.S).group(1)
        steps = []
        for line in body.splitlines():
            m = re.match(r"\s*r\[(\d+)\] = r\[(\d+)\] & r\[(\d+)\];$", line)
            if m:
                steps.append((*map(int, m.groups()), False))
                continue
            m = re.match(r"\s*r\[(\d+)\] = and_or\(r\[(\d+)\], r\[(\d+)\], r\[(\d+)\]\);$", line)
            assert m and m.group(1) == m.group(4), line
            steps.append((*map(int, m.groups()[:3]), True))
        P["STEPS"].append(steps)
    assert len(P["ARCS"]) == P["M"] and len(set(P["ARCS"])) == P["M"]
    return P


def _closure(P, k, c):
    """Closure k on counter value c (Python ints as one-bit words)."""
    if P["RESULT"][k] >= 254:
        return P["RESULT"][k] == 255
    low = 5 * ((k + 1) // 2)
    r = [0] * P["SLOTS"]
    for b in range(P["M"]):
        r[b] = (k & 1) if b < low else (c >> b) & 1
    for d, a, b, acc in P["STEPS"][k]:
        x = r[a] & r[b]
        r[d] = r[d] | x if acc else x
    return bool(r[P["RESULT"][k]])


def _bfs(net, up, directed):
    adj = [[] for _ in range(net.n)]
    for i, (a, b) in enumerate(net.arcs):
        if up[i]:
            adj[a].append(b)
            if not directed:
                adj[b].append(a)
    seen, todo = {net.s}, [net.s]
    for x in todo:
        for y in adj[x]:
            if y not in seen:
                seen.add(y)
                todo.append(y)
    return net.t in seen


def _cases():
    out = [("bridge", W.bridge(), False), ("parallel", W.parallel(3, [0.5] * 3), False),
           ("apart", W.Network("apart", 4, [(0, 1), (2, 3)], 0, 3, np.full(2, 0.5)), False),
           ("grid3x4", W.grid(3, 4), False), ("series", W.series(6, np.full(6, 0.9)), False)]
    for seed, (n, m) in enumerate([(6, 11), (8, 15), (9, 16), (7, 17)]):
        out.append((f"rand{m}", W.random_connected(n, m, seed=300 + seed), False))
    out.append(("multi", W.random_multigraph(6, 13, seed=31), False))
    for seed in range(2):
        rng = np.random.default_rng(seed)
        arcs = [tuple(int(x) for x in rng.choice(7, 2, replace=False)) for _ in range(13)]
        out.append((f"di{seed}", W.Network(f"di{seed}", 7, arcs, 0, 6, np.full(13, 0.9)), True))
    return out


@pytest.mark.parametrize("levels", [1, 2, 3])
@pytest.mark.parametrize("name,net,directed", _cases(), ids=[c[0] for c in _cases()])
def test_cube_closures(name, net, directed, levels):
    P = _plan(net, directed, levels)
    M, rng = P["M"], np.random.default_rng(7)
    assert P["LEVELS"] == max(1, min(levels, M // 5))
    for c in ([int(x) for x in rng.integers(0, 1 << M, size=120)] if M > 7 else range(1 << M)):
        for k in range(2 * P["LEVELS"] - 1):
            low = 5 * ((k + 1) // 2)
            v = (c | ((1 << low) - 1)) if k & 1 else c >> low << low
            up = [False] * len(net.arcs)
            for b in range(M):
                up[P["ARCS"][b]] = bool((v >> b) & 1)
            assert _closure(P, k, c) == _bfs(net, up, directed), (name, k, c)


@pytest.mark.parametrize("levels", [2, 3])
@pytest.mark.parametrize("name,net,directed", [c for c in _cases() if 10 <= len(c[1].arcs) <= 16],
                         ids=[c[0] for c in _cases() if 10 <= len(c[1].arcs) <= 16])
def test_cube_levels_count_every_vector_once(name, net, directed, levels):
    import oracle
    P = _plan(net, directed, levels)

    def count(level, c):
        """Connected vectors under prefix c of a level's word."""
        total = 0
        for j in range(min(32, 1 << P["M"])):  # (the kernel masks bits past the last arc)
            v = c | j << (5 * level)
            if level == 0:
                total += _closure(P, 0, v)
            elif _closure(P, 2 * level, v):
                total += 1 << (5 * level)
            elif _closure(P, 2 * level - 1, v):
                total += count(level - 1, v)
        return total
    top = 5 * P["LEVELS"]
    got = sum(count(P["LEVELS"] - 1, x << top) for x in range(1 << max(0, P["M"] - top)))
    o = oracle.reliability(net.n, net.arcs, net.p, net.s, net.t, directed=directed)
    assert got << (len(net.arcs) - P["M"]) == o.count


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("name,net,directed,levels",
                         [("grid5x5", W.grid(5, 5), False, 3), ("rand12", W.random_connected(8, 12, 1), False, 2),
                          ("rand62", W.random_connected(30, 62, 4), False, 3), ("di0", *_cases()[-2][1:], 1)],
                         ids=["grid5x5", "rand12", "rand62", "di0"])
def test_cube_source_compiles(tmp_path, name, net, directed, levels, grad):
    """The specialised kernels through the hiprtc that the library loads (it
    ends the process where it cannot place a value in a scalar register)."""
    import subprocess
    B = _B()
    rtc = [x.split()[-1] for x in open("/proc/self/maps") if "libhiprtc.so" in x]
    if not rtc:
        pytest.skip("no hiprtc library loaded")
    old = B.bat_get_option("BAT_CUBE_LEVELS")
    try:
        B.bat_set_option("BAT_CUBE_LEVELS", levels)
        src = B.bat_jit_source(net.n, net.arcs, net.s, net.t, grad=grad, perm=5, directed=directed)
    finally:
        B.bat_set_option("BAT_CUBE_LEVELS", old)
    text, out = tmp_path / "k.hip.txt", tmp_path / "k.co"
    text.write_text(src)
    import os
    helper = os.path.join(os.path.dirname(B.__file__), "bat_jitc")
    subprocess.run([helper, rtc[0], str(text), str(out), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops"], check=True, capture_output=True)
    assert out.stat().st_size > 0
