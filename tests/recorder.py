"""Runs the library in a process of its own on a HIP runtime that only writes
down what is asked of it (hip_recorder.cpp), so that the order of copies,
launches and waits, launch shapes and error paths can be checked without a
GPU.
"""
import json
import os
import subprocess
import sys
import tempfile
from dataclasses import dataclass, field

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
_lib = None

_PRELUDE = """
import ctypes, json, os, sys
ctypes.CDLL(os.environ["HIP_RECORDER"], ctypes.RTLD_GLOBAL)
sys.modules["torch"] = None  # (it would bring a runtime of its own)
sys.path.insert(0, %r)
import numpy as np
import paper_2209_09711_amd as B
import bat_workloads as W
""" % ROOT


@dataclass
class Op:
    kind: str            # copy, launch, record, wait, sync, alloc, device-sync, event-sync
    args: list
    failed: bool
    stream: int = 0      # of copy, launch, record, wait, sync
    after: set = field(default_factory=set)  # earlier operations that are done before it


def library():
    global _lib
    if _lib is None:
        out = os.path.join(tempfile.mkdtemp(prefix="hip_recorder"), "librecorder.so")
        rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", f"-I{rocm}/include",
                        os.path.join(HERE, "hip_recorder.cpp"), "-o", out], check=True, capture_output=True)
        _lib = out
    return _lib


def run(code, fail="", env=()):
    """Run `code` (B, W and np at hand) on the recorder.  `fail`: see
    hip_recorder.cpp.  Returns (what the code left in `result`, the log)."""
    with tempfile.TemporaryDirectory() as d:
        log = os.path.join(d, "log")
        text = _PRELUDE + "result = None\n" + code + "\nprint('\\n' + json.dumps(result))\n"
        p = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=300, cwd=d,
                           env={**os.environ, "HIP_RECORDER": library(), "HIP_RECORDER_LOG": log,
                                "HIP_RECORDER_FAIL": fail, "BAT_JIT_CACHE": "0", **dict(env)})
        assert p.returncode == 0, p.stderr[-2000:]
        lines = open(log).read().splitlines() if os.path.exists(log) else []
    return json.loads(p.stdout.splitlines()[-1]), _ordered([_op(x) for x in lines])


def _op(line):
    w = line.split()
    failed = w[-1] == "failed"
    args = w[1:-1] if failed else w[1:]
    op = Op(w[0], args, failed)
    if op.kind in ("copy", "launch", "wait", "sync"):
        op.stream = int(args[0])
    elif op.kind == "record":
        op.stream = int(args[1])
    return op


def _ordered(ops):
    """Fill in each operation's `after` from streams, events and waits of
    the host."""
    done = set()                 # the host has waited for these
    tail, event = {}, {}         # per stream / event: what is done when it is reached
    for i, op in enumerate(ops):
        if op.failed:
            continue
        if op.kind == "sync":
            done |= tail.get(op.stream, set())
        elif op.kind == "device-sync":
            for t in tail.values():
                done |= t
        elif op.kind == "event-sync":
            done |= event.get(int(op.args[0]), set())
        elif op.kind in ("copy", "launch", "record", "wait"):
            before = tail.get(op.stream, set()) | done
            if op.kind == "wait":
                before = before | event.get(int(op.args[1]), set())
            op.after = before
            tail[op.stream] = before | {i}
            if op.kind == "record":
                event[int(op.args[0])] = before | {i}
    return ops
