"""The kernel of uni-greedy schedules of up to 1024 processors, compiled from its own source for the CPU and run on emulated
wavefronts (tests/wavefront): its reads and writes of LDS stay inside the allocation and see only what has been written, and
a byte is used as one type unless it may alias another; pairs and start times are the oracle's; lists that are broken on purpose end with a status."""
from __future__ import annotations

import ctypes as C
import os
import subprocess

import numpy as np
import pytest

import oracle as O
import prs_inputs
from paper_1310_4645_amd import binding as B

STALLED = 3                                          # PRS_CFG_STALLED
HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "wavefront", "uni_list.cpp")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    llvm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    out = str(tmp_path_factory.mktemp("emu") / "libemu.so")
    subprocess.check_call([llvm, "-x", "c++", "-std=c++17", "-O0", "-fno-omit-frame-pointer", "-ffp-contract=off", "-fPIC", "-shared", "-w",
                           "-I", os.path.join(HERE, "wavefront"), SRC, "-o", out])
    lib = C.CDLL(out)
    lib.emu_waits.restype = C.c_int64
    lib.emu_first_fault.restype = C.c_char_p
    lib.prs_workspace_bytes.restype = C.c_size_t
    return lib


def _ptr(a):
    return None if a is None else a.ctypes.data


def _run(lib, host, p_max, q_max, gaps, limit=2_000_000, backwards=False, types=True, poke=(0, 0, 0, 2)):
    """greedy_schedule_batch on the emulated wavefronts; outputs with a margin around every configuration."""
    n, cost = len(host), B.PRS_COST_I64 if host.cost == "i64" else B.PRS_COST_F64
    number = np.int64 if host.cost == "i64" else np.float64
    pairs = np.array([(int(host.p[i]) - 1) * len(O.equi_sizes(int(host.m[i]), int(host.q_req[i]))) for i in range(n)])
    start = np.cumsum(np.concatenate([[3], pairs[:-1] + gaps[:n - 1]])).astype(np.int64)
    total = int(start[-1] + pairs[-1] + 9)
    arrays = [np.ascontiguousarray(a) for a in (host.p.astype(np.int32), host.q_req.astype(np.int32), host.m.astype(np.int64),
                                                host.alpha.astype(number), host.beta.astype(number), host.gamma.astype(number))]
    cfg = B._Configs(*[_ptr(a) for a in arrays])
    off = np.append(start, total)
    out = [np.full(total, -7, np.int32) for _ in range(3)] + [np.full(total, -7, number)]
    T, status = np.zeros(n, number), np.full(n, -9, np.int32)
    size = lib.prs_workspace_bytes(B.PRS_CALL_SCHEDULE, B.PRS_UNI, cost, C.c_int64(n), p_max, q_max)
    ws = np.zeros(size + 256, np.uint8)
    base = (_ptr(ws) + 255) // 256 * 256
    lib.emu_begin(int(types), C.c_int64(limit), int(backwards), *[C.c_int64(int(v)) for v in poke])
    rc = lib.greedy_schedule_batch(C.byref(cfg), C.c_int64(n), B.PRS_UNI, cost, p_max, q_max, C.c_void_p(_ptr(off)), C.c_int64(total),
                                   *[C.c_void_p(_ptr(a)) for a in out], C.c_void_p(_ptr(T)), C.c_void_p(_ptr(status)), C.c_void_p(base),
                                   C.c_size_t(size), None, None)
    assert rc == 0
    return start, pairs, out, T, status


def _check(lib, host, p_max, q_max, seed, **more):
    gaps = np.random.default_rng(seed).integers(0, 4, len(host))
    start, pairs, out, T, status = _run(lib, host, p_max, q_max, gaps, **more)
    assert lib.emu_faults() == 0, lib.emu_first_fault().decode()
    assert not lib.emu_stopped() and np.all(status == 0)
    want = [np.full_like(a, -7) for a in out]
    for i in range(len(host)):
        r = O.uni_greedy(int(host.p[i]), O.equi_sizes(int(host.m[i]), int(host.q_req[i])), host.alpha[i].item(), host.beta[i].item(),
                         host.gamma[i].item(), host.cost)
        for w, v in zip(want, (r.src, r.dst, r.seg, r.t)):
            w[start[i]:start[i] + pairs[i]] = v
        assert T[i] == r.T
    for got, w in zip(out, want):
        assert np.array_equal(got, w)


def _machines(p, q, cost, seed):
    rng = np.random.default_rng(seed)
    p, q = np.array(p, np.int32), np.array(q, np.int32)
    n = len(p)
    m = (q.astype(np.int64) * 3 - rng.integers(0, 2, n) * (q > 1))
    if cost == "i64":
        costs = [rng.choice([1, 2, 10], n), rng.integers(0, 3, n), rng.integers(0, 3, n)]
    else:
        costs = [rng.choice([0.1, 1e-5, 0.3], n), rng.choice([0.1, 1e-6, 0.0], n), rng.choice([0.0, 1e-20, 0.1, 3e-6], n)]
    number = np.int64 if cost == "i64" else np.float64
    return prs_inputs.SweepConfigs(p, q, m, *[c.astype(number) for c in costs], cost)


# bound on the machines, then processors and segments: every group size, groups without a configuration, the largest machines,
# one segment, more segments than lanes
_BATCHES = {"one machine": (1024, [5], [3]),
            "one of one segment": (64, [64], [1]),
            "few": (256, [2, 3, 17, 33, 65, 129, 256], [9, 1, 40, 3, 2, 5, 34]),
            "large": (1024, [961, 3], [17, 1]),
            "pairs only": (16, [2] * 70, list(range(1, 71)))}


@pytest.mark.parametrize("cost", ["i64", "f64"])
@pytest.mark.parametrize("batch", list(_BATCHES))
def test_lists_stay_inside_lds_and_give_the_oracles_pairs(emu, batch, cost):
    p_max, p, q = _BATCHES[batch]
    _check(emu, _machines(p, q, cost, 5), p_max, max(q), 7, backwards=cost == "f64")


@pytest.mark.parametrize("share", [0.02, 0.3, 0.7, 2.0])
def test_machines_begun_beside_large_ones(emu, share):
    """Wavefronts of the launch of large machines take small ones as long as a large one is not done, the launch that follows the rest:
    none is left out or run twice, whenever that is."""
    p, q = [2, 300, 17, 33, 1000, 65, 129, 256, 40, 5] * 2, [9, 1, 40, 3, 2, 5, 34, 2, 17, 1] * 2
    host = _machines(p, q, "i64", 5)
    try:
        emu.emu_help(C.c_int64(1 << 40))
        _check(emu, host, 1100, 40, 7)
        emu.emu_help(C.c_int64(max(1, int(share * emu.emu_waits()))))
        _check(emu, host, 1100, 40, 7)
    finally:
        emu.emu_help(C.c_int64(0))


def test_broken_lists_end_with_a_status(emu):
    """A link of the one machine names another of its processors all of a sudden, or a ready time becomes infinite, at any time: the
    kernel comes to an end, inside its LDS, and says so if a list was out of order or no pair could be formed any more."""
    host = _machines([40], [30], "f64", 3)
    gaps = np.zeros(1, np.int64)
    _run(emu, host, 1024, 30, gaps)
    waits = emu.emu_waits()
    times = 64 * 30 * 2                                          # where the ready times begin: behind the links, 30 processors a lane
    rng = np.random.default_rng(11)
    seen = set()
    for k in range(60):
        when, i, to = rng.integers(waits // 10, waits - waits // 10), rng.integers(0, 40), rng.integers(0, 40)
        word = (2 * (to if k % 3 == 0 else i), 2 * to, 2) if k % 4 else (times + 8 * i, 0x7FF0000000000000, 8)
        *_, T, status = _run(emu, host, 1024, 30, gaps, limit=4 * waits, poke=(when, *word))
        assert not emu.emu_stopped(), k
        assert emu.emu_faults() == 0, emu.emu_first_fault().decode()
        assert status[0] in (0, STALLED)
        seen.add((int(status[0]), bool(np.isnan(T[0]))))
    assert (STALLED, True) in seen and (STALLED, False) in seen        # given up, and marked on the way
