"""HIP-graph replay of a group's COCG iteration blocks (problems that launch
kernels of their own) against plain launches.

A graph holds the same kernels with the same arguments as the plain
iterations, so every replay must give the plain iterate bit for bit.  Replays
are interleaved with the library's own eager work (scalar reads, recovery,
true residual) and with reloads of new data into the same group.  Each test
also asserts that replays took place: a single context launches plainly.
"""
import os
import random
import sys
import threading

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1602_04691_amd as ori  # noqa: E402

REPLAYS = os.environ.get("ORI_CHECK_GUARDS", "0") in ("", "0")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def load(g, ns, k, seed):
    cases = [workloads.make_case(n, k, seed=seed + n) for n in ns]
    ori.ori_group_load_all(g, [k] * len(ns), [gpu(c["h"]) for c in cases], [gpu(c["N"]) for c in cases],
                           [gpu(c["u0"]) for c in cases])


def solve(g, ns, graph, **opts):
    us = [torch.full((n ** 3,), complex("nan"), dtype=torch.complex128, device="cuda") for n in ns]
    before = ori.ori_group_graph_iterations(g)
    st, infos = ori.ori_group_solve(g, us, multi=False, graph=graph, raise_on_error=False, **opts)
    keys = ("iterations", "matvecs", "matvecs_c64", "refinements", "rel_res_recursive", "rel_res_true")
    return st, [[i[k] for k in keys] for i in infos], us, ori.ori_group_graph_iterations(g) - before


def same(a, b):
    return a[:2] == b[:2] and all(torch.equal(x, y) for x, y in zip(a[2], b[2]))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("every", [1, 3])
def test_every_replay_count_equals_plain_launches(precision, every):
    ns, k = (8, 12, 16, 48), 5.0
    say(f"[group graph] n in {ns} precision={precision} check_every={every}")
    with ori.ori_group_create(ns) as g:
        for seed in (31, 32):  # the cached graphs serve the reloaded data too
            load(g, ns, k, seed)
            for max_iter in [*range(1, 4 * every + 2), 1000]:
                opts = dict(tol=1e-10, max_iter=max_iter, precision=precision, check_every=every)
                plain, replay = solve(g, ns, False, **opts), solve(g, ns, True, **opts)
                assert same(plain, replay), max_iter
                assert plain[3] == 0 and (replay[3] > 0) == (max_iter >= every and REPLAYS)
            assert plain[0] == ori.ORI_OK
            say(f"   {replay[3]} iterations in replays")


def test_replays_of_concurrent_groups():
    # groups driven from four threads at once (each its own streams), each
    # building and replaying its own graphs, while a fifth thread allocates and
    # frees device memory through torch: every result equals the one of plain
    # launches in one thread, bit for bit, over three rounds
    sets = [(12, 16), (20, 9), (24, 11, 6), (18, 18)]
    say(f"[group graph, threads] {sets}")
    ref = []
    for j, ns in enumerate(sets):
        with ori.ori_group_create(ns) as g:
            load(g, ns, 4.0, 90 + j)
            ref.append(solve(g, ns, False, tol=1e-10))
    torch.cuda.synchronize()
    stop, errors = threading.Event(), []

    def churn():
        rng = random.Random(5)
        while not stop.is_set():
            t = torch.empty(rng.randint(1, 64) << 18, dtype=torch.float32, device="cuda")
            t.fill_(1.0)
            del t
            torch.cuda.empty_cache()

    def worker(j, ns):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s), ori.ori_group_create(ns) as g:
                load(g, ns, 4.0, 90 + j)
                got = solve(g, ns, True, tol=1e-10)
            s.synchronize()
            if not same(ref[j], got) or (got[3] > 0) != REPLAYS:
                errors.append((ns, got[3]))
        except BaseException as e:  # reported below
            errors.append((ns, repr(e)))

    th = threading.Thread(target=churn)
    th.start()
    try:
        for _ in range(3):
            ws = [threading.Thread(target=worker, args=a) for a in enumerate(sets)]
            for w in ws:
                w.start()
            for w in ws:
                w.join()
    finally:
        stop.set()
        th.join()
    assert not errors, errors
