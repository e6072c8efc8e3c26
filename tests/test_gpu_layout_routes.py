"""Layout knobs that select no kernel decide no route: the tuner does not
choose by them, and a group runs in common launches whatever their value."""
import os
import sys

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1602_04691_amd as ori  # noqa: E402


MULTI_LAUNCHES = os.environ.get("ORI_CHECK_GUARDS", "0") in ("", "0")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [34, 38, 52, 98])
def test_tuner_leaves_idle_knobs_alone(n):
    # padded lengths 72 and 80 (planes: neither blocks nor Z tiles to choose),
    # 108 and 200 (no prefetch variant, no second Z plan).  Sizes that no other
    # test uses: the process keeps what the tuner picks
    say(f"[tune] n={n}")
    c = workloads.make_case(n, 3.0, seed=5)
    with ori.ori_create(n) as ctx:
        ori.ori_load(ctx, 3.0, gpu(c["h"]), gpu(c["N"]), gpu(c["u0"]))
        start = [ori.ori_get_layout(ctx, p) for p in (0, 1)]
        res = ori.ori_tune(ctx, reps=1)
    for (lay, ms), s in zip((res["fp64"], res["c64"]), start):
        say(f"   {lay} {ms}")
        assert ms > 0
        if n != 38:
            assert lay["prefetch"] == 0 and lay["zplan"] == 0
        if n <= 40 and lay["narrow"] == lay["prefetch"] == lay["zplan"] == 0:
            assert lay == s


@pytest.mark.parametrize("ns,env", [((33, 50), "ZPF"), ((12, 24), "ZNP"), ((12, 24), "BLK_LG"), ((48, 96), "BLK_LG")])
@pytest.mark.parametrize("prec", [0, 1])
def test_group_in_common_launches_whatever_the_idle_knobs(ns, env, prec, monkeypatch):
    # n = 48, 96 in blocks of 2^4 rows: beyond the Z pass's per-lane
    # addressing at L = 96, so the common launches take smaller blocks
    k = 3.0
    cases = [workloads.make_case(n, k, seed=60 + n) for n in ns]
    out = []
    for value in (None, "4" if env == "BLK_LG" else "0", "1"):
        if value is not None:
            monkeypatch.setenv("ORI_TUNE_" + env, value)
        with ori.ori_group_create(ns) as g:
            ori.ori_group_load_all(g, [k, k], [gpu(c["h"]) for c in cases], [gpu(c["N"]) for c in cases],
                                   [gpu(c["u0"]) for c in cases])
            us = [torch.empty(n ** 3, dtype=torch.complex128, device="cuda") for n in ns]
            ori.ori_group_solve(g, us, tol=1e-10, precision=prec)
            ran = ori.ori_group_multi_iterations(g)
        say(f"[routes] n={ns} precision={prec} {env}={value}: {ran} iterations in common launches")
        assert (ran > 0) == MULTI_LAUNCHES
        out.append(us)
    for us in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(us, out[0]))
