"""The host runs a block of iterations ahead of its checks: the scalars that it
reads for a block are those of the block's last iteration, whatever the next
block is doing meanwhile.  Every report (status, iterations, products, residual
of the recursion) and every bit of the result equal those of a run that waits
for each block before it launches the next one."""
import sys

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1602_04691_amd as ori  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


KEYS = ("iterations", "refinements", "matvecs", "matvecs_c64", "rel_res_recursive", "rel_res_true")


def report(info):
    return [info[k] for k in KEYS]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,R", [(16, 1), (12, 3), (48, 1)])
@pytest.mark.parametrize("every", [1, 2, 3])
def test_blocks_report_what_a_waiting_run_reports(n, R, every, prec, monkeypatch):
    k = 5.0
    say(f"[ahead] n={n} nrhs={R} check_every={every} precision={prec}")
    c = workloads.make_case(n, k, seed=31)
    u0 = np.concatenate([workloads.plane_wave(n, k, d) for d in workloads.fibonacci_directions(R)])
    ctx = {}
    try:
        for wait in (True, False):
            if wait:  # with the checks of the guard bands every block is waited for
                monkeypatch.setenv("ORI_CHECK_GUARDS", "1")
            else:
                monkeypatch.delenv("ORI_CHECK_GUARDS")
            ctx[wait] = ori.ori_create(n, nrhs=R)
            ori.ori_load(ctx[wait], k, gpu(c["h"]), gpu(c["N"]), gpu(u0))
        for max_iter in [*range(1, 3 * every + 3), 1000]:
            out = {}
            for wait in (True, False):
                u = torch.full((R * n ** 3,), complex("nan"), dtype=torch.complex128, device="cuda")
                st, info = ori.ori_solve(ctx[wait], u, tol=1e-11, max_iter=max_iter, precision=prec,
                                         check_every=every, raise_on_error=False)
                out[wait] = (st, report(info), [report(ori.ori_batch_info(ctx[wait], i)) for i in range(R)], u)
            assert out[True][:3] == out[False][:3], max_iter
            assert torch.equal(out[True][3], out[False][3]), max_iter
        assert st == ori.ORI_OK
    finally:
        for x in ctx.values():
            ori.ori_destroy(x)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("every", [1, 2, 3])
def test_group_blocks_report_what_a_waiting_run_reports(every, prec):
    # members that leave in different blocks
    ns, ks = (5, 9, 20, 33), (1.0, 3.0, 5.0, 2.0)
    say(f"[ahead, group] n in {ns} check_every={every} precision={prec}")
    cases = [workloads.make_case(n, k, seed=60 + n) for n, k in zip(ns, ks)]
    with ori.ori_group_create(ns) as g:
        ori.ori_group_load_all(g, ks, [gpu(c["h"]) for c in cases], [gpu(c["N"]) for c in cases],
                               [gpu(c["u0"]) for c in cases])
        out = []
        for multi in (False, True):  # plain launches of each problem: every block is waited for
            us = [torch.empty(n ** 3, dtype=torch.complex128, device="cuda") for n in ns]
            _, infos = ori.ori_group_solve(g, us, tol=1e-10, precision=prec, multi=multi, graph=False,
                                           check_every=every)
            out.append((us, [report(i) for i in infos]))
        assert out[0][1] == out[1][1]
        assert all(torch.equal(a, b) for a, b in zip(out[0][0], out[1][0]))


@pytest.mark.parametrize("every", [2, 4])
def test_blocks_cut_short_by_one_members_budget(every):
    # in mixed precision the members' inner iterations differ from the second
    # cycle on, so a max_iter in between leaves them different budgets: the
    # block in which the smaller one ends is short, and the others go on with
    # full blocks whose scalars the host finds all the same
    ns, ks = (9, 20, 33), (1.0, 5.0, 8.0)
    say(f"[ahead, budgets] n in {ns} check_every={every}")
    cases = [workloads.make_case(n, k, seed=60 + n) for n, k in zip(ns, ks)]
    uneven = 0
    with ori.ori_group_create(ns) as g:
        ori.ori_group_load_all(g, ks, [gpu(c["h"]) for c in cases], [gpu(c["N"]) for c in cases],
                               [gpu(c["u0"]) for c in cases])
        for max_iter in range(5, 41):
            out = []
            for multi in (False, True):
                us = [torch.empty(n ** 3, dtype=torch.complex128, device="cuda") for n in ns]
                st, infos = ori.ori_group_solve(g, us, tol=1e-13, precision=1, inner_tol=1e-4, max_iter=max_iter,
                                                multi=multi, graph=False, check_every=every, raise_on_error=False)
                out.append((st, [report(i) for i in infos], us))
            assert out[0][:2] == out[1][:2], max_iter
            assert all(torch.equal(a, b) for a, b in zip(out[0][2], out[1][2])), max_iter
            uneven += len({i["iterations"] for i in infos}) > 1 and st != ori.ORI_OK
    say(f"   {uneven} of 36 runs ended with uneven iterations")
    assert uneven >= 3
