"""The padded lengths between the powers of two: every one with n = L / 2, and
with an n that leaves a zero gap, against the product by torch's FFTs in 64
bits; partial last workgroups and idle lanes included (odd n, batches)."""
import math
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1602_04691_amd as ori  # noqa: E402
import workloads  # noqa: E402

LENGTHS = (72, 100, 108, 144, 160, 200, 216, 288, 320, 360, 400, 432, 576, 640, 720, 768)


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def green_product(n, k, side, x):
    # y = G0 x by a (2n)^3 cyclic convolution in complex128
    L = 2 * n
    d = torch.arange(L, dtype=torch.float64, device="cuda")
    d = torch.minimum(d, L - d) * (side / n)
    r = (d[:, None, None] ** 2 + d[None, :, None] ** 2 + d[None, None, :] ** 2).sqrt()
    r[0, 0, 0] = 1.0
    g = torch.polar(1.0 / (4 * math.pi * r), k * r)
    g[0, 0, 0] = 0.0
    f = torch.fft.fftn(x.view(n, n, n), s=(L, L, L)) * torch.fft.fftn(g)
    return torch.fft.ifftn(f)[:n, :n, :n].reshape(-1)


@pytest.mark.parametrize("L", LENGTHS)
@pytest.mark.parametrize("gap", [0, 1])
def test_product_at_every_length_between(L, gap):
    n = L // 2 - gap
    k, side = 4.3, 1.1
    say(f"[lengths] L={L} n={n}")
    P = n ** 3
    g = torch.Generator(device="cuda").manual_seed(7 * L + gap)
    x = torch.randn(P, dtype=torch.complex128, device="cuda", generator=g)
    one = torch.ones(P, dtype=torch.complex128, device="cuda")
    ref = green_product(n, k, side, x)
    with ori.ori_create(n, side=side) as ctx:
        ori.ori_load(ctx, k, one, None, x)
        y = torch.empty_like(x)
        # complex128: a few ulps times log2 L per transform, as the parity
        # tests; complex64: 6e-8 times the stages
        for prec, bar in ((ori.ORI_FP64, 1e-14), (ori.ORI_MIXED, 1e-6)):
            base = ori.ori_get_layout(ctx, prec)
            for lay in (base, dict(base, narrow=1, znarrow=1 - base["znarrow"]), dict(base, blk_lg=0, prefetch=1)):
                ori.ori_set_layout(ctx, prec, **lay)
                y.fill_(complex("nan"))
                ori.ori_matvec(ctx, x, y, op=ori.ORI_OP_GREEN, precision=prec)
                e = ((y - ref).norm() / ref.norm()).item()
                w = ((y - ref).abs().max() / ref.abs().max()).item()
                say(f"   precision {prec} {lay}: {e:.2e} (largest {w:.2e})")
                assert e <= bar and w <= 4 * bar
        assert ori.ori_check_guards(ctx) == 0


def test_blocks_beyond_the_per_lane_addressing():
    # n = 320 (L = 640): i1 blocks of 2^6 rows, more than the 2^4 that divide
    # the element distances, take the 64-bit addressing: bitwise the default's
    n, k = 320, 3.0
    say("[lengths] n=320 blk_lg=6")
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(n ** 3, dtype=torch.complex128, device="cuda", generator=g)
    one = torch.ones_like(x)
    with ori.ori_create(n) as ctx:
        ori.ori_load(ctx, k, one, None, x)
        for prec in (ori.ORI_FP64, ori.ORI_MIXED):
            ys = []
            for lg in (ori.ori_get_layout(ctx, prec)["blk_lg"], 6):
                ori.ori_set_layout(ctx, prec, **dict(ori.ori_get_layout(ctx, prec), blk_lg=lg))
                y = torch.empty_like(x)
                ori.ori_matvec(ctx, x, y, op=ori.ORI_OP_GREEN, precision=prec)
                ys.append(y)
            assert torch.equal(*ys)


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_and_group_at_the_lengths_between(prec):
    # a batch equals its single solves and a group its own, bit for bit, at
    # lengths with idle lanes (n = 36: L = 72, 288 of 320 threads) and without
    k, R = 3.0, 3
    say(f"[lengths] batch n=36 x3, group (33, 36, 50, 54, 70), precision {prec}")
    c = workloads.make_case(36, k, seed=11)
    u0 = np.concatenate([workloads.plane_wave(36, k, d) for d in workloads.fibonacci_directions(R)])
    with ori.ori_create(36, nrhs=R) as ctx:
        ori.ori_load(ctx, k, gpu(c["h"]), gpu(c["N"]), gpu(u0))
        u = torch.empty(R * 36 ** 3, dtype=torch.complex128, device="cuda")
        ori.ori_solve(ctx, u, tol=1e-10, precision=prec)
    for i in range(R):
        one, _ = ori.solve(36, k, gpu(c["h"]), gpu(c["N"]), gpu(u0[i * 36 ** 3:(i + 1) * 36 ** 3]), tol=1e-10,
                           precision=prec)
        assert torch.equal(u[i * 36 ** 3:(i + 1) * 36 ** 3], one)
    ns = (33, 36, 50, 54, 70)
    cases = [workloads.make_case(n, k, seed=60 + n) for n in ns]
    res = ori.solve_many([dict(n=n, k=k, h=gpu(c["h"]), N=gpu(c["N"]), u0=gpu(c["u0"])) for n, c in zip(ns, cases)],
                         tol=1e-10, precision=prec)
    for n, c, (u, info) in zip(ns, cases, res):
        one, _ = ori.solve(n, k, gpu(c["h"]), gpu(c["N"]), gpu(c["u0"]), tol=1e-10, precision=prec)
        assert torch.equal(u, one), n
        assert info["rel_res_true"] <= 2e-10
