"""F2, Z and I2 in one launch (small problems) against the three passes: the
same bits, at the smallest and largest planes, lengths with idle lanes and a
zero gap, odd batches, and at the line where the passes take over."""
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1602_04691_amd as ori  # noqa: E402
import workloads  # noqa: E402
import oracle as O  # noqa: E402
import numpy as np  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


# padded lengths 10 (the smallest with two stages), 12, 16, 20, 24, 32, 40, 48,
# 64, 72, 80 (the largest); 4 * 64 planes are the most one launch takes, 5 * 64
# go to the passes
@pytest.mark.parametrize("n,R", [(4, 1), (5, 1), (6, 3), (7, 1), (9, 5), (12, 1), (13, 1), (17, 2), (24, 1), (25, 4),
                                 (32, 4), (32, 5), (33, 1), (36, 3), (37, 1), (40, 3), (41, 1)])
@pytest.mark.parametrize("prec", [0, 1])
def test_plane_equals_the_passes(n, R, prec):
    k = 3.7
    say(f"[plane] n={n} nrhs={R} precision={prec}")
    c = workloads.make_case(n, k, seed=400 + n)
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(R * n ** 3, dtype=torch.complex128, device="cuda", generator=g)
    h, N = torch.from_numpy(c["h"]).cuda(), torch.from_numpy(c["N"]).cuda()
    with ori.ori_create(n, nrhs=R) as ctx:
        ori.ori_load(ctx, k, h, N, x)
        out = []
        for nar in (0, 1):  # narrow strided tiles: always the three passes
            ori.ori_set_layout(ctx, prec, **dict(ori.ori_get_layout(ctx, prec), narrow=nar))
            y = torch.full_like(x, complex("nan"))
            ori.ori_matvec(ctx, x, y, op=ori.ORI_OP_SYMMETRIC, precision=prec)
            u = torch.full_like(x, complex("nan"))
            _, info = ori.ori_solve(ctx, u, tol=1e-11, precision=prec)
            out.append((y, u, info["iterations"]))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
        assert out[0][2] == out[1][2]
        assert ori.ori_check_guards(ctx) == 0
    if n <= 9:  # and against the dense sums
        D = O.coupling(c["h"], c["N"], n)
        S = np.sqrt(D.astype(complex))
        x0 = x[: n ** 3].cpu().numpy()
        ref = x0 + S * O.scatter_dense(O.cell_points(n), k, np.ones(n ** 3), S * x0)
        d = np.linalg.norm(out[0][0][: n ** 3].cpu().numpy() - ref) / np.linalg.norm(ref)
        assert d <= (1e-12 if prec == 0 else 2e-6)
