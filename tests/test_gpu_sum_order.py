"""GPU: the place of the bias in the sums of the bf16 route kernels, which decides
how a hidden activation rounds: added to the finished sum by shapes without a
persistent kernel, the first term of the sum in shapes with one (both there and
in the feature-split kernel, whose logits are then the same).

Every layer is x -> 2^24 + x[0] - 2^24 x[16], and x[0] = x[16] = 1 at its input.
The products lie in different K blocks, so with the bias last it gives exactly 1,
while 2^24 + 1 is no fp32 number: with the bias first the 1 is lost. The expected
logits follow by the same fp32 additions."""
import numpy as np
import pytest

import workload
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

BIG = np.float32(2.0 ** 24)
# hidden, layers, M, K, embedding width, value head, rows, grids (they pick 32, 64 or 128 rows a block), bias last
SHAPES = [
    (32, 2, 5, 3, 64, False, 100, (256, 2, 1), True),
    (64, 3, 5, 3, 30, True, 100, (256, 2, 1), True),
    (64, 2, 16, 4, 64, True, 100, (256, 2, 1), True),
    (128, 3, 8, 3, 64, False, 100, (256, 2, 1, 0), True),
    (256, 3, 5, 3, 384, False, 200, (256, 4, 1, 0), True),
    (256, 3, 15, 3, 64, False, 200, (256, 4, 1), True),    # two output tiles
    (256, 2, 5, 3, 64, False, 200, (256, 4, 1), True),     # one K block less than the persistent two-layer shape
    (512, 3, 5, 3, 128, False, 200, (256, 4, 1), True),
    (512, 2, 16, 4, 128, False, 200, (256, 4, 1), True),
    (256, 3, 5, 3, 64, False, 500, (256, 8, 1, 0), False),
    (256, 2, 8, 3, 64, True, 500, (256, 8, 1, 0), False),
    (512, 3, 16, 4, 128, True, 500, (256, 8, 1, 0), False),
]


def _layer(x0, x16, last):
    """bias 2^24, products x[0] and -2^24 x[16] in fp32, one K block after the other."""
    acc = np.float32(0) if last else BIG
    acc = np.float32(acc + x0)
    acc = np.float32(acc + np.float32(-BIG * x16))
    return np.float32(acc + BIG) if last else acc


@pytest.mark.parametrize("H,L,M,K,ed,value,n,grids,last", SHAPES, ids=["-".join(map(str, s[:5])) for s in SHAPES])
def test_bias_place(H, L, M, K, ed, value, n, grids, last):
    torch = need_gpu()
    import paper_2606_11440_amd as P
    A, F = M * K, ed + 4 * M + 1
    cfg = workload.configs.get("c2", E=1, M=M, K=K, embed_dim=ed, feat_dim=F, widths=[H] * (L - 1) + [A],
                               value_head=value)
    W, b, k = [], [], F
    x0 = x16 = np.float32(1)
    for rows in [H] * (L - 1) + [A + value]:
        w = np.zeros((rows, k), np.float32)
        w[:, 0], w[:, 16] = 1, -BIG
        W.append(w)
        b.append(np.full(rows, BIG, np.float32))
        y = _layer(x0, x16, last)
        x0 = x16 = max(y, np.float32(0))   # 0, 1 or a power of two: exact in bf16
        k = rows
    emb = torch.zeros((4, ed), dtype=torch.bfloat16, device="cuda")
    emb[:, 0] = emb[:, 16] = 1
    dev = lambda x, t: torch.as_tensor(x, dtype=t).cuda()  # noqa: E731
    arr = P.make_arrivals(dev([0, n], torch.int32), dev(np.arange(n) % 4, torch.int32),
                          dev(np.full(n, 50), torch.int16), dev(np.full(n, 3), torch.int16))
    pool = P.Pool(cfg, W, b, emb, np.full((1, M), 2, np.int32))
    for grid in grids:
        pool.set_launch(grid)
        act = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        lg = torch.full((n, A), float("nan"), device="cuda")
        pool.route(arr, act, lg)
        z = lg.cpu().numpy()
        assert (z == y).all(), (grid, y, np.unique(z)[:4])
        assert (act.cpu().numpy() == 0).all()
    assert pool.error() == 0
    pool.close()
