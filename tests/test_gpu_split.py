"""GPU: the feature-split bf16 route kernel (a block per 32, 64 or 128 rows,
every hidden layer's features split over its waves) in lockstep with the oracle
at the sizes where it can go wrong: one row, a row less and more than a row
tile and than a block, envs without rows, embeddings that are not a multiple of
16 or of 8 wide, feature vectors longer than one LDS pass, one to three output
tiles, a bad q_idx. Tolerances are those of the other lockstep tests. The grid
given to set_launch picks the rows per block."""
import numpy as np
import pytest

import workload
from gpu_util import Pair, note

pytestmark = pytest.mark.gpu

ROWS = (1, 31, 32, 33, 64, 65, 127, 128, 129, 300)
# hidden, layers, M, K, embedding width, zero padding of the feature vector, value head
SHAPES = [
    (32, 2, 5, 3, 64, 0, False),
    (64, 3, 3, 4, 30, 0, True),        # embedding rows not 16-byte aligned
    (64, 2, 16, 4, 64, 0, True),       # 65 outputs: three output tiles
    (128, 3, 8, 4, 40, 7, True),       # 33 outputs; an embedding block that ends in tail features
    (256, 3, 5, 3, 384, 0, False),     # two LDS passes over the features
    (256, 2, 8, 3, 64, 0, True),
    (512, 3, 16, 4, 128, 0, False),
    (512, 2, 16, 4, 440, 7, True),     # 512 features: the longest vector
]


@pytest.mark.parametrize("H,L,M,K,ed,pad,value", SHAPES, ids=["-".join(map(str, s[:5])) for s in SHAPES])
def test_split_lockstep(H, L, M, K, ed, pad, value):
    E = 7
    cfg = workload.configs.get("c2", E=E, T=3 * len(ROWS), lam=16.0, qcap=64, M=M, K=K, embed_dim=ed,
                               feat_dim=ed + 4 * M + 1 + pad, widths=[H] * (L - 1) + [M * K], value_head=value)
    note(f"[split] H={H} L={L} M={M} K={K} ed={ed}")
    p = Pair(cfg, seed=91, Q=300)
    rng = np.random.default_rng(3)
    for t in range(cfg["T"]):
        rows = ROWS[t // 3]
        # rows per block: 32 (a grid of at least a block per 32 rows), 64, or the largest
        p.gpu.set_launch((256, (rows + 63) // 64, 1)[t % 3])
        p.counts[t] = rng.multinomial(rows, [0.4, 0.0, 0.3, 0.1, 0.0, 0.2, 0.0])
        if value and t % 2:
            p.step_rl(p.arrivals(t), seed=700 + t)
        else:
            p.step(p.arrivals(t))
        if t % 5 == 4:
            p.compare_state(ctx=f"t={t}")
    note(f"  rows={p.rows_checked} near-tie flips={p.flips}")
    assert p.gpu.error() == 0
    p.close()


@pytest.mark.parametrize("blocks", [256, 2, 1])
def test_split_bad_row(blocks):
    """A q_idx out of range routes its row to -1 with zero logits, and no other row."""
    cfg = workload.configs.get("c2", E=2, T=1, embed_dim=128, feat_dim=128 + 21, widths=[256, 256, 15])
    p = Pair(cfg, seed=5, Q=64)
    p.gpu.set_launch(blocks)
    p.counts[0] = (60, 37)
    arr = p.arrivals(0)
    good = _route(p, arr, cfg["A"])
    for r, v in ((0, -1), (41, 64), (96, 1 << 30)):
        arr["q_idx"][r] = v
    act, lg = _route(p, arr, cfg["A"])
    bad = np.isin(np.arange(97), (0, 41, 96))
    assert (act[bad] == -1).all() and (lg[bad] == 0).all()
    assert (act[~bad] == good[0][~bad]).all() and (lg[~bad] == good[1][~bad]).all()
    assert p.gpu.error() == 1
    p.close()


def _route(p, arr, A):
    n = int(arr["q_idx"].size)
    act = p.torch.full((n,), -7, dtype=p.torch.int32, device="cuda")
    lg = p.torch.full((n, A), float("nan"), device="cuda")
    p.gpu.route(p.P.device_arrivals(arr), act, lg)
    return act.cpu().numpy(), lg.cpu().numpy()
