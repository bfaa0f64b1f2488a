"""GPU: the masked argmax and the draw of the route kernels on logits chosen
exactly (a policy with zero weights, whose logits are its biases): ties, signed
zeros, the lowest finite value, infinities and NaN, with every model enabled
and with some disabled. The greedy action is the oracle's: a scan over the valid
actions that takes each whose logit exceeds the best one's, so NaN is passed
over but for the lowest valid action's, which nothing exceeds (-1 when none is
valid); a drawn action is always valid, follows the same rule where logits are
NaN and never has probability 0 beside finite logits. The envs' masks differ, and their border lies
between two 32-row tiles of a 64-row one and inside a 32-row tile."""
import numpy as np
import pytest

import oracle
import workload
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

INF, NAN, LOW = np.inf, np.nan, np.finfo(np.float32).min
# dtype, hidden, layers, M, K, launch (route blocks), rows of either env: the 32-row, 64-row (a lane per row) and
# fp32 epilogues, one and two output tiles, split and persistent kernels
POOLS = [("bf16", 256, 3, 5, 3, -1, 150, 150), ("bf16", 256, 3, 5, 3, 1, 150, 150), ("bf16", 64, 3, 16, 4, -1, 150, 150),
         ("bf16", 512, 3, 16, 4, 1, 150, 150), ("f32", 64, 3, 5, 3, -1, 150, 150), ("f32", 32, 3, 16, 4, -1, 150, 150),
         ("bf16", 256, 3, 5, 3, 1, 224, 190), ("bf16", 256, 3, 5, 3, 1, 205, 300),
         ("bf16", 256, 2, 8, 3, 1, 544, 500), ("bf16", 256, 2, 8, 3, 1, 525, 600)]


def _logits(A):
    r = np.random.default_rng(1)
    z = [np.zeros(A), np.where(np.arange(A) % 2, 0.0, -0.0), np.full(A, LOW), np.full(A, -INF),
         np.full(A, NAN), np.where(np.arange(A) % 3, NAN, -INF), np.where(np.arange(A) == A - 1, 1.0, -INF),
         np.where(np.arange(A) == A // 2, INF, 0.0), r.normal(size=A)]
    z[-1][r.integers(0, A, 3)] = NAN
    z.append(np.round(r.normal(size=A) * 2) / 2)   # several ties
    z.append(r.permutation(A) * 1e-41)             # subnormal
    z += [np.where(np.arange(A) % 2, r.normal(size=A), NAN), np.where(np.arange(A) % 2, -INF, NAN)]
    return [np.asarray(x, np.float32) for x in z]


@pytest.mark.parametrize("dtype,H,L,M,K,blocks,n0,n1", POOLS, ids=["-".join(map(str, p)) for p in POOLS])
def test_exact_logits(dtype, H, L, M, K, blocks, n0, n1):
    torch = need_gpu()
    import paper_2606_11440_amd as P
    A, E, n = M * K, 2, n0 + n1
    of_env = (slice(0, n0), slice(n0, n))
    ed = 128 if H == 512 else 64
    cfg = workload.configs.get("c2" if dtype == "bf16" else "c1", E=E, M=M, K=K, embed_dim=ed,
                               feat_dim=ed + 4 * M + 1, widths=[H] * (L - 1) + [A])
    emb = torch.zeros((8, ed), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    dev = lambda x, t: torch.as_tensor(x, dtype=t).cuda()  # noqa: E731
    rows = dict(offsets=np.array([0, n0, n], np.int32), q_idx=np.arange(n, dtype=np.int32) % 8,
                budget=np.full(n, 50, np.int16), base_svc=np.full(n, 3, np.int16))
    arr = P.make_arrivals(dev([0, n0, n], torch.int32), dev(np.arange(n) % 8, torch.int32),
                          dev(np.full(n, 50), torch.int16), dev(np.full(n, 3), torch.int16))
    for z in _logits(A):
        W = [np.zeros((H, ed + 4 * M + 1), np.float32), np.zeros((H, H), np.float32), np.zeros((A, H), np.float32)]
        b = [np.zeros(H, np.float32), np.zeros(H, np.float32), z]
        if L == 2:
            del W[1], b[1]
        pool = P.Pool(cfg, W, b, emb, np.full((E, M), 2, np.int32))
        orc = oracle.Oracle(cfg, W, b, np.zeros((8, ed)), np.full((E, M), 2, np.int32))
        pool.set_launch(blocks)
        off = (0, M - 1)   # models disabled in env 1
        for m in off:
            pool.set_enabled(1, m, 0)
            orc.set_enabled(1, m, 0)
        act = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        pool.route(arr, act)
        drawn = act.clone()
        ent = torch.empty(n, device="cuda")
        pool.route_sample(arr, 5, drawn, entropy=ent)
        greedy = act.clone()
        pool.route_sample(arr, 5, greedy, greedy=True)
        torch.cuda.synchronize()
        scan, _ = orc.route(rows)
        valid = np.ones((E, A), bool)
        for m in off:
            valid[1, m * K:(m + 1) * K] = False
        for e in range(E):
            got = act[of_env[e]].cpu().numpy()
            ok, first = valid[e] & ~np.isnan(z), int(np.nonzero(valid[e])[0][0])
            want = first if np.isnan(z[first]) else int(np.nonzero(ok & (z == z[ok].max()))[0][0])
            assert (scan[of_env[e]] == want).all()
            assert (got == want).all(), (z, e, want, got[:4])
            assert (greedy[of_env[e]].cpu().numpy() == want).all()
            d = drawn[of_env[e]].cpu().numpy()
            assert valid[e][d].all()
            assert (d == first).all() if np.isnan(z[first]) else not np.isnan(z[d]).any()
            if np.isfinite(z[valid[e]]).any() and not np.isnan(z).any() and not np.isposinf(z).any():
                assert not np.isneginf(z[d]).any()
            if np.isfinite(z).all():
                p = np.exp((z[valid[e]] - z[valid[e]].max()).astype(np.float64))
                p /= p.sum()
                h = -(p * np.log(np.maximum(p, 1e-300))).sum()
                # fp32 sums of at most 64 terms, |z| p bounded by the shift except at the lowest value
                if z.min() > -100:
                    assert np.allclose(ent[of_env[e]].cpu().numpy(), h, atol=1e-5)
        for m in range(M):
            pool.set_enabled(1, m, 0)
        pool.route(arr, act)
        pool.route_sample(arr, 6, drawn)
        torch.cuda.synchronize()
        assert (act[n0:].cpu().numpy() == -1).all() and (drawn[n0:].cpu().numpy() == -1).all()
        assert pool.error() == 0
        pool.close()
