"""GPU: state exports. The export kernel writes a range in one launch, or in
several when it exceeds the staging buffer, and sorts each queue's unsorted part
in LDS (on the host past 4,096 entries): whatever the range, every env's part is
the same, and the queues are in service order. (Content against the oracle is
compared by every lockstep test.)"""
import numpy as np
import pytest

import workload
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


# E, qcap, requests per env-tick, ticks: one launch; several launches (11 MB of queues); pools past 4,096 entries
@pytest.mark.parametrize("E,qcap,lam,T", [(3, 100, 6.0, 20), (70, 2048, 64.0, 40), (3, 16384, 1000.0, 30)])
def test_export_ranges_agree(E, qcap, lam, T):
    torch = need_gpu()
    import paper_2606_11440_amd as P
    cfg = workload.configs.get("c2", E=E, T=T, lam=lam, qcap=qcap, widths=[64, 64, 15], zipf_s=2.0)
    W, b = workload.gen.weights(cfg, 3, 0.1)
    emb = torch.randn((64, 64), generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    pool = P.Pool(cfg, W, b, emb, workload.gen.capacities(cfg, 3), workload.gen.logit_bias(cfg))
    counts = workload.gen.counts(cfg, 3)
    for t in range(T):
        pool.tick(P.device_arrivals(workload.gen.tick(cfg, 3, t, counts[t], 64)))
    whole = pool.state()
    assert whole["t"] == T and pool.error() == 0
    if qcap > 4096:
        assert whole["qlen"].max() > 4096 + 64
    bare = pool.state(with_queues=False)
    for k, v in whole.items():
        if k != "queues" and k != "t":
            np.testing.assert_array_equal(bare[k], v, err_msg=k)
    for e0, n in [(e, 1) for e in range(0, E, max(1, E // 3))] + [(E - 2, 2), (1, E - 1)]:
        part = pool.state(e0, n)
        assert part["t"] == T
        for k, v in part.items():
            if k != "t":
                np.testing.assert_array_equal(v, whole[k][e0:e0 + n], err_msg=f"{k} of envs {e0}..{e0 + n}")
    for e in range(E):
        for m in range(cfg["M"]):
            q, n = whole["queues"][e, m].astype(np.int64), int(whole["qlen"][e, m])
            order = (q[:n, 0] << 32) + q[:n, 1]
            assert (np.diff(order) > 0).all() and not q[n:].any(), (e, m)
    pool.close()
