"""GPU parity of the dual update (im_dual_update, Eq. 7) and of the Q16 cost
counter it reads: lambda bit-exact with the oracle (both take the same
correctly rounded fp64 steps over exact integer sums), the cost counters
bit-exact in every state comparison; the closed-form ramp of a single-slot
FCFS model, a c2 workload with updates every few ticks (two sampled envs
followed by the oracle, all envs reduced on the GPU: so the oracle runs the
whole small pool here) and no-completion calls."""
import numpy as np
import pytest

import workload
from gpu_util import Pair, need_gpu, note

pytestmark = pytest.mark.gpu


def _lam(torch, v):
    return torch.tensor([v], dtype=torch.float64, device="cuda")


def test_dual_closed_form_ramp():
    torch = need_gpu()
    from helpers import tiny_cfg
    cfg = tiny_cfg(M=1, K=1, widths=[32, 1], key_mode="fcfs", qcap=16, cap_hi=1, T=200)
    note("[dual_ramp]")
    p = Pair(cfg, seed=1, Q=4)
    lam_g, lam_o = _lam(torch, 0.2), 0.2
    for t in range(cfg["T"]):
        if t % 5 == 0:
            arr = dict(offsets=np.array([0, 1], np.int32), q_idx=np.array([0], np.int32),
                       budget=np.array([8], np.int16), base_svc=np.array([4], np.int16))
        else:
            z = np.zeros(0, np.int32)
            arr = dict(offsets=np.array([0, 0], np.int32), q_idx=z, budget=z.astype(np.int16),
                       base_svc=z.astype(np.int16))
        p.step(arr)
        if t % 10 == 9:
            p.gpu.dual_update(0.001, 1.0, lam_g)
            lam_o = p.orc.dual_update(lam_o, 0.001, 1.0)
            torch.cuda.synchronize()
            assert lam_g.item() == lam_o, (t, lam_g.item(), lam_o)
    assert lam_o == pytest.approx(0.2 - 20 * 0.0005, abs=1e-12)
    p.compare_state(ctx="ramp end")
    p.close()


@pytest.mark.parametrize("name,E", [("c2", 6), ("c4", 8)])
def test_dual_matches_oracle(name, E):
    torch = need_gpu()
    cfg = workload.configs.get(name, E=E, T=50)
    note(f"[dual_matches_oracle] {name} E={E}")
    p = Pair(cfg, seed=31, Q=256)
    lam_g, lam_o = _lam(torch, 0.3), 0.3
    for t in range(cfg["T"]):
        p.step(p.arrivals(t))
        if t % 7 == 6:
            for _ in range(2):                 # the second call has no new completions
                p.gpu.dual_update(0.05, 0.9, lam_g)
                lam_o = p.orc.dual_update(lam_o, 0.05, 0.9)
            torch.cuda.synchronize()
            assert lam_g.item() == lam_o, (t, lam_g.item(), lam_o)
            p.compare_state(ctx=f"{name} t={t}")
    p.close()


@pytest.mark.parametrize("E", [1, 1023, 1025])
def test_dual_running_totals_follow_the_counters(E):
    """More envs than running totals, and a state restore between updates: each
    update equals Eq. 7 over the difference of the exported counters' sums."""
    torch = need_gpu()
    import paper_2606_11440_amd as P
    cfg = workload.configs.get("c2", E=E, M=2, K=1, T=30, lam=3.0, qcap=32, embed_dim=64, feat_dim=73,
                               widths=[64, 2], svc_mu=0.0)
    W, b = workload.gen.weights(cfg, 3, 0.1)
    emb = torch.zeros((16, 64), dtype=torch.bfloat16, device="cuda")
    pool = P.Pool(cfg, W, b, emb, workload.gen.capacities(cfg, 3))
    counts = workload.gen.counts(cfg, 3)
    lam, want, last, saved = _lam(torch, 0.4), 0.4, (0, 0), None
    for t in range(cfg["T"]):
        pool.tick(P.device_arrivals(workload.gen.tick(cfg, 3, t, counts[t], 16)))
        if t == 9:
            saved = pool.state()
        if t == 14 or t == 22:
            pool.write_state(0, saved)      # back to tick 10: the totals fall with the counters
        if t % 4 == 3:
            pool.dual_update(0.05, 2.0, lam)
            s = pool.state()
            tot = (int(s["completed"].sum()), int(s["cost_q16"].sum()))
            dn, dc = tot[0] - last[0], tot[1] - last[1]
            last = tot
            if dn > 0:
                want = want + 0.05 * (dc / (65536.0 * dn) - 1.0)
                want = min(max(want, 0.0), 2.0)
            torch.cuda.synchronize()
            assert lam.item() == want, (t, lam.item(), want)
    assert last[0] > 0 and pool.error() == 0
    pool.close()


@pytest.mark.parametrize("steps", [1, 3])
@pytest.mark.parametrize("E,first,count", [(1, 0, 1), (300, 299, 1), (2100, 1000, 100), (2100, 5, 1), (2100, 0, 2100),
                                           (2100, 700, 1300)])
def test_dual_totals_after_a_partial_restore(E, first, count, steps):
    """Envs restored with other counters (a range that wraps round the shards of
    the running totals, one env, more envs than shards): the next update takes
    exactly the difference, and the other envs' totals stay."""
    torch = need_gpu()
    import paper_2606_11440_amd as P
    cfg = workload.configs.get("c2", E=E, M=3, K=1, T=12, lam=3.0, qcap=32, embed_dim=64, feat_dim=77,
                               widths=[64, 3], svc_mu=0.0, max_steps=steps)
    W, b = workload.gen.weights(cfg, 3, 0.1)
    emb = torch.zeros((16, 64), dtype=torch.bfloat16, device="cuda")
    pool = P.Pool(cfg, W, b, emb, workload.gen.capacities(cfg, 3))
    counts = workload.gen.counts(cfg, 3)
    lam, want, last = _lam(torch, 0.4), 0.4, (0, 0)
    for t in range(cfg["T"]):
        pool.tick(P.device_arrivals(workload.gen.tick(cfg, 3, t, counts[t], 16)))
        if t in (5, 9):
            s = pool.state(first, count)
            s["completed"] += 2 + np.arange(count)[:, None] % 3
            s["cost_q16"] += 70000 * (1 + np.arange(count)[:, None] % 5)
            s["q_done"] += 1 + np.arange(count) % 2
            if steps > 1:
                pool.write_chain_state(first, s, pool.chain_state(first, count))
            else:
                pool.write_state(first, s)
        if t in (4, 5, 9, 11):
            pool.dual_update(0.05, 2.0, lam)
            s = pool.state()
            tot = (int((s["q_done"] if steps > 1 else s["completed"]).sum()), int(s["cost_q16"].sum()))
            dn, dc = tot[0] - last[0], tot[1] - last[1]
            last = tot
            if dn > 0:
                want = min(max(want + 0.05 * (dc / (65536.0 * dn) - 1.0), 0.0), 2.0)
            torch.cuda.synchronize()
            assert lam.item() == want, (t, lam.item(), want)
    assert last[0] > 0 and pool.error() == 0
    pool.close()
