"""GPU: fp32 feature-split route kernel with 32-row blocks, then 16-row blocks
for a remainder that fits one per compute unit: logits and actions of ticks
around those edges (a round is 32 rows per compute unit) in lockstep with the
oracle, with a bad q_idx in either kind of block. Tolerances are those of the
other lockstep tests. Also over the kernel's other shapes: hidden widths 64 to 256,
two and three layers, one to four output tiles, more feature groups than one LDS
pass holds, greedy and RL outputs, with a tail of 16-row blocks and without one."""
import numpy as np
import pytest

import workload
from gpu_util import Pair, need_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("whole,rest", [(0, 1), (1, 0), (1, 1), (1, 16), (1, 17), (2, 33)])
@pytest.mark.parametrize("half", [0, 1])
def test_f32_tail_lockstep(whole, rest, half):
    torch = need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 32 * cus * whole + 16 * cus * half + rest
    cfg = workload.configs.get("c1", E=70, T=2, qcap=512, max_arrivals=8192, widths=[64, 64, 15])
    note(f"[f32 tail] {n} rows")
    p = Pair(cfg, seed=23, Q=300)
    rng = np.random.default_rng(n)
    share = rng.dirichlet(np.ones(70))
    share[[0, 33, 69]] = 0.0
    share /= share.sum()
    p.counts[0] = rng.multinomial(n, share)
    arr = p.arrivals(0)
    bad = [0, n - 1]
    for r in bad:
        arr["q_idx"][r] = -5
    act = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    lg = torch.full((n, cfg["A"]), float("nan"), device="cuda")
    p.gpu.route(p.P.device_arrivals(arr), act, lg)
    a, z = act.cpu().numpy(), lg.cpu().numpy()
    assert (a[bad] == -1).all() and (z[bad] == 0).all() and not np.isnan(z).any()
    assert (np.delete(a, bad) >= 0).all()
    assert p.gpu.error() == 1
    p.gpu.clear_error()
    p.counts[1] = rng.multinomial(n, share)
    p.step(p.arrivals(1))
    p.compare_state(ctx=f"{n} rows")
    p.close()


# hidden, layers, M, K, embedding width, value head
SHAPES = [(64, 2, 16, 4, 384, False), (128, 3, 8, 3, 65, True), (128, 2, 5, 3, 64, True), (256, 3, 10, 5, 408, True),
          (256, 2, 16, 2, 100, False)]


@pytest.mark.parametrize("tail", [True, False])
@pytest.mark.parametrize("H,L,M,K,ed,value", SHAPES, ids=["-".join(map(str, s[:5])) for s in SHAPES])
def test_f32_tail_shapes(H, L, M, K, ed, value, tail):
    torch = need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 32 * cus + 37 if tail else 32 * cus - 19   # one round of 32-row blocks, then 16-row ones; 32-row blocks only
    cfg = workload.configs.get("c1", E=33, T=2, qcap=1024, max_arrivals=8192, M=M, K=K, embed_dim=ed,
                               feat_dim=ed + 4 * M + 1, widths=[H] * (L - 1) + [M * K], value_head=value)
    note(f"[f32 tail shapes] H={H} L={L} A={M * K} ed={ed} {n} rows")
    p = Pair(cfg, seed=24, Q=300)
    rng = np.random.default_rng(n + H)
    share = rng.dirichlet(np.ones(33))
    share[[0, 15, 32]] = 0.0
    share /= share.sum()
    for t in range(2):
        p.counts[t] = rng.multinomial(n, share)
        if value and t == 1:
            p.step_rl(p.arrivals(t), seed=77)
        else:
            p.step(p.arrivals(t))
    p.compare_state(ctx=f"{n} rows")
    assert p.gpu.error() == 0
    note(f"  near-tie flips={p.flips} of {p.rows_checked}")
    p.close()
