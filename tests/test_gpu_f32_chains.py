"""GPU: the fp32 feature-split route kernel in chain pools, where the row count is
known on the device only and picks the blocks' row tiles there: ticks with few and
with many rows under a bound above 16 rows per compute unit, in lockstep with the
oracle. Tolerances are those of the other lockstep tests."""
import numpy as np
import pytest

import workload
from gpu_util import Pair, need_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,L", [(64, 2), (128, 3)])
def test_f32_chain_blocks_lockstep(H, L):
    torch = need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    M, K, slots = 5, 3, 8
    E = 16 * cus // (M * slots) + 9            # the pending calls alone may exceed a tile per unit
    # arrivals on top of what is pending: few, around one and two tiles per unit, and past a round
    arrivals = [3, 0, 17, 16 * cus - 700, 16 * cus - 300, 16 * cus, 24 * cus + 5, 32 * cus - 200, 32 * cus, 5]
    cfg = workload.configs.get("c1", E=E, M=M, K=K, T=len(arrivals), qcap=64, cap_lo=slots, cap_hi=slots, max_steps=3,
                               svc_mu=0.0, max_arrivals=4096, widths=[H] * (L - 1) + [M * K])
    p = Pair(cfg, seed=29, Q=200)
    rng = np.random.default_rng(H)
    share = rng.dirichlet(np.ones(E))
    share[[0, E // 2, E - 1]] = 0.0
    share /= share.sum()
    seen = []
    for t, n in enumerate(arrivals):
        p.counts[t] = rng.multinomial(n, share)
        before = p.rows_checked
        p.step(p.arrivals(t))
        seen.append(p.rows_checked - before)
    p.compare_state(ctx="end")
    note(f"[f32 chains] H={H} rows per tick {seen}, near-tie flips {p.flips}")
    assert min(seen) <= 16 * cus < max(seen) and any(16 * cus < n <= 32 * cus for n in seen)
    assert p.gpu.error() == 0
    p.close()
