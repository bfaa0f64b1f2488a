"""GPU: the persistent route kernels whose waves own 64 rows, a row context per
lane (86 -> 256 -> 256 -> 15 and 104 -> 256 -> 24), greedy and RL outputs, in
lockstep with the oracle on a grid of one block: ticks a row more and less than
whole 64-row tiles and than both MFMA tiles of one, envs without rows, a bad
q_idx in either tile. Tolerances are those of the other lockstep tests."""
import numpy as np
import pytest

import workload
from gpu_util import Pair, note

pytestmark = pytest.mark.gpu

# rows per tick: all above the row counts at which one block takes a light or 32-row shape
ROWS = (1024, 1025, 1055, 1056, 1057, 1087, 1089)


@pytest.mark.parametrize("name", ["c2", "c4"])
def test_rows64_lockstep(name):
    cfg = workload.configs.get(name, E=9, T=2 * len(ROWS), qcap=512, value_head=True)
    note(f"[rows64] {name}")
    p = Pair(cfg, seed=17, Q=400)
    p.gpu.set_launch(1)
    rng = np.random.default_rng(9)
    p.counts[0] = rng.multinomial(ROWS[0], [0.3, 0.0, 0.02, 0.2, 0.08, 0.0, 0.1, 0.29, 0.01])
    arr = p.arrivals(0)
    n = int(arr["q_idx"].size)
    bad = (0, 31, 32, 63, 64 + 40, n - 1)
    for r in bad:
        arr["q_idx"][r] = -5
    f = dict(device="cuda")
    act, lp = p.torch.full((n,), -7, dtype=p.torch.int32, **f), p.torch.full((n,), float("nan"), **f)
    val, lg = lp.clone(), p.torch.full((n, cfg["A"]), float("nan"), **f)
    p.gpu.route_sample(p.P.device_arrivals(arr), 3, act, lp, None, val, lg)
    a, z, v = act.cpu().numpy(), lg.cpu().numpy(), val.cpu().numpy()
    for r in range(n):
        if r in bad:
            assert a[r] == -1 and lp[r] == 0 and v[r] == 0 and (z[r] == 0).all()
    ok = ~np.isin(np.arange(n), bad)
    assert (a[ok] >= 0).all() and (z[ok] != 0).any(1).all() and not np.isnan(z).any()
    assert p.gpu.error() == 1
    p.gpu.clear_error()
    for t in range(cfg["T"]):
        p.counts[t] = rng.multinomial(ROWS[t // 2], [0.3, 0.0, 0.02, 0.2, 0.08, 0.0, 0.1, 0.29, 0.01])
        if t % 2:
            p.step_rl(p.arrivals(t), seed=900 + t, greedy=t % 4 == 3)
        else:
            p.step(p.arrivals(t))
        if t % 4 == 3:
            p.compare_state(ctx=f"t={t}")
    assert p.gpu.error() == 0
    note(f"  rows={p.rows_checked} near-tie flips={p.flips}")
    p.close()
