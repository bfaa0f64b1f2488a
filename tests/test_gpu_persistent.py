"""GPU: every persistent bf16 route kernel and launch shape in lockstep with the
oracle, on a grid of one block with the row counts that select it (ticks of up to
64 rows per block, 128 for hidden width 512, go to the feature-split kernel):
86 -> 256 -> 256 -> 15 very light (65 to 128 rows), light (to 384) and heavy,
greedy and RL; 104 -> 256 -> 24 greedy, RL below 1,024 rows and from there on;
193 -> 512 -> 512 -> 64 with two and with three output tiles (a value row). Row
counts at the edges of those ranges and of 32- and 64-row tiles; envs without
rows; a bad q_idx at both ends of a tick and inside it. Tolerances are those of
the other lockstep tests."""
import numpy as np
import pytest

import workload
from gpu_util import Pair, note

pytestmark = pytest.mark.gpu

# workload, value head (then RL outputs, else greedy), rows per tick
CASES = [
    ("c2", False, (65, 96, 97, 127, 128)),                  # very light: 8 waves of 32 rows, pipelined
    ("c2", False, (129, 160, 255, 383, 384)),               # light: 16 waves of 32 rows
    ("c2", False, (385, 449, 513, 640)),                    # 8 waves of 64 rows
    ("c2", True, (65, 129, 193, 384)),                      # 16 waves of 32 rows
    ("c2", True, (385, 448, 513)),                          # 8 waves of 64 rows
    ("c4", False, (65, 128, 191, 770)),                     # 12 waves of 64 rows
    ("c4", True, (65, 511, 513, 1023)),                     # 16 waves of 32 rows
    ("c4", True, (1024, 1089)),                             # 12 waves of 64 rows
    ("c3", False, (129, 255, 257, 300)),                    # streamed, two output tiles
    ("c3", True, (129, 256, 289)),                          # three output tiles
]
SHARE = [0.3, 0.0, 0.02, 0.2, 0.08, 0.0, 0.1, 0.29, 0.01]


@pytest.mark.parametrize("name,value,rows", CASES, ids=[f"{c[0]}-{'rl' if c[1] else 'greedy'}-{c[2][0]}" for c in CASES])
def test_persistent_lockstep(name, value, rows):
    cfg = workload.configs.get(name, E=9, T=2 * len(rows), qcap=512, value_head=value)
    note(f"[persistent] {name} {'rl' if value else 'greedy'} {rows}")
    p = Pair(cfg, seed=37, Q=300)
    p.gpu.set_launch(1)
    rng = np.random.default_rng(rows[0])
    for t in range(cfg["T"]):
        p.counts[t] = rng.multinomial(rows[t // 2], SHARE)
        if value:
            p.step_rl(p.arrivals(t), seed=1300 + t, greedy=t % 4 == 3)
        else:
            p.step(p.arrivals(t))
        if t % 2:
            p.compare_state(ctx=f"t={t}")
    assert p.gpu.error() == 0
    note(f"  rows={p.rows_checked} near-tie flips={p.flips}")
    p.close()


@pytest.mark.parametrize("name,value,rows", CASES, ids=[f"{c[0]}-{'rl' if c[1] else 'greedy'}-{c[2][0]}" for c in CASES])
def test_persistent_bad_rows(name, value, rows):
    """A q_idx out of range gives its row no action and zero outputs, and changes no other row."""
    cfg = workload.configs.get(name, E=9, T=1, qcap=512, value_head=value)
    p = Pair(cfg, seed=38, Q=300)
    p.gpu.set_launch(1)
    n = rows[-1]
    p.counts[0] = np.random.default_rng(1).multinomial(n, SHARE)
    arr = p.arrivals(0)
    good = _outputs(p, arr, value)
    bad = (0, 31, 40, n - 1)
    for r, v in zip(bad, (-1, 300, 1 << 30, -(1 << 31))):
        arr["q_idx"][r] = v
    got = _outputs(p, arr, value)
    at = np.isin(np.arange(n), bad)
    assert (got["actions"][at] == -1).all()
    for k, x in got.items():
        if k != "actions":
            assert (x[at] == 0).all(), k
        np.testing.assert_array_equal(x[~at], good[k][~at], err_msg=k)
        assert np.isfinite(x).all(), k
    assert p.gpu.error() == 1
    p.close()


def _outputs(p, arr, value):
    n, A = int(arr["q_idx"].size), p.cfg["A"]
    f = dict(device="cuda")
    new = lambda *s: p.torch.full(s, float("nan"), **f)  # noqa: E731
    out = dict(actions=p.torch.full((n,), -7, dtype=p.torch.int32, **f), logits=new(n, A))
    dev = p.P.device_arrivals(arr)
    if value:
        out.update(logp=new(n), entropy=new(n), value=new(n))
        p.gpu.route_sample(dev, 11, out["actions"], out["logp"], out["entropy"], out["value"], out["logits"])
    else:
        p.gpu.route(dev, out["actions"], out["logits"])
    return {k: x.cpu().numpy() for k, x in out.items()}
