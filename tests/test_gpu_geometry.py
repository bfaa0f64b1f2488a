"""GPU: results independent of launch shapes, and exact pins of the features
the bf16 route kernels gather.

* Launch shapes (im_set_launch): the same pool state ticked with the default
  persistent route grid (one block per compute unit), grids of 37 and of 1
  block, and the kernels that launch one block per group of rows, with 4, 2
  and 1 envs per schedule workgroup. Actions, logits and the whole integer
  state are identical bit for bit across the persistent grids and workgroup
  sizes; the block-per-group kernels agree with them within the logit tolerance
  (and the integer state is compared where no near tie flipped an action).
* Feature columns: a policy whose layers are 0/1 selections (layer 1 picks one
  input column per hidden unit, deeper layers pass it on, the output layer
  reads it out) turns each logit into one feature, rounded to bf16 (twice,
  which is once). Every load-statistic column and the budget column of the
  c2, c3 and c4 shapes is read this way through the kernels of small ticks (the
  default grid) and, on a grid of one block, through the persistent kernels and
  compared bit for bit with the oracle's feature vector (Eq. 1 restated): a
  swapped, shifted or mis-scaled column fails, which the 2e-2 logit tolerance
  of the lockstep tests could hide."""
import numpy as np
import pytest

import oracle
import workload
from gpu_util import Pair, need_gpu, note
from helpers import assert_state_equal, logits_close, near_tie

pytestmark = pytest.mark.gpu


def _run(cfg, seed, route_blocks, sched_waves, T):
    torch = need_gpu()
    import paper_2606_11440_amd as P
    p = Pair(cfg, seed=seed, Q=1024, e0=0, e1=1)
    p.gpu.set_launch(route_blocks, sched_waves)
    acts, lgs = [], []
    for t in range(T):
        arr = p.arrivals(t)
        n = max(int(arr["q_idx"].size), 1)
        dev = P.device_arrivals(arr)
        act = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        lg = torch.full((n, cfg["A"]), float("nan"), dtype=torch.float32, device="cuda")
        p.gpu.route(dev, act, lg)
        p.gpu.schedule(dev, act)
        torch.cuda.synchronize()
        acts.append(act.cpu().numpy())
        lgs.append(lg.cpu().numpy())
    s = p.gpu.state()
    assert p.gpu.error() == 0
    p.close()
    return acts, lgs, s


@pytest.mark.parametrize("name,over", [("c2", dict(E=700, lam=64.0)), ("c4", dict(E=1500)),
                                       ("c3", dict(E=300)), ("c1", dict(E=300))])
def test_launch_shapes_identical(name, over):
    cfg = workload.configs.get(name, T=10, **over)
    note(f"[launch_shapes] {name} E={cfg['E']}")
    shapes = [(-1, 4), (37, 2), (1, 1), (0, 4)]
    ref = _run(cfg, 60, *shapes[0], cfg["T"])
    rtol = 2e-2 if cfg["dtype"] == "bf16" else 1e-4
    for rb, sw in shapes[1:]:
        acts, lgs, s = _run(cfg, 60, rb, sw, cfg["T"])
        if rb != 0:
            for t in range(cfg["T"]):
                np.testing.assert_array_equal(acts[t], ref[0][t], err_msg=f"actions grid {rb} t={t}")
                np.testing.assert_array_equal(lgs[t], ref[1][t], err_msg=f"logits grid {rb} t={t}")
            assert_state_equal(s, ref[2], ctx=f"grid {rb} waves {sw}")
            continue
        # one block per group of rows: the same arithmetic per row, so the same
        # bits are expected; the tolerance is the contract
        flips, bitwise = 0, True
        for t in range(cfg["T"]):
            a, b = lgs[t].astype(np.float64), ref[1][t].astype(np.float64)
            bitwise &= bool(np.array_equal(lgs[t], ref[1][t]))
            assert logits_close(a, b, rtol).all(), f"generic kernel logits t={t}"
            for r in np.nonzero(acts[t] != ref[0][t])[0]:
                assert near_tie(b[r], int(ref[0][t][r]), int(acts[t][r]), rtol), (t, r)
                flips += 1
        note(f"  block-per-group kernels: logits bitwise equal {bitwise}, flips {flips}")
        if flips == 0:
            assert_state_equal(s, ref[2], ctx="a block per group")


def _select_weights(cfg, cols):
    """0/1 layers: hidden unit r of every layer carries input column cols[r];
    output a reads hidden unit a (a < len(cols)); all biases 0."""
    D, widths = cfg["feat_dim"], cfg["widths"]
    W, b = [], []
    fan_in = D
    for li, w in enumerate(widths):
        m = np.zeros((w, fan_in), np.float32)
        for r, c in enumerate(cols):
            m[r, c if li == 0 else r] = 1.0
        W.append(m)
        b.append(np.zeros(w, np.float32))
        fan_in = w
    return W, b


# grid 1: ticks of about 96 (very light shape), 144 (light), 480 rows (64-row tiles) on c2's persistent kernels
SHAPES = [("c2", dict(E=6, lam=24.0), -1), ("c4", dict(E=6, lam=40.0), -1), ("c3", dict(E=4, lam=24.0), -1),
          ("c2", dict(E=4, lam=24.0), 1), ("c2", dict(E=6, lam=24.0), 1), ("c2", dict(E=20, lam=24.0), 1),
          ("c4", dict(E=6, lam=40.0), 1), ("c3", dict(E=8, lam=24.0), 1)]


@pytest.mark.parametrize("name,over,blocks", SHAPES, ids=[f"{s[0]}-{s[1]['E']}-{s[2]}" for s in SHAPES])
def test_feature_columns_exact(name, over, blocks):
    torch = need_gpu()
    import paper_2606_11440_amd as P
    cfg = workload.configs.get(name, T=14, **over)
    Ed, M, A = cfg["embed_dim"], cfg["M"], cfg["A"]
    tail = list(range(Ed, Ed + 4 * M + 1))          # 4M load statistics, then the budget
    note(f"[feature_columns] {name}: {len(tail)} columns, {A} per pool")
    Q = 256
    table, emb_vals = workload.gen.embedding(cfg, 61, rows=Q)
    cap = workload.gen.capacities(cfg, 61)
    emb_dev = torch.from_numpy(table.view(np.int16)).cuda()
    counts = workload.gen.counts(cfg, 61)
    checked = 0
    for c0 in range(0, len(tail), A):
        cols = tail[c0:c0 + A]
        W, b = _select_weights(cfg, cols)
        gpu = P.Pool(cfg, W, b, emb_dev, cap, None)
        gpu.set_launch(blocks)
        orc = oracle.Oracle(cfg, W, b, emb_vals, cap, None, E=cfg["E"], threads=4)
        for t in range(cfg["T"]):
            arr = workload.gen.tick(cfg, 61, t, counts[t], Q)
            n = int(arr["q_idx"].size)
            if n == 0:
                continue
            dev = P.device_arrivals(arr)
            act = torch.full((n,), -7, dtype=torch.int32, device="cuda")
            lg = torch.full((n, A), float("nan"), dtype=torch.float32, device="cuda")
            gpu.route(dev, act, lg)
            torch.cuda.synchronize()
            g = lg.cpu().numpy()
            o_act, o_lg = orc.route(arr)
            off = arr["offsets"]
            for e in range(cfg["E"]):
                for i in range(int(off[e]), int(off[e + 1])):
                    x = orc.features(e, int(arr["q_idx"][i]), int(arr["budget"][i]))
                    want = np.array([oracle.round_bf16(float(x[c])) for c in cols], np.float64)
                    np.testing.assert_array_equal(g[i, :len(cols)].astype(np.float64), want,
                                                  err_msg=f"{name} cols {cols[0]}.. t={t} row {i}")
                    np.testing.assert_array_equal(o_lg[i, :len(cols)], want, err_msg="oracle")
                    checked += 1
            gpu.schedule(dev, act)
            orc.schedule(arr, act.cpu().numpy())
        assert_state_equal(gpu.state(), orc.state(), ctx=f"{name} cols {cols[0]}..")
        assert gpu.error() == 0
        gpu.close()
    note(f"  rows checked {checked}")
    assert checked > 100
