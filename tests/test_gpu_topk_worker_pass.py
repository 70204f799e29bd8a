"""The step ahead taken along by the Top-K Delta pass (saef_topk_round)
against the two halves, which run it as a kernel of its own: every byte of the
state after every iteration, at the edges of words, tiles and runs of tiles."""
import numpy as np
import pytest
import torch

from paper_2008_05823_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = {
    "tiny": [1, 3, 63, 64, 65],
    "one_tensor": [5000],                     # not pipelined over tensor groups
    "tile_edges": [511, 512, 513, 2047, 2048, 2049, 4097, 40000],
    "runs": [2048 * 2050 + 77, 2048 * 2049, 5],
}


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("K,mode,mu,shift,pct", [(1, 1, 0.0, 0, 1.0), (3, 1, 0.9, 1, 20.0),
                                                 (8, 1, 0.0, 3, 5.0), (5, 0, 0.5, 2, 1.0)])
def test_round_equals_halves(sizes, K, mode, mu, shift, pct):
    print(f"[case] {sizes} K={K} mode={mode} mu={mu} shift={shift} pct={pct}", flush=True)
    from paper_2008_05823_amd import saef as S
    w = W.custom(SIZES[sizes], K=K, period=3, mode=mode, scale_range=(1e-3, 1.0), seed=K + 21)
    off, n, d_pad = w.layout()
    pad = torch.from_numpy(~W.tensor_mask(w)).cuda()
    W64 = d_pad // 64

    def buf(rows):
        b = torch.zeros(rows * d_pad + shift, device="cuda")[shift:].view(rows, d_pad)
        b[:, pad] = float("nan")          # padding is neither read nor written
        return b

    def state():
        lay = S.Layout(off, n, d_pad, K)
        plan = S.TopK(lay, W.topk_keep(w, pct))
        s = {"layout": lay, "plan": plan, "x": buf(1)[0], "e": buf(K), "e_srv": buf(1)[0],
             "xh": buf(K), "m": buf(K) if mu else None, "g": buf(K),
             "sel": torch.zeros((K, W64), dtype=torch.int64, device="cuda"),
             "rank": torch.zeros((K, W64), dtype=torch.int32, device="cuda"),
             "vals": torch.zeros((K, plan.total), device="cuda"),
             "srv_sel": torch.zeros(W64, dtype=torch.int64, device="cuda"),
             "srv_rank": torch.zeros(W64, dtype=torch.int32, device="cuda"),
             "srv_vals": torch.zeros(plan.total, device="cuda")}
        s["x"][~pad] = torch.from_numpy(W.initial_x(w)).cuda()[~pad]
        return s

    a, b = state(), state()
    msg = ("sel", "rank", "vals", "srv_sel", "srv_rank", "srv_vals")
    for t in range(5):
        # the data scale falls and rises: thresholds inside and outside the lists
        g = torch.from_numpy(W.gradients(w, t) * np.float32([1, 1, 0.01, 30, 1][t])).cuda()
        for s in (a, b):
            s["g"][:, ~pad] = g[:, ~pad]
        S.saef_topk_round(a["plan"], t, w.period, K, w.lr, mu, mode, a["g"], a["m"], a["e"],
                          a["e_srv"], a["x"], a["xh"], *[a[k] for k in msg])
        S.saef_topk_round_begin(b["plan"], t, w.period, K, mode, S.VARIANT_SAEF, b["e"],
                                b["sel"], b["e_srv"], b["x"], b["xh"])
        S.saef_topk_round_end(b["plan"], t, w.period, K, w.lr, mu, mode, b["g"], b["m"], b["e"],
                              b["e_srv"], b["x"], *[b[k] for k in msg])
        for k in ("x", "e", "e_srv", "xh", "m", *msg):
            if a[k] is not None:
                bits = torch.int64 if a[k].dtype == torch.int64 else torch.int32
                assert torch.equal(a[k].view(bits), b[k].view(bits)), (k, t)
        assert S.saef_status(a["layout"]) == S.OK and S.saef_status(b["layout"]) == S.OK
