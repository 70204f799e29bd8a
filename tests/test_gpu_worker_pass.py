"""The one-pass worker step of saef_round (step ahead and compression from one
read of the errors) against the two halves, which run them as two kernels:
every byte of the state after every iteration, at the edges of words, waves,
tiles and runs of tiles."""
import pytest
import torch

from paper_2008_05823_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = {
    "tiny": [1, 3, 63, 64, 65],
    "tile_edges": [511, 512, 513, 1023, 1025, 2047, 2048, 2049, 4097],
    "runs": [2048 * 2050 + 77, 5],   # more than 2048 tiles: runs of 64 tiles
}


def _state(w, mu, shift):
    """Device state of workload w; `shift` elements past an aligned start."""
    from paper_2008_05823_amd import saef as S
    off, n, d_pad = w.layout()
    pad = torch.from_numpy(~W.tensor_mask(w)).cuda()

    def buf(rows):
        b = torch.zeros(rows * d_pad + shift, device="cuda")[shift:]
        b = b.view(rows, d_pad)
        b[:, pad] = float("nan")          # padding is neither read nor written
        return b

    s = {"S": S, "layout": S.Layout(off, n, d_pad, w.K), "pad": pad,
         "x": buf(1)[0], "e": buf(w.K), "e_srv": buf(1)[0], "xh": buf(w.K),
         "m": buf(w.K) if mu else None,
         "signs": torch.zeros((w.K, d_pad // 64), dtype=torch.int64, device="cuda"),
         "scales": torch.zeros((w.K, w.L), device="cuda"),
         "srv_signs": torch.zeros(d_pad // 64, dtype=torch.int64, device="cuda"),
         "srv_scales": torch.zeros(w.L, device="cuda"), "g": buf(w.K)}
    s["x"][~pad] = torch.from_numpy(W.initial_x(w)).cuda()[~pad]
    return s


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("K,mode,mu,shift", [(1, 1, 0.0, 0), (3, 1, 0.9, 1), (8, 1, 0.0, 3),
                                             (5, 0, 0.0, 0), (4, 0, 0.5, 2)])
def test_round_equals_halves(sizes, K, mode, mu, shift):
    print(f"[case] {sizes} K={K} mode={mode} mu={mu} shift={shift}", flush=True)
    w = W.custom(SIZES[sizes], K=K, period=3, mode=mode, scale_range=(1e-3, 1.0), seed=K + 11)
    a, b = _state(w, mu, shift), _state(w, mu, shift)
    S = a["S"]
    for t in range(5):
        g = torch.from_numpy(W.gradients(w, t)).cuda()
        for s in (a, b):
            s["g"][:, ~s["pad"]] = g[:, ~s["pad"]]
        tail = ("signs", "scales", "srv_signs", "srv_scales")
        if mu:
            S.saef_round_momentum(a["layout"], t, w.period, K, w.lr, mu, mode, a["g"], a["m"],
                                  a["e"], a["e_srv"], a["x"], a["xh"], *[a[k] for k in tail])
        else:
            S.saef_round(a["layout"], t, w.period, K, w.lr, mode, a["g"], a["e"], a["e_srv"],
                         a["x"], a["xh"], *[a[k] for k in tail])
        S.saef_round_begin(b["layout"], t, w.period, K, mode, S.VARIANT_SAEF, b["e"], b["e_srv"],
                           b["x"], b["xh"], *[b[k] for k in tail])
        S.saef_round_end(b["layout"], t, w.period, K, w.lr, mu, mode, b["g"], b["m"], b["e"],
                         b["e_srv"], b["x"], *[b[k] for k in tail])
        for k in ("x", "e", "e_srv", "xh", "m", *tail):
            if a[k] is not None:
                bits = torch.int64 if a[k].dtype == torch.int64 else torch.int32
                assert torch.equal(a[k].view(bits), b[k].view(bits)), (k, t)
        assert S.saef_status(a["layout"]) == S.OK and S.saef_status(b["layout"]) == S.OK
