"""Small layouts, where the aggregation and the in-place corrections add up
the tile partials themselves, against the same tensors in a layout with one
more tensor of 65 tiles, where kernels of their own write the scales: messages
and states to the bit, at the edges of the rule (64 and 65 tiles in a tensor,
2048 and 2049 tiles, 16 and 17 workers)."""
import pytest
import torch

from paper_2008_05823_amd import workloads as W

pytestmark = pytest.mark.gpu

TILE = 2048
SIZES = {
    "small": [1, 64, 2049, 3 * TILE],
    "64_tiles": [64 * TILE, 5],
    "65_tiles": [64 * TILE + 1, 5],
    "2048_tiles": [7] * 2047 + [TILE],
    "2049_tiles": [7] * 2047 + [TILE + 1],
}


def _run(call, sizes, K, mode, x0, g0, pad):
    """State after two iterations of `sizes`, its layout longer by `pad`."""
    from paper_2008_05823_amd import saef as S
    w = W.custom(sizes + [pad] if pad else sizes, K=K, mode=mode)
    off, n, d_pad = w.layout()
    lay = S.Layout(off, n, d_pad, K)
    d0, L0 = x0.numel(), len(sizes)

    def zeros(r, cols=d_pad, dtype=torch.float32):
        return torch.zeros((r, cols), dtype=dtype, device="cuda")
    s = {"e": zeros(K), "e_srv": zeros(1)[0], "x": zeros(1)[0], "xh": zeros(K),
         "signs": zeros(K, d_pad // 64, torch.int64), "scales": zeros(K, w.L),
         "srv_signs": zeros(1, d_pad // 64, torch.int64)[0], "srv_scales": zeros(1, w.L)[0]}
    g = zeros(K)
    s["x"][:d0], g[:, :d0] = x0, g0
    msg = (s["signs"], s["scales"])
    srv = (s["srv_signs"], s["srv_scales"])
    for t in range(2):
        if call == "round":
            S.saef_round(lay, t, 0, K, w.lr, mode, g, s["e"], s["e_srv"], s["x"], s["xh"], *msg,
                         *srv)
        else:
            S.saef_step_ahead(lay, K, s["x"], s["e"], s["xh"])
            S.saef_compress(lay, K, w.lr, g, s["e"], *msg)
            S.saef_aggregate(lay, K, mode, *msg, s["x"], s["e_srv"], *srv)
    assert S.saef_status(lay) == S.OK
    cut = {"signs": d0 // 64, "srv_signs": d0 // 64, "scales": L0, "srv_scales": L0}
    return {k: v[..., :cut.get(k, d0)].clone() for k, v in s.items()}


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("call,K,mode", [("round", 1, 1), ("round", 5, 0), ("round", 16, 1),
                                         ("round", 17, 1), ("single", 3, 1), ("single", 16, 0),
                                         ("single", 17, 1)])
def test_folded_equals_finalized(sizes, call, K, mode):
    print(f"[case] {sizes} {call} K={K} mode={mode}", flush=True)
    w = W.custom(SIZES[sizes], K=K, mode=mode, scale_range=(1e-3, 1.0), seed=K + 3)
    x0 = torch.from_numpy(W.initial_x(w)).cuda()
    g0 = torch.from_numpy(W.gradients(w, 0)).cuda()
    a = _run(call, SIZES[sizes], K, mode, x0, g0, 0)
    b = _run(call, SIZES[sizes], K, mode, x0, g0, 65 * TILE)
    for k in a:
        assert torch.equal(a[k], b[k]), k
    assert (a["scales"] > 0).all()
