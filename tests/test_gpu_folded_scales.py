"""The iteration whose aggregation adds up the worker partials itself (small
layouts) against the single calls, which finalize the scales in a kernel of
their own: messages and server state to the bit, at the edges of the rule (64
and 65 tiles in a tensor, 2048 and 2049 tiles, 16 and 17 workers)."""
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


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("K,mode", [(1, 1), (5, 0), (16, 1), (17, 1)])
def test_round_equals_single_calls(sizes, K, mode):
    print(f"[case] {sizes} K={K} mode={mode}", flush=True)
    from paper_2008_05823_amd import saef as S
    w = W.custom(SIZES[sizes], K=K, mode=mode, scale_range=(1e-3, 1.0), seed=K + 3)
    off, n, d_pad = w.layout()
    lay = S.Layout(off, n, d_pad, K)
    rows = lambda r: torch.zeros((r, d_pad), device="cuda")
    x = torch.from_numpy(W.initial_x(w)).cuda()
    g = torch.from_numpy(W.gradients(w, 0)).cuda()
    words = lambda r: torch.zeros((r, d_pad // 64), dtype=torch.int64, device="cuda")

    def state():
        return {"e": rows(K), "e_srv": rows(1)[0], "x": x.clone(), "signs": words(K),
                "scales": torch.full((K, w.L), -1.0, device="cuda"), "srv_signs": words(1)[0],
                "srv_scales": torch.full((w.L,), -1.0, device="cuda")}
    a, b = state(), state()
    S.saef_round(lay, 0, 0, K, w.lr, mode, g, a["e"], a["e_srv"], a["x"], rows(K), a["signs"],
                 a["scales"], a["srv_signs"], a["srv_scales"])
    S.saef_compress(lay, K, w.lr, g, b["e"], b["signs"], b["scales"])
    S.saef_aggregate(lay, K, mode, b["signs"], b["scales"], b["x"], b["e_srv"], b["srv_signs"],
                     b["srv_scales"])
    keys = ["signs", "scales"] + (["srv_signs", "srv_scales"] if mode else ["x"])
    for k in keys:
        assert torch.equal(a[k], b[k]), k
    assert (a["scales"] >= 0).all()
    assert S.saef_status(lay) == S.OK
