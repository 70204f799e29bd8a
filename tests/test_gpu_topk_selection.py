"""The Top-K selection at the sizes and data where its kernels differ: tensors of
one tile, of one group of tiles and just past it, of more tiles than the LDS
counts hold and of more than 4096 tiles (the refined ranges); values that are
mostly equal (ties by index), clustered at the cut, all zero, or spread; every
kept index, value and rank against a stable sort of the magnitudes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TILE = 2048
SIZES = {
    "one_tile": [1, 64, 100, 2047, 2048],
    "one_group": [2049, 64 * TILE - 1, 64 * TILE],
    "large": [64 * TILE + 1, 80 * TILE + 5, 300 * TILE],
    "many_tiles": [2048 * TILE + 1, 130 * TILE],
    "huge": [4097 * TILE + 3, 65 * TILE, 5],
}
DATA = ("spread", "ties", "clusters", "zeros")


def _values(kind, n, gen):
    v = torch.randn(n, generator=gen, device="cuda")
    u = torch.rand(n, generator=gen, device="cuda")
    if kind == "ties":          # 3% at one magnitude, the rest small and repeated
        v = torch.where(u < 0.03, torch.sign(v) * 7.0, torch.round(v * 4) / 1024)
    elif kind == "clusters":    # 1% near 100, the rest near 1
        v = torch.where(u < 0.01, v.sign() * (100 + v.abs()), v)
    elif kind == "zeros":
        v = torch.where(u < 0.9, 0.0 * v, torch.full_like(v, 2.0))
    return v


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("pct", [0.1, 1.0, 2.0, 40.0])
@pytest.mark.parametrize("K", [1, 3])
def test_selection(sizes, pct, K):
    from paper_2008_05823_amd import saef as S
    n = SIZES[sizes]
    off, d_pad = [], 0
    for v in n:
        off.append(d_pad)
        d_pad += (v + 63) // 64 * 64
    keep = [max(1, int(np.ceil(v * pct / 100))) for v in n]
    W64 = d_pad // 64
    lay = S.Layout(off, n, d_pad, K)
    plan = S.TopK(lay, keep)
    sel = torch.zeros((K, W64), dtype=torch.int64, device="cuda")
    rank = torch.zeros((K, W64), dtype=torch.int32, device="cuda")
    vals = torch.zeros((K, plan.total), device="cuda")
    zero = torch.zeros((K, d_pad), device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    # each data set twice: without and with the previous call's threshold
    for step, kind in enumerate(("spread", "spread", "ties", "ties", "clusters", "zeros",
                                 "zeros", "clusters", "spread")):
        print(f"[case] {sizes} pct={pct} K={K} step={step} {kind}", flush=True)
        e = torch.full((K, d_pad), float("nan"), device="cuda")
        for o, v in zip(off, n):
            for k in range(K):
                e[k, o:o + v] = _values(kind, v, gen)
        before = e.clone()
        S.saef_topk_compress(plan, K, 0.0, 0.0, zero, None, e, sel, rank, vals)
        bits = ((sel.view(torch.uint8).reshape(K, -1, 1) >>
                 torch.arange(8, dtype=torch.uint8, device="cuda")) & 1).reshape(K, d_pad).bool()
        at = 0
        for o, v, q in zip(off, n, keep):
            for k in range(K):
                x = before[k, o:o + v]
                want = torch.sort(x.abs(), descending=True, stable=True).indices[:q].sort().values
                got = bits[k, o:o + v].nonzero()[:, 0]
                assert torch.equal(got, want), (kind, step, o, v, k)
                assert torch.equal(vals[k, at:at + q], x[want])
                cnt = bits[k, o:o + (v + 63) // 64 * 64].view(-1, 64).sum(1)
                first = torch.cumsum(cnt, 0) - cnt
                assert torch.equal(rank[k, o // 64:o // 64 + cnt.numel()].long(), first)
                left = x.clone()
                left[want] = 0.0
                assert torch.equal(e[k, o:o + v], left)
            at += q
        assert S.saef_status(lay) == S.OK
