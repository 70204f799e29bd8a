"""Top-K plans whose thresholds jump from one call to the next: values scaled up
and down, first calls, rows first used late, bins full of equal values.  The kept
set against a stable sort of the magnitudes, at the sizes where the selection
takes another way (16, 20 and 64 tiles; plans that are split over two streams;
more than 4096 tiles), and the time of such a call against one that finds its
threshold where the last call left it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TILE = 2048
PLANS = {                                      # (tensor sizes, workers)
    "small": ([16 * TILE, 20 * TILE, 1, 100], 3),
    "wide": ([20 * TILE + 1, 64 * TILE, 2047], 3),
    "large": ([64 * TILE + 1, 16 * TILE, 17 * TILE - 5, 1025 * TILE + 3], 2),
    "many_pairs": ([18 * TILE] * 100, 3),      # 256 (row, tensor)s and more
    "split": ([2100 * TILE + 9, 700 * TILE, 16 * TILE], 6),   # over two streams
    "huge": ([4097 * TILE + 3, 65 * TILE], 2),
}
SCALES = (1.0, 4.0, 0.25, 16.0, 1 / 16, 1000.0, 1e-3, 2.0, 0.5)


class _Plan:
    def __init__(self, sizes, K, pct):
        from paper_2008_05823_amd import saef as S
        self.S, self.n, self.K = S, sizes, K
        self.off, self.d_pad = [], 0
        for v in sizes:
            self.off.append(self.d_pad)
            self.d_pad += (v + 63) // 64 * 64
        self.keep = [max(1, int(np.ceil(v * pct / 100))) for v in sizes]
        W64 = self.d_pad // 64
        self.layout = S.Layout(self.off, sizes, self.d_pad, K)
        self.plan = S.TopK(self.layout, self.keep)
        dev = {"device": "cuda"}
        self.sel = torch.zeros((K, W64), dtype=torch.int64, **dev)
        self.rank = torch.zeros((K, W64), dtype=torch.int32, **dev)
        self.vals = torch.zeros((K, self.plan.total), **dev)
        self.zero = torch.zeros((K, self.d_pad), **dev)
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(41)

    def values(self, kind="normal"):
        v = torch.randn((self.K, self.d_pad), generator=self.gen, device="cuda")
        if kind == "ties":       # 30% at one magnitude, the rest smaller
            v = torch.where(torch.rand(v.shape, generator=self.gen, device="cuda") < 0.3,
                            v.sign() * 7.0, v / 8)
        return v

    def compress(self, e, rows=None):
        r = self.K if rows is None else rows
        self.S.saef_topk_compress(self.plan, r, 0.0, 0.0, self.zero[:r], None, e[:r], self.sel[:r],
                                  self.rank[:r], self.vals[:r])

    def check(self, before, after, sel, rank, vals):
        rows = before.shape[0]
        bits = ((sel.view(torch.uint8).reshape(rows, -1, 1) >>
                 torch.arange(8, dtype=torch.uint8, device="cuda")) & 1).reshape(rows, -1).bool()
        at = 0
        for o, v, q in zip(self.off, self.n, self.keep):
            for k in range(rows):
                x = before[k, o:o + v]
                want = torch.sort(x.abs(), descending=True, stable=True).indices[:q].sort().values
                assert torch.equal(bits[k, o:o + v].nonzero()[:, 0], want)
                assert torch.equal(vals[k, at:at + q], x[want])
                cnt = bits[k, o:o + (v + 63) // 64 * 64].view(-1, 64).sum(1)
                assert torch.equal(rank[k, o // 64:o // 64 + cnt.numel()].long(),
                                   torch.cumsum(cnt, 0) - cnt)
                left = x.clone()
                left[want] = 0.0
                assert torch.equal(after[k, o:o + v], left)
            at += q


@pytest.mark.parametrize("plan", PLANS)
@pytest.mark.parametrize("pct", [1.0, 10.0, 30.0])
def test_kept_set(plan, pct):
    sizes, K = PLANS[plan]
    p = _Plan(sizes, K, pct)
    base = p.values()
    steps = [(f"{s:g}", base * s) for s in SCALES]
    steps += [("ties", p.values("ties")), ("1", base)]
    steps += [("per row", base * (64.0 ** torch.arange(K, device="cuda"))[:, None])]
    # a few rows first, the others later on the same plan
    for tag, v in [("rows", base), ("rows", base * 3)]:
        e = v.clone()
        p.compress(e, rows=1)
        p.check(v[:1], e[:1], p.sel[:1], p.rank[:1], p.vals[:1])
    for tag, v in steps:
        print(f"[case] {plan} pct={pct} {tag}", flush=True)
        e = v.clone()
        p.compress(e)
        p.check(v, e, p.sel, p.rank, p.vals)
    assert p.S.saef_status(p.layout) == p.S.OK


@pytest.mark.parametrize("plan", PLANS)
def test_server_row(plan):
    """The server's first selection after several worker calls, then jumps."""
    sizes, K = PLANS[plan]
    p = _Plan(sizes, K, 2.0)
    W64, total = p.d_pad // 64, p.plan.total
    ss = torch.zeros((1, W64), dtype=torch.int64, device="cuda")
    sr = torch.zeros((1, W64), dtype=torch.int32, device="cuda")
    sv = torch.zeros((1, total), device="cuda")
    base, es0 = p.values(), p.values()[:1] * 0.3
    for _ in range(3):
        p.compress(base.clone())
    for s in (1.0, 1000.0, 1e-3, 4.0, 0.25):
        print(f"[case] {plan} server {s:g}", flush=True)
        p.compress(base * s)
        es = es0 * s
        # the sum that the server forms: the mean over the workers in binary64
        mean = torch.zeros(p.d_pad, dtype=torch.float64, device="cuda")
        for k in range(K):
            at = 0
            bits = ((p.sel[k].view(torch.uint8).reshape(-1, 1) >>
                     torch.arange(8, dtype=torch.uint8, device="cuda")) & 1).reshape(-1).bool()
            for o, v, q in zip(p.off, p.n, p.keep):
                mean[o:o + v][bits[o:o + v]] += p.vals[k, at:at + q].double()
                at += q
        before = es + (mean / K).float()
        x = torch.zeros(p.d_pad, device="cuda")
        p.S.saef_topk_aggregate(p.plan, K, p.S.MODE_DC, p.sel, p.rank, p.vals, x, es[0], ss[0],
                                sr[0], sv[0])
        p.check(before, es, ss, sr, sv)
    assert p.S.saef_status(p.layout) == p.S.OK


def _us(f):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    a.record()
    f()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) * 1e3


# Bounds: measured 2.0-2.7 (large, split) and 4.0-4.5 (one small tensor, whose warm
# call takes 25 us); a single workgroup that radix-selects among all elements
# of a tensor takes 20 to 50 and 15 to 21 times the warm call.
@pytest.mark.parametrize("sizes,K,bound", [([1024 * TILE + 77], 2, 7.0),
                                           ([3000 * TILE, 300 * TILE], 8, 7.0),
                                           ([64 * TILE], 1, 9.0)])
def test_time_of_a_jump(sizes, K, bound):
    p = _Plan(sizes, K, 1.0)
    base = p.values()
    e = torch.empty_like(base)

    def call(v, q=p):
        e.copy_(v)
        return _us(lambda: q.compress(e))
    for _ in range(4):
        call(base)
    warm = min(call(base) for _ in range(5))
    took = {}
    for s in (1000.0, 1e-3, 16.0, 1 / 16):
        took[f"{s:g}"] = min(max(0.0, (call(base), call(base), call(base * s))[2])
                             for _ in range(3))
    took["first call"] = min(call(base, _Plan(sizes, K, 1.0)) for _ in range(3))
    if K > 1:
        late = []
        for _ in range(3):
            q = _Plan(sizes, K, 1.0)
            for _ in range(3):
                e.copy_(base)
                q.compress(e, rows=1)
            late.append(call(base, q))
        took["rows used late"] = min(late)
    print(f"[case] {sizes} K={K}: warm {warm:.0f} us,",
          {k: f"{v:.0f}" for k, v in took.items()}, flush=True)
    assert all(v < bound * warm for v in took.values()), (warm, took)
