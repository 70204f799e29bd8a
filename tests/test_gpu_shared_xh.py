"""An xh that shares its address range with a message (the message lies in the
padding between xh's rows): the step ahead then runs as a kernel of its own
before the compression.  Every byte as with buffers apart."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [5000, 70, 4097, 1]


def _sizes():
    """Offsets, sizes, the elements they take and a d_pad twice that."""
    off, at = [], 0
    for v in SIZES:
        off.append(at)
        at += (v + 63) // 64 * 64
    return off, at, 2 * at


def _xh(K, used, d_pad, kind):
    """xh (K, d_pad) and, per name in `kind`, a tensor inside its padding."""
    flat = torch.zeros(K * d_pad, device="cuda")
    at, inside = used, {}
    for name, shape, dtype in kind:
        size = torch.Size(shape).numel() * torch.empty(0, dtype=dtype).element_size() // 4
        at += at % 2
        assert at + size <= d_pad
        inside[name] = flat[at:at + size].view(dtype).view(shape)
        at += size
    return flat.view(K, d_pad), inside


@pytest.mark.parametrize("shared", ["signs", "scales", "srv_signs", "srv_scales"])
@pytest.mark.parametrize("mu", [0.0, 0.9])
def test_sign_round(shared, mu):
    from paper_2008_05823_amd import saef as S
    print(f"[case] sign {shared} mu={mu}", flush=True)
    K, L = 3, len(SIZES)
    off, used, d_pad = _sizes()
    msgs = [("signs", (K, d_pad // 64), torch.int64), ("scales", (K, L), torch.float32),
            ("srv_signs", (d_pad // 64,), torch.int64), ("srv_scales", (L,), torch.float32)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    x0 = torch.randn(d_pad, generator=gen, device="cuda")
    gs = [torch.randn((K, d_pad), generator=gen, device="cuda") for _ in range(5)]
    states = []
    for inside in ([], [m for m in msgs if m[0] == shared]):
        s = {n: torch.zeros(sh, dtype=dt, device="cuda") for n, sh, dt in msgs}
        s["xh"], part = _xh(K, used, d_pad, inside)
        s.update(part)
        s.update(lay=S.Layout(off, SIZES, d_pad, K), x=x0.clone(),
                 e=torch.zeros((K, d_pad), device="cuda"), e_srv=torch.zeros(d_pad, device="cuda"),
                 m=torch.zeros((K, d_pad), device="cuda"))
        states.append(s)
    for t, g in enumerate(gs):
        for s in states:
            rest = (s["x"], s["xh"], s["signs"], s["scales"], s["srv_signs"], s["srv_scales"])
            if mu:
                S.saef_round_momentum(s["lay"], t, 4, K, 0.1, mu, S.MODE_DC, g, s["m"], s["e"],
                                      s["e_srv"], *rest)
            else:
                S.saef_round(s["lay"], t, 4, K, 0.1, S.MODE_DC, g, s["e"], s["e_srv"], *rest)
        a, b = states
        for k in ("x", "e", "e_srv", "m", "signs", "scales", "srv_signs", "srv_scales"):
            assert torch.equal(a[k], b[k]), (k, t)
        assert torch.equal(a["xh"][:, :used], b["xh"][:, :used]), t
        assert S.saef_status(a["lay"]) == S.OK and S.saef_status(b["lay"]) == S.OK


@pytest.mark.parametrize("shared", ["rank", "vals", "srv_sel", "srv_rank", "srv_vals", "m"])
def test_topk_round(shared):
    from paper_2008_05823_amd import saef as S
    print(f"[case] top-k {shared}", flush=True)
    K, mu = 3, 0.9
    off, used, d_pad = _sizes()
    keep = [max(1, v // 20) for v in SIZES]
    W64, total = d_pad // 64, sum(keep)
    i32, i64, f32 = torch.int32, torch.int64, torch.float32
    msgs = [("sel", (K, W64), i64), ("rank", (K, W64), i32), ("vals", (K, total), f32),
            ("srv_sel", (W64,), i64), ("srv_rank", (W64,), i32), ("srv_vals", (total,), f32)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    x0 = torch.randn(d_pad, generator=gen, device="cuda")
    gs = [torch.randn((K, d_pad), generator=gen, device="cuda") for _ in range(5)]
    states = []
    for inside in ([], [m for m in msgs if m[0] == shared]):
        s = {n: torch.zeros(sh, dtype=dt, device="cuda") for n, sh, dt in msgs}
        s["xh"], part = _xh(K, used, d_pad, inside)
        s.update(part)
        lay = S.Layout(off, SIZES, d_pad, K)
        s.update(lay=lay, plan=S.TopK(lay, keep), x=x0.clone(),
                 e=torch.zeros((K, d_pad), device="cuda"), e_srv=torch.zeros(d_pad, device="cuda"),
                 m=torch.zeros((K, d_pad), device="cuda"))
        states.append(s)
    if shared == "m":   # the rows of m in the padding of the rows of xh
        both = torch.zeros(K * d_pad + used, device="cuda")
        states[1]["xh"] = both[:K * d_pad].view(K, d_pad)
        states[1]["m"] = both[used:].view(K, d_pad)
    for t, g in enumerate(gs):
        for s in states:
            S.saef_topk_round(s["plan"], t, 4, K, 0.1, mu, S.MODE_DC, g, s["m"], s["e"],
                              s["e_srv"], s["x"], s["xh"], *[s[n] for n, _, _ in msgs])
        a, b = states
        for k in ("x", "e", "e_srv", *[n for n, _, _ in msgs]):
            assert torch.equal(a[k], b[k]), (k, t)
        for k in ("xh", "m"):
            assert torch.equal(a[k][:, :used], b[k][:, :used]), (k, t)
        assert S.saef_status(a["lay"]) == S.OK and S.saef_status(b["lay"]) == S.OK
