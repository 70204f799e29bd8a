"""Arguments of the whole-iteration calls: one that an iteration's second half
refuses is refused before anything is enqueued, on averaging iterations and for
plans that are not pipelined as well."""
import pytest
import torch

from paper_2008_05823_amd import workloads as W

pytestmark = pytest.mark.gpu


def _topk_state(w, pct):
    from paper_2008_05823_amd import saef as S
    off, n, d_pad = w.layout()
    K, W64 = w.K, d_pad // 64
    lay = S.Layout(off, n, d_pad, K)
    plan = S.TopK(lay, W.topk_keep(w, pct))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda")
    s = {"x": rnd(d_pad), "e": rnd(K, d_pad), "e_srv": rnd(d_pad), "xh": rnd(K, d_pad),
         "g": rnd(K, d_pad), "sel": torch.zeros((K, W64), dtype=torch.int64, device="cuda"),
         "rank": torch.zeros((K, W64), dtype=torch.int32, device="cuda"),
         "vals": rnd(K, plan.total),
         "srv_sel": torch.zeros(W64, dtype=torch.int64, device="cuda"),
         "srv_rank": torch.zeros(W64, dtype=torch.int32, device="cuda"),
         "srv_vals": rnd(plan.total)}
    return S, lay, plan, s


@pytest.mark.parametrize("sizes", [[5000], [5000, 70, 4097]])
@pytest.mark.parametrize("period", [0, 1])
@pytest.mark.parametrize("call", ["round", "end"])
@pytest.mark.parametrize("wrong", ["srv_vals", "srv_sel", "e_srv"])
def test_refused_before_anything_is_enqueued(sizes, period, call, wrong):
    print(f"[case] {sizes} period={period} {call} {wrong}", flush=True)
    w = W.custom(sizes, K=2, period=period, seed=3)
    S, lay, plan, s = _topk_state(w, 5)
    before = {k: v.clone() for k, v in s.items()}
    a = dict(s, **{wrong: None})
    with pytest.raises(S.SaefError) as err:
        if call == "round":
            S.saef_topk_round(plan, 1, period, 2, 0.1, 0.0, S.MODE_DC, a["g"], None, a["e"],
                              a["e_srv"], a["x"], a["xh"], a["sel"], a["rank"], a["vals"],
                              a["srv_sel"], a["srv_rank"], a["srv_vals"])
        else:
            S.saef_topk_round_end(plan, 1, period, 2, 0.1, 0.0, S.MODE_DC, a["g"], None, a["e"],
                                  a["e_srv"], a["x"], a["sel"], a["rank"], a["vals"],
                                  a["srv_sel"], a["srv_rank"], a["srv_vals"])
    assert err.value.rc == S.EINVAL
    assert S.saef_status(lay) == S.OK
    for k, v in s.items():
        assert torch.equal(v, before[k]), k
