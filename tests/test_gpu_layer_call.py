"""A layer forward as one library call against the same layer issued call by call: the same bits, top-1 and top-k, both dtypes, with the plan
from the routed ids and from others, both schedules, and the errors of the steps."""
import pytest
import torch

import oracle  # noqa: F401

pytestmark = pytest.mark.gpu


def _layer(dtype, k, T=300, d=128, F=256, E=16):
    import paper_2605_11537_amd as moe
    g = torch.Generator(device="cuda").manual_seed(5)
    rn = lambda *s: (torch.randn(s, generator=g, device="cuda") * 0.2).to(dtype)  # noqa: E731
    w1, w2 = rn(E, d, F), rn(E, F, d)
    if dtype == torch.bfloat16:
        w1, w2 = moe.moe_pack_weights(w1), moe.moe_pack_weights(w2)
    layer = moe.MoeLayer(T, d, F, E, 4, 20, dtype) if k == 0 else moe.MoeLayerTopK(T, d, F, E, k, 4, 20 * k, dtype, renormalize=True)
    return layer, (rn(T, d), rn(d, E), torch.zeros(E, device="cuda"), w1, w2)


def _poisoned(layer, out=None):
    """Every buffer that a forward writes holds something else."""
    for t in (*layer.route_out, *layer.plan_out.values(), *layer.disp_out.values(), layer.y_perm, layer.out, out):
        if t is not None:
            t.fill_(-9 if t.dtype == torch.int32 else float("nan"))


def _results(layer, out):
    K = int(layer.disp_out["expert_offset"][-1])
    tables = {k: v for k, v in {**layer.plan_out, **layer.disp_out}.items() if v is not None and k != "x_perm"}
    return {k: v.clone() for k, v in dict(out=out, idx=layer.route_out[0], prob=layer.route_out[1], y=layer.y_perm[:K], **tables).items()}


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("k", [0, 1, 3])
def test_one_call_equals_the_calls(dtype, k, monkeypatch):
    from paper_2605_11537_amd import binding
    layer, args = _layer(dtype, k)
    other = torch.randint(0, 16, (77,), dtype=torch.int32, device="cuda")
    ev = [torch.cuda.Event() for _ in range(5)]
    calls, one_call = [], binding._layer_forward
    monkeypatch.setattr(binding, "_layer_forward", lambda *a: calls.append(1) or one_call(*a))
    for kw in (dict(), dict(residual=1, schedule=1), dict(plan_ids=other), dict(plan_ids=other, out=torch.empty_like(args[0]))):
        got = []
        for how in (dict(), dict(marks=ev)):
            _poisoned(layer, kw.get("out"))
            got.append(_results(layer, layer.forward(*args, **kw, **how)))
        assert all(torch.equal(got[0][n], got[1][n]) for n in got[1])
        assert torch.isfinite(got[0]["out"].float()).all() and int(got[0]["idx"].min()) >= 0
    assert len(calls) == 4                                           # and none of the calls with marks


def test_plan_from_no_ids():
    """An empty prediction is one all the same: a slot per expert.  It goes call by call."""
    for k in (0, 2):
        layer, args = _layer(torch.bfloat16, k)
        _poisoned(layer)
        layer.forward(*args, plan_ids=torch.empty(0, dtype=torch.int32, device="cuda"))
        assert (layer.plan_out["replicas"] == 1).all() and (layer.plan_out["plan_counts"] == 0).all() and int(layer.plan_out["n_slots"]) == 16


def test_one_call_refuses_what_the_calls_refuse():
    import paper_2605_11537_amd as moe
    layer, args = _layer(torch.bfloat16, 0)
    with pytest.raises(ValueError):
        layer.forward(args[0].t().contiguous().t(), *args[1:])               # strides
    with pytest.raises(ValueError):
        layer.forward(args[0], args[1].float(), *args[2:])                   # router in another type
    with pytest.raises(ValueError):
        layer.forward(*args, out=torch.empty(args[0].shape, dtype=torch.bfloat16))   # not on the device
    for T in (0, 300):                                               # no choice at all
        none = moe.MoeLayerTopK(T, 128, 256, 16, 0, 4, 20, torch.bfloat16)
        with pytest.raises(moe.MoeError):
            none.forward(args[0][:T], *args[1:])
    layer.ffn_ws = layer.ffn_ws[:256]
    with pytest.raises(moe.MoeError, match="moe_expert_ffn: workspace"):
        layer.forward(*args)
