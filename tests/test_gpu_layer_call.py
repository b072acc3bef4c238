"""A layer forward as one library call against the same layer issued call by call: the same bits, top-1 and top-k, both dtypes, with the plan
from the routed ids, from others and from none, both schedules, and the errors of the steps."""
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


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("k", [0, 1, 3])
def test_one_call_equals_the_calls(dtype, k):
    layer, args = _layer(dtype, k)
    other = torch.randint(0, 16, (77,), dtype=torch.int32, device="cuda")
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    ev = [torch.cuda.Event() for _ in range(5)]
    for kw in (dict(), dict(residual=1, schedule=1), dict(plan_ids=other), dict(plan_ids=none, out=torch.empty_like(args[0]))):
        got = layer.forward(*args, **kw).clone()
        ids, inv = layer.route_out[0].clone(), layer.disp_out["inv"].clone()
        ref = layer.forward(*args, marks=ev, **kw)
        assert torch.equal(got, ref) and torch.equal(ids, layer.route_out[0]) and torch.equal(inv, layer.disp_out["inv"])


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
