"""A top-1 layer whose second product makes the output: the same bits as the product and moe_combine by themselves, tokens without a
row included, in every kernel that does it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# dtype, T, d, F, E, R, capacity; the second product's kernel; whether it makes the output (a host test asks the library's rules for both)
CASES = [
    (("f32", 512, 64, 256, 8, 4, 80), "32 columns", True),
    (("f32", 33, 256, 256, 8, 2, 3), "32 columns", True),
    (("f32", 1, 64, 64, 4, 0, 1), "32 rows, short k", True),
    (("f32", 700, 256, 192, 5, 3, 90), "32 rows, short k", True),
    (("f32", 1500, 256, 256, 32, 8, 59), "32 rows, several units", True),
    (("f32", 1500, 256, 256, 4, 3, 260), "64 rows, several units", True),
    (("f32", 1500, 512, 512, 32, 8, 59), "32 rows, staged", True),
    (("f32", 1500, 512, 512, 4, 2, 300), "64 rows, staged", True),
    (("f32", 700, 128, 320, 16, 4, 40), "32 rows", True),
    (("f32", 900, 128, 320, 2, 4, 100), "64 rows", True),
    (("f32", 2048, 64, 256, 16, 0, 60), "64 rows, several units", True),            # the longest batches, most tokens without a row
    (("f32", 6000, 128, 256, 16, 2, 100), "64 rows, several units", True),
    (("f32", 6001, 128, 256, 16, 2, 100), "64 rows, several units", False),         # and layers whose output moe_combine makes
    (("f32", 2049, 64, 256, 16, 0, 60), "64 rows, several units", False),
    (("f32", 1200, 192, 256, 24, 0, 1), "32 rows, several units", True),            # next to all tokens without a row: 48 pieces in a row,
    (("f32", 900, 320, 320, 4, 0, 2), "64 rows", True),                             # 80,
    (("f32", 2048, 64, 192, 32, 0, 1), "32 rows, short k", True),                   # 16
    (("f32", 4096, 256, 256, 8, 0, 3), "64 rows, several units", True),             # the largest output
    (("f32", 4097, 256, 256, 8, 0, 3), "64 rows, several units", False),
    (("bf16", 37, 256, 1024, 64, 8, 4), "few rows", False),
    (("bf16", 1, 128, 256, 1, 0, 1), "columns", True),                              # a row,
    (("bf16", 200, 256, 384, 24, 3, 9), "columns", True),                           # tiles of 32 rows,
    (("bf16", 900, 128, 128, 16, 2, 56), "columns", True),                          # of 64
    (("bf16", 500, 256, 256, 9, 6, 200), "columns", True),                          # and 128 rows, slots of several tiles
    (("bf16", 1200, 1024, 4096, 16, 2, 90), "columns listed", True),                # weight streams with a work list
    (("bf16", 1500, 1024, 4096, 16, 0, 200), "columns listed", True),
    (("bf16", 1500, 128, 128, 64, 0, 20), "columns", True),                         # the longest batch, most tokens without a row
    (("bf16", 1100, 128, 256, 20, 0, 1), "columns", True),                          # next to all tokens without a row: 16 pieces in a row,
    (("bf16", 1000, 768, 768, 24, 0, 2), "columns", True),                          # 96
    (("bf16", 1501, 128, 128, 64, 0, 20), "columns", False),
    (("bf16", 700, 256, 512, 8, 0, 90), "lds", False),
]


@pytest.mark.parametrize("case", [c for c, _, _ in CASES], ids=lambda c: "-".join(str(v) for v in c))
def test_same_bits_as_the_calls(case):
    import paper_2605_11537_amd as moe
    name, T, d, F, E, R, C = case
    dt = dict(f32=torch.float32, bf16=torch.bfloat16)[name]
    g = torch.Generator(device="cuda").manual_seed(T + d)

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(dt)
    x, wr, b = rand(T, d), rand(d, E, std=0.1), torch.zeros(E, device="cuda")
    b[0] = 1.0
    w1, w2 = rand(E, d, F, std=0.05), rand(E, F, d, std=0.05)
    if dt == torch.bfloat16:
        w1, w2 = moe.moe_pack_weights(w1), moe.moe_pack_weights(w2)
    layer = moe.MoeLayer(T, d, F, E, R, C, dt)
    ev = [torch.cuda.Event() for _ in range(5)]
    for residual in (0, 1):
        for schedule in (0, 1):
            got = []
            for how in (dict(), dict(marks=ev)):                 # one call, call by call
                layer.y_perm.fill_(float("nan"))
                layer.out.fill_(float("nan"))
                out = layer.forward(x, wr, b, w1, w2, residual=residual, schedule=schedule, **how)
                kept = int(layer.disp_out["expert_offset"][-1])
                got.append((out.clone(), layer.y_perm[:kept].clone()))
            assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), (residual, schedule)
            dropped = layer.disp_out["inv"] < 0
            assert torch.equal(got[0][0][dropped], x[dropped])


def test_refused_output_is_an_error_behind_the_products():
    """Arguments of the last step are refused as it refuses them, with the steps before it enqueued."""
    import paper_2605_11537_amd as moe
    T, d, F, E = 64, 64, 64, 4
    layer = moe.MoeLayer(T, d, F, E, 0, T, torch.float32)
    x, wr, b = torch.randn(T, d, device="cuda"), torch.randn(d, E, device="cuda"), torch.zeros(E, device="cuda")
    w1, w2 = torch.randn(E, d, F, device="cuda"), torch.randn(E, F, d, device="cuda")
    layer.y_perm.fill_(float("nan"))
    with pytest.raises(moe.MoeError, match="moe_combine: out aliases"):
        layer.forward(x, wr, b, w1, w2, out=x)
    assert torch.isfinite(layer.y_perm).all()


@pytest.mark.parametrize("dt,T,d,F,E,R,C", [(torch.float32, 512, 64, 256, 8, 4, 80), (torch.float32, 1500, 256, 256, 4, 3, 260),
                                            (torch.bfloat16, 200, 256, 384, 24, 3, 9), (torch.bfloat16, 1500, 128, 128, 64, 0, 20)])
def test_output_in_what_the_products_read(dt, T, d, F, E, R, C):
    """An output in the products' workspace or in the second weights, which a caller with no more use for them may name: as that of the calls."""
    import paper_2605_11537_amd as moe
    g = torch.Generator(device="cuda").manual_seed(T)

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, generator=g, device="cuda") * std).to(dt)
    x, wr, b = rand(T, d), rand(d, E, std=0.1), torch.zeros(E, device="cuda")
    w1, w2 = rand(E, d, F, std=0.05), rand(E, F, d, std=0.05)
    if dt == torch.bfloat16:
        w1, w2 = moe.moe_pack_weights(w1), moe.moe_pack_weights(w2)
    layer = moe.MoeLayer(T, d, F, E, R, C, dt)
    want = layer.forward(x, wr, b, w1, w2, marks=[torch.cuda.Event() for _ in range(5)]).clone()
    in_ws = layer.ffn_ws[: T * d * want.element_size()].view(dt).view(T, d)
    assert torch.equal(layer.forward(x, wr, b, w1, w2, out=in_ws), want)
    last = w2.clone()
    if last.numel() >= T * d:
        assert torch.equal(layer.forward(x, wr, b, w1, last, out=last.view(-1)[-T * d:].view(T, d)), want)
