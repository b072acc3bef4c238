"""Row movement at the edges of its trips: rows of one piece up to just over one trip, a ragged last workgroup, and
outputs on both sides of the size from which they are written past the caches."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(T, d, dtype, k, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(T, d, device="cuda", generator=g).to(dtype)
    y = torch.randn(k * T, d, device="cuda", generator=g).to(dtype)
    inv = torch.randperm(k * T, device="cuda", generator=g).to(torch.int32)
    inv[torch.rand(k * T, device="cuda", generator=g) < 0.3] = -1
    p = torch.rand(k * T, device="cuda", generator=g)
    return x, y, inv.view(k, T), p.view(k, T)


@pytest.mark.parametrize("residual", [0, 1])
@pytest.mark.parametrize("T,d,dtype", [
    (1, 8, torch.bfloat16), (17, 768, torch.bfloat16), (33, 776, torch.bfloat16), (100, 248, torch.float32),
    (1000, 8, torch.bfloat16), (333, 24, torch.bfloat16), (2500, 72, torch.bfloat16), (130, 132, torch.float32),   # 1, 3, 9, 33 pieces
    (2049, 264, torch.bfloat16), (2049, 4096, torch.bfloat16), (7, 8200, torch.bfloat16),    # more rows: 32 lanes; 256 lanes
    (43688, 768, torch.bfloat16), (43691, 768, torch.bfloat16),      # 64 MiB are 43690.7 such rows
])
def test_rows(T, d, dtype, residual):
    import paper_2605_11537_amd as moe
    x, y, inv, p = _case(T, d, dtype, 1, T + d)
    out = moe.moe_combine(y, x, inv[0], p[0], residual)
    kept = inv[0] >= 0
    # in binary64, rounded once: the kernel's one rounding of a binary32 multiply-add can differ by one unit in the last place
    ref = x.double()
    yk = y.double()[inv[0].clamp(min=0).long()]
    ref[kept] = (ref[kept] if residual else 0.0) + p[0][kept, None].double() * yk[kept]
    ulp = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    assert torch.equal(out[~kept], x[~kept])
    mag = (x.double().abs() if residual else 0.0) + p[0][:, None].double() * yk.abs()
    assert ((out.double() - ref).abs() <= ulp * ref.abs() + 2.0 ** -23 * mag).all()
    # the row copy
    ids = torch.randint(0, 7, (T,), device="cuda", dtype=torch.int32)
    o = moe.moe_dispatch(x, ids, None, 7, max(1, T // 9), 7)
    K = int(o["expert_offset"][7])
    assert torch.equal(o["x_perm"][:K], x[o["perm"][:K].long()])


@pytest.mark.parametrize("residual", [0, 1])
@pytest.mark.parametrize("T,d,dtype,k", [
    (17, 776, torch.bfloat16, 3), (9, 8, torch.bfloat16, 8), (50, 392, torch.float32, 2), (777, 40, torch.bfloat16, 2),
    (2049, 264, torch.bfloat16, 2), (4097, 264, torch.bfloat16, 3), (3, 4104, torch.bfloat16, 2),
])
def test_rows_topk(T, d, dtype, k, residual):
    import paper_2605_11537_amd as moe
    x, y, inv, p = _case(T, d, dtype, k, T * k)
    out = moe.moe_combine_topk(y, x, inv, p, residual)
    acc = x.double() if residual else torch.zeros(T, d, dtype=torch.float64, device="cuda")
    mag = acc.abs()
    for j in range(k):
        t = torch.where((inv[j] >= 0)[:, None], p[j][:, None].double() * y.double()[inv[j].clamp(min=0).long()], 0.0)
        acc, mag = acc + t, mag + t.abs()
    none = (inv < 0).all(0)
    assert torch.equal(out[none], x[none])
    ulp = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    assert ((out.double() - acc).abs() <= ulp * acc.abs() + (k + 1) * 2.0 ** -23 * mag)[~none].all()


def test_rows_past_one_grid_dimension():
    """More rows than 2^32 threads hold at 32 per row: short rows, some dropped."""
    import paper_2605_11537_amd as moe
    T, d, n_y = (1 << 27) + 5, 8, 1000
    x = torch.arange(T, device="cuda", dtype=torch.int32).remainder_(251).to(torch.bfloat16)[:, None].expand(T, d).contiguous()
    y = torch.arange(n_y * d, device="cuda", dtype=torch.float32).remainder_(127).to(torch.bfloat16).view(n_y, d)
    inv = torch.arange(T, device="cuda", dtype=torch.int32).remainder_(n_y + 1).sub_(1)
    one = torch.ones(T, device="cuda")
    ref = torch.cat([torch.zeros(1, d, dtype=torch.bfloat16, device="cuda"), y])
    for k, out in ((1, moe.moe_combine(y, x, inv, one)),
                   (2, moe.moe_combine_topk(y, x, torch.stack([inv, torch.full_like(inv, -1)]), torch.stack([one, one])))):
        for lo in (0, T // 2, T - 100000):
            i = inv[lo:lo + 100000].long()
            want = torch.where((i < 0)[:, None], x[lo:lo + 100000], ref[i + 1])
            assert torch.equal(out[lo:lo + 100000], want), (k, lo)
