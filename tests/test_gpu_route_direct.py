"""moe_route / moe_route_topk on the shapes that take the router matrix as it lies (binary32, or an expert count /
width the packed kernels do not have): ragged token tiles, d that is no multiple of a matrix step, every number of
columns per lane, more experts than one column group, k up to the limit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f64, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,dtype,k", [
    (1, 8, 1, synth.BF16, 1),            # the smallest: half a matrix step, one expert
    (1, 8, 1, synth.F32, 1),
    (33, 24, 33, synth.BF16, 1),         # odd E: one column per lane, two groups; last step half empty
    (33, 24, 33, synth.F32, 2),
    (65, 40, 34, synth.BF16, 3),         # two columns per lane
    (31, 72, 66, synth.BF16, 1),         # two columns per lane, two groups
    (31, 72, 66, synth.F32, 3),
    (64, 136, 100, synth.BF16, 8),       # four columns per lane, part of the lanes past E
    (64, 136, 100, synth.F32, 1),
    (45, 200, 256, synth.BF16, 2),       # eight columns per lane (d is no multiple of 128)
    (45, 776, 256, synth.F32, 2),        # eight columns, binary32, many steps
    (40, 104, 1024, synth.BF16, 8),      # the most experts: four groups
    (40, 104, 1024, synth.F32, 1),
    (37, 48, 1023, synth.F32, 2),        # odd and over one group
])
def test_route_direct(T, d, E, dtype, k):
    import paper_2605_11537_amd as moe
    x = synth.normal_tensor((T, d), 1.0, [171, T, d], dtype)
    wr = synth.normal_tensor((d, E), 0.3, [172, E, d], dtype)
    b = (np.random.default_rng(E).standard_normal(E) * 0.1).astype(np.float32)
    ref = f64(x) @ f64(wr) + b.astype(np.float64)
    # a sum of d products in binary32, in any order: each of the d + 1 roundings is at most 2^-24 of the sum of magnitudes
    bound = (d + 2) * 2.0 ** -24 * (np.abs(f64(x)) @ np.abs(f64(wr)) + np.abs(b)).max()
    if k == 1:
        idx, prob, logits = moe.moe_route(to_dev(x), to_dev(wr), to_dev(b), want_logits=True)
        idx, prob = idx.view(1, T), prob.view(1, T)
    else:
        idx, prob, logits = moe.moe_route_topk(to_dev(x), to_dev(wr), to_dev(b), k, False, want_logits=True)
    got = to_host(logits)
    assert np.abs(got - ref).max() <= bound
    # ids and weights follow from the kernel's own logits: largest first, the lower id first among equals
    order = np.argsort(-got.astype(np.float64), axis=1, kind="stable")[:, :k].T
    assert (to_host(idx) == order).all()
    z = np.exp(got.astype(np.float64) - got.max(axis=1, keepdims=True))
    p = (z / z.sum(axis=1, keepdims=True))[np.arange(T)[None, :], order]
    assert np.abs(to_host(prob) / p - 1).max() <= 2e-6 + E * 2.0 ** -24


# the packed kernel's tiles: 128 / 256 experts x 32 / 64 tokens (above 8192), k chunks of 64, or of 128 where d has two and more
@pytest.mark.parametrize("T,d,E,k", [
    (1, 128, 128, 1),
    (33, 256, 128, 2),
    (31, 384, 128, 1),                   # an odd number of deep chunks
    (8193, 128, 128, 3),
    (8193, 384, 128, 1),
    (31, 128, 256, 2),
    (8192, 640, 256, 1),
    (8193, 128, 256, 1),                 # one row past the last full tile
    (16415, 384, 256, 3),
])
def test_route_packed_tiles(T, d, E, k):
    test_route_direct(T, d, E, synth.BF16, k)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
def test_route_direct_specials(dtype):
    """An infinite bias, a token with a NaN and a token of subnormal size: each stays in its own row or column."""
    import paper_2605_11537_amd as moe
    T, d, E = 40, 32, 48
    x = torch.from_numpy(f64(synth.normal_tensor((T, d), 1.0, [5], dtype)).astype(np.float32))
    w = torch.from_numpy(f64(synth.normal_tensor((d, E), 0.3, [6], dtype)).astype(np.float32))
    x[7, 3] = float("nan")
    x[9] = 0.0
    x[9, 4] = 2.0 ** -130                                   # subnormal in both formats
    w[4] *= 0.0
    w[4, 11] = 2.0 ** 20
    b = torch.zeros(E)
    b[2] = float("-inf")
    t = torch.bfloat16 if dtype == synth.BF16 else torch.float32
    idx, prob, logits = moe.moe_route(x.cuda().to(t), w.cuda().to(t), b.cuda(), want_logits=True)
    lg = logits.cpu()
    assert torch.isnan(lg[7, 3:]).all() and torch.isnan(prob.cpu()[7])
    rows = [r for r in range(T) if r != 7]
    assert not torch.isnan(lg[rows]).any() and (lg[rows][:, 2] == float("-inf")).all()
    assert (idx.cpu()[rows] != 2).all() and (prob.cpu()[rows] > 0).all()
    # subnormal operands count (2^-130 times 2^20), and stay where they are: the matrix row they meet is zero elsewhere
    assert lg[9, 11] == 2.0 ** -110
    others = [c for c in range(E) if c not in (2, 11)]
    assert (lg[9][others] == 0).all()
    # the other rows: sums of d products in binary32, in any order
    plain = [r for r in range(T) if r not in (7, 9)]
    cols = [c for c in range(E) if c != 2]
    xs, ws = x.to(t).double()[plain], w.to(t).double()[:, cols]
    bound = (d + 2) * 2.0 ** -24 * (xs.abs() @ ws.abs())
    assert ((lg[plain][:, cols].double() - xs @ ws).abs() <= bound).all()
