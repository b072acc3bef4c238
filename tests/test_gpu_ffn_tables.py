"""The expert products on slot tables that do not match the batch: rows past max_rows, which the kernels leave alone.  Every row
before it is computed."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f64, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("dtype,max_rows,rows", [
    (synth.F32, 64, [400] * 8),
    (synth.F32, 100, [30, 0, 50, 60, 700, 1, 900, 33]),
    (synth.BF16, 50, [5] * 4 + [0] + [5] * 5 + [60] + [300] * 150),  # few rows for this many slots: 32-column tiles
    (synth.BF16, 200, [20, 100, 60, 70, 700, 900, 300]),             # the 128-column tiles
])
def test_rows_past_the_batch(dtype, max_rows, rows, schedule):
    import paper_2605_11537_amd as moe
    d, F, S = 128, 256, len(rows)
    E = S
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    se = np.arange(S, dtype=np.int32)
    x = synth.normal_tensor((max_rows, d), 1.0, [91, S], dtype)
    w1 = synth.normal_tensor((E, d, F), 0.05, [92, S], dtype)
    w2 = synth.normal_tensor((E, F, d), 0.05, [93, S], dtype)
    ref = f64(oracle.ffn(x, w1, w2, np.minimum(so, max_rows), se, S))
    pack = (lambda w: w) if dtype == synth.F32 else moe.moe_pack_weights
    t = torch.float32 if dtype == synth.F32 else torch.bfloat16
    y = torch.full((max_rows, d), 7.0, dtype=t, device="cuda")
    moe.moe_expert_ffn(to_dev(x), pack(to_dev(w1)), pack(to_dev(w2)), to_dev(so), to_dev(se),
                       torch.tensor([S], dtype=torch.int32, device="cuda"), E, F, schedule=schedule, out=y)
    got = f64(to_host(y))
    if dtype == synth.F32:                      # d and F roundings of binary32 sums, far inside
        assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    else:                                       # half an ulp of the stored y, and of every stored h carried through W2
        assert (np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-3 * np.abs(ref).max()).all()
