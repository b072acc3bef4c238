"""The bf16 expert products of batches with few rows: most slots empty (one to four slots per thread of the search), few slots
with a long k, tiles that are walked and tiles side by side, the smallest and a long k, both schedules."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f64, to_dev, to_host

pytestmark = pytest.mark.gpu


def _spread(n_slots, rows):
    r = np.zeros(n_slots, int)
    r[np.random.default_rng(n_slots).permutation(n_slots)[:len(rows)]] = rows
    return list(r)


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("d,F,E,rows,used", [
    (128, 256, 20, _spread(144, [1, 2, 33, 32, 3]), 144),       # mostly empty: both products; two steps of k per wavefront
    (128, 128, 50, _spread(700, [5, 40, 1, 1, 1]), 700),        # three slots per thread
    (256, 1152, 4, [7, 0, 31, 33, 20], 5),                      # few slots: the second product only (18 steps: one refill and a half)
    (128, 256, 6, _spread(60, [4, 9]), 41),                     # entries past n_slots are not slots
])
def test_ffn_few_rows(d, F, E, rows, used, schedule):
    import paper_2605_11537_amd as moe
    if used < len(rows):
        rows = [r if i < used else 0 for i, r in enumerate(rows)]
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    se = np.sort(np.random.default_rng(E).integers(0, E, len(rows))).astype(np.int32)
    n = int(so[-1])
    T = n + 2
    perm = np.random.default_rng(d).permutation(T).astype(np.int32)
    x = synth.normal_tensor((T, d), 1.0, [81, d, F], synth.BF16)
    w1 = synth.normal_tensor((E, d, F), 0.05, [82, d, F], synth.BF16)
    w2 = synth.normal_tensor((E, F, d), 0.05, [83, d, F], synth.BF16)
    ref = f64(oracle.ffn(np.ascontiguousarray(x[perm]), w1, w2, so, se, used))[:n]
    y = torch.full((T, d), 7.0, dtype=torch.bfloat16, device="cuda")
    moe.moe_expert_ffn(to_dev(x), moe.moe_pack_weights(to_dev(w1)), moe.moe_pack_weights(to_dev(w2)), to_dev(so),
                       to_dev(se), torch.tensor([used], dtype=torch.int32, device="cuda"), E, F, row_index=to_dev(perm),
                       schedule=schedule, out=y)
    got = f64(to_host(y))
    assert (got[n:] == 7.0).all()
    # half an ulp of the stored y, and of every stored h carried through W2 (a rounding of h can fall the other way)
    assert (np.abs(got[:n] - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-3 * np.abs(ref).max()).all()
