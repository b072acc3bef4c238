"""The bf16 expert products of batches with few rows: most slots empty (one to four slots per thread of the search, and one slot too many
for it), few slots with a long k, every number of row blocks per pass, more units than workgroups, k that fills, misses and exceeds
the steps in flight, both schedules (whose results are the same bits)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f64, few_rows, to_dev, to_host

pytestmark = pytest.mark.gpu


def _spread(n_slots, rows):
    r = np.zeros(n_slots, int)
    r[np.random.default_rng(n_slots).permutation(n_slots)[:len(rows)]] = rows
    return list(r)


@pytest.mark.parametrize("d,F,E,rows,products", [
    (128, 1024, 20, _spread(150, [1, 2, 33, 32, 3]), (True, True)),           # two steps of k per wavefront; 16
    (384, 640, 9, _spread(150, [31, 7]), (True, True)),                       # six and ten: half a burst past the end
    (128, 896, 9, _spread(150, [31, 7]), (False, False)),                     # matrices too small for it
    (128, 1024, 30, _spread(400, [40, 65, 1, 90]), (True, True)),             # two slots per thread; passes of 2, 3, 1 and 3 blocks
    (256, 512, 50, _spread(700, [5, 40, 1, 1, 1]), (True, True)),             # three slots per thread
    (128, 1024, 40, _spread(1024, [130, 1, 200, 64, 100]), (True, True)),     # four; a second pass of 2 and of 72 rows
    (128, 1024, 40, _spread(1025, [130, 1, 200, 64, 100]), (False, False)),   # one slot too many: the 128-column kernel
    (256, 1152, 4, [7, 0, 31, 33, 20], (False, True)),                        # few slots: the second product only, 18 steps
    (256, 1408, 3, [20, 40, 1], (False, True)),                               # 22 steps: half a burst after a round
    (128, 3072, 4, [20, 40, 1, 60], (False, True)),                           # 48 steps: four rounds
    (128, 3072, 25, _spread(400, [33, 40, 70, 1, 20]), (True, True)),         # 96 column tiles x 9 row tiles, 5 experts: units queue
    (128, 1024, 3, [20, 10, 2] + [0] * 60, (False, True)),                    # a slot more would be too few empty ones
])
def test_ffn_few_rows(d, F, E, rows, products):
    import paper_2605_11537_amd as moe
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    se = np.sort(np.random.default_rng(E).integers(0, E, len(rows))).astype(np.int32)
    n = int(so[-1])
    T = n + 2
    assert (few_rows(T, len(rows), d, F), few_rows(T, len(rows), F, d)) == products
    perm = np.random.default_rng(d).permutation(T).astype(np.int32)
    x = synth.normal_tensor((T, d), 1.0, [81, d, F], synth.BF16)
    w1 = synth.normal_tensor((E, d, F), 0.05, [82, d, F], synth.BF16)
    w2 = synth.normal_tensor((E, F, d), 0.05, [83, d, F], synth.BF16)
    ref = f64(oracle.ffn(np.ascontiguousarray(x[perm]), w1, w2, so, se, len(rows)))[:n]
    w1p, w2p = moe.moe_pack_weights(to_dev(w1)), moe.moe_pack_weights(to_dev(w2))
    out = []
    for schedule in (0, 1):
        y = torch.full((T, d), 7.0, dtype=torch.bfloat16, device="cuda")
        moe.moe_expert_ffn(to_dev(x), w1p, w2p, to_dev(so), to_dev(se),
                           torch.tensor([len(rows)], dtype=torch.int32, device="cuda"), E, F, row_index=to_dev(perm),
                           schedule=schedule, out=y)
        got = f64(to_host(y))
        assert (got[n:] == 7.0).all()
        # half an ulp of the stored y, and of every stored h carried through W2 (a rounding of h can fall the other way)
        assert (np.abs(got[:n] - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-3 * np.abs(ref).max()).all()
        out.append(y)
    assert torch.equal(out[0], out[1])
