"""The bf16 expert products over every way the chunk pipeline can end (1, 2, 3 chunks left, an even and an odd number
of rounds before) and every tile height (1, 2 and 4 row blocks), streamed once and shared between slots."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f64, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F", [(128, 384), (384, 640), (512, 768), (896, 256)])
def test_ffn_chunk_counts(d, F):
    import paper_2605_11537_amd as moe
    rows = [1, 32, 33, 64, 65, 128, 129, 31, 5]
    se = np.array([0, 1, 2, 3, 4, 5, 6, 7, 7], np.int32)             # the last two slots share an expert
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    E, n = 8, int(so[-1])
    T = n + 3
    perm = np.random.default_rng(d).permutation(T).astype(np.int32)
    x = synth.normal_tensor((T, d), 1.0, [61, d], synth.BF16)
    w1 = synth.normal_tensor((E, d, F), 0.05, [62, d], synth.BF16)
    w2 = synth.normal_tensor((E, F, d), 0.05, [63, d], synth.BF16)
    ref = f64(oracle.ffn(np.ascontiguousarray(x[perm]), w1, w2, so, se, len(rows)))[:n]
    y = moe.moe_expert_ffn(to_dev(x), moe.moe_pack_weights(to_dev(w1)), moe.moe_pack_weights(to_dev(w2)), to_dev(so),
                           to_dev(se), torch.tensor([len(rows)], dtype=torch.int32, device="cuda"), E, F,
                           row_index=to_dev(perm))
    got = f64(to_host(y))[:n]
    # half an ulp of the stored y, and of every stored h carried through W2 (a rounding of h can fall the other way)
    assert (np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-3 * np.abs(ref).max()).all()
