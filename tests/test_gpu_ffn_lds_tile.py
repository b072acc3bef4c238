"""The bf16 expert products on the 128-row LDS tile: every number of row blocks in the last tile, 128 and 256 columns, the shortest k, several tiles
and slots of one expert, gathered rows with bad numbers, slots on both sides of one per thread, ReLU of infinities and NaN."""
import numpy as np
import pytest
import torch

import oracle  # noqa: F401  (built before the GPU is touched)
import synth
from gpu_util import assert_close, f64, to_dev, to_host

pytestmark = pytest.mark.gpu


def _case(d, F, E, rows, se, gather, seed):
    rng = np.random.default_rng(seed)
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    se = np.array(se, np.int32) if se else np.arange(len(rows), dtype=np.int32)
    n, T = int(so[-1]), int(so[-1]) + 3
    x = synth.normal_tensor((T, d), 1.0, [7, d, F], synth.BF16)
    w1 = synth.normal_tensor((E, d, F), 0.05, [8, d, F], synth.BF16)
    w2 = synth.normal_tensor((E, F, d), 0.05, [9, d, F], synth.BF16)
    index = rng.permutation(T).astype(np.int32) if gather else None
    return so, se, n, T, x, w1, w2, index


def _run(so, se, x, w1, w2, index, E, F):
    import paper_2605_11537_amd as moe
    y = torch.full(x.shape, 7.0, dtype=torch.bfloat16, device="cuda")
    moe.moe_expert_ffn(to_dev(x), moe.moe_pack_weights(to_dev(w1)), moe.moe_pack_weights(to_dev(w2)), to_dev(so), to_dev(se),
                       torch.tensor([len(se)], dtype=torch.int32, device="cuda"), E, F, out=y, row_index=to_dev(index))
    return to_host(y)


SHAPES = [
    (128, 256, 4, [65, 96, 97, 128], None, True),                        # 3, 3, 4, 4 blocks; k = 128
    (384, 128, 3, [129, 160, 31], None, False),                          # a second tile of one row, of 32 rows; 128 columns
    (256, 512, 2, [300, 20, 0, 150], [0, 0, 1, 1], True),                # tiles over the slots of an expert
    (512, 4096, 16, [200] * 16, None, True),                             # 256 columns in the first product
    (256, 2048, 8, [190 + i for i in range(8)], None, False),
    (128, 128, 260, [70] * 260, None, False),                            # more slots than threads
    (256, 512, 64, [1030] + [49] * 62 + [28], None, True),               # 64 rows per slot on average, one long slot
    (512, 4096, 24, [97, 33, 64, 1, 96, 128] * 4, None, True),           # wavefronts with no, one and two row blocks, side by side; 256 columns
]


@pytest.mark.parametrize("d,F,E,rows,se,gather", SHAPES)
def test_ffn_lds_tile(d, F, E, rows, se, gather):
    so, se, n, T, x, w1, w2, index = _case(d, F, E, rows, se, gather, d + F)
    src = x[:n]
    if gather:
        index[1], index[n // 2] = -5, T
        src = x[np.where((index >= 0) & (index < T), index, 0)][:n]
    got = _run(so, se, x, w1, w2, index, E, F)
    assert (f64(got[n:]) == 7.0).all()
    e_of = np.repeat(se, rows)
    for e in np.unique(e_of):
        r = e_of == e
        # h is rounded to bf16 between the products, as the library does
        h = torch.from_numpy(np.maximum(f64(src[r]) @ f64(w1[e]), 0.0)).to(torch.bfloat16).double().numpy()
        assert_close(got[:n][r], torch.from_numpy(h @ f64(w2[e])).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16),
                     synth.BF16, f"expert {e}")


@pytest.mark.parametrize("rows", [96, 4200])
def test_ffn_lds_tile_relu_of_nan(rows):
    """A token of NaN ends at the ReLU, which gives 0 for it as the other tile kernels do; one with an infinity does not; neither reaches
    its neighbours."""
    d, F = 256, 512
    so, se, n, T, x, w1, w2, index = _case(d, F, 1, [rows], None, False, 3)
    x = to_dev(x)
    x[5] = float("nan")
    x[7, 3] = float("inf")
    got = f64(_run(so, se, to_host(x), w1, w2, None, 1, F))
    assert np.isfinite(np.delete(got, [5, 7], 0)).all() and (got[5] == 0.0).all() and not np.isfinite(got[7]).any()
