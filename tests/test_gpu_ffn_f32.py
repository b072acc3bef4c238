"""The binary32 expert products: slots around the 16-row blocks and the tiles of 32 and 64 rows, every number of blocks in the last
tile, one to many steps of k, units dealt one by one and several to a workgroup, more slots than a workgroup has threads, both
schedules, with and without the gather."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f64, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("d,F,E,rows,se,gather", [
    (64, 64, 3, [1, 0, 16, 17], None, False),                              # one step of k per wavefront
    (64, 320, 4, [15, 48, 49, 64, 65, 31, 33, 0, 130], None, True),        # tiles of 32 rows: one and two blocks; five steps
    (448, 192, 2, [200, 3], None, True),                                   # seven steps, three steps
    (64, 128, 40, [(7 * i) % 23 for i in range(600)], None, False),        # three slots per thread
    (64, 512, 40, [(7 * i) % 23 for i in range(600)], None, False),        # more units than workgroups of a short k
    # 128 rows per expert and more: tiles of 64 rows, whose last ones have 2, 3, 4 and 1 blocks; one slot or several per expert
    (320, 448, 3, [96, 112, 250], [0, 1, 2], True),
    (256, 320, 4, [50, 46, 0, 112, 100, 150, 129], [0, 0, 0, 1, 2, 2, 3], True),    # k = 256: several units per workgroup allowed
    (256, 3072, 8, [190] * 8, list(range(8)), False),                      # and more than there are workgroups
    (256, 64, 5, [20, 40, 33, 64, 1], None, True),                         # k = 256 with tiles of 32 rows
])
def test_ffn_f32_tiles(d, F, E, rows, se, gather, schedule):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(d + F)
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    # slots of one expert are neighbours
    se = np.array(se, np.int32) if se else np.sort(rng.integers(0, E, len(rows))).astype(np.int32)
    n, T = int(so[-1]), int(so[-1]) + 5
    x = synth.normal_tensor((T, d), 1.0, [1, d, F], synth.F32)
    w1 = synth.normal_tensor((E, d, F), 0.1, [2, d, F], synth.F32)
    w2 = synth.normal_tensor((E, F, d), 0.1, [3, d, F], synth.F32)
    index = rng.permutation(T).astype(np.int32) if gather else None
    src = x[index] if gather else x
    y = torch.full((T, d), 7.0, device="cuda")
    moe.moe_expert_ffn(to_dev(x), to_dev(w1), to_dev(w2), to_dev(so), to_dev(se),
                       torch.tensor([len(rows)], dtype=torch.int32, device="cuda"), E, F, out=y, schedule=schedule,
                       row_index=to_dev(index))
    got = to_host(y)
    assert (got[n:] == 7.0).all()                                    # rows outside the slots stay as they are
    e_of = np.repeat(se, rows)
    a, b1, b2 = f64(src[:n]), f64(w1), f64(w2)
    for e in np.unique(e_of):
        r = e_of == e
        h = np.maximum(a[r] @ b1[e], 0.0)
        ref = h @ b2[e]
        # errors of sums in binary32, in any order: the first product's, carried through |W2|, and the second's own
        u = 2.0 ** -24
        h_err = (d + 2) * u * (np.abs(a[r]) @ np.abs(b1[e]))
        bound = h_err @ np.abs(b2[e]) + (F + 2) * u * (np.abs(h) @ np.abs(b2[e]))
        assert (np.abs(got[:n][r] - ref) <= bound + 1e-30).all()
