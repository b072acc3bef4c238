"""The binary32 expert products with tokens staged through LDS (k = 384, 512, .. by 128) and with tiles of 32 columns (few units): ragged tiles,
one and several steps of k per wavefront, gathered rows with bad numbers, slots on both sides of one per thread."""
import numpy as np
import pytest
import torch

import oracle  # noqa: F401  (built before the GPU is touched)
import synth
from gpu_util import f64, to_dev, to_host

pytestmark = pytest.mark.gpu


# shape: d, F, E, rows and expert per slot, gathered;  what it takes: rows of a tile, first and second product with 32 columns, and staged
SHAPES = [
    ((384, 512, 2, [1, 33], None, True), (32, (1, 1), (1, 1))),                                   # odd numbers of steps
    ((256, 128, 3, [32, 0, 17, 64], [0, 1, 2, 2], False), (32, (1, 0), (0, 0))),                  # k = 256; k = 128 is short
    ((512, 4096, 8, [31, 32, 33, 15, 16, 17, 48, 1], list(range(8)), True), (32, (0, 1), (1, 1))),
    ((640, 1024, 3, [430, 500, 270], [0, 1, 2], True), (64, (0, 0), (1, 1))),                     # cost ranges inside an expert
    ((512, 1536, 2, [610, 700], [0, 1], True), (64, (0, 0), (1, 1))),
    ((512, 384, 2, [300, 290], [0, 1], True), (64, (0, 0), (0, 0))),                              # too few tiles
    ((384, 448, 30, [(5 * i) % 9 for i in range(300)], None, False), (32, (0, 0), (1, 0))),       # more slots than threads; k = 448
]


@pytest.mark.parametrize("d,F,E,rows,se,gather", [s for s, _ in SHAPES])
def test_ffn_f32_staged(d, F, E, rows, se, gather):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(d * F)
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    se = np.array(se, np.int32) if se else np.sort(rng.integers(0, E, len(rows))).astype(np.int32)
    n, T = int(so[-1]), int(so[-1]) + 3
    x = synth.normal_tensor((T, d), 1.0, [4, d, F], synth.F32)
    w1 = synth.normal_tensor((E, d, F), 0.1, [5, d, F], synth.F32)
    w2 = synth.normal_tensor((E, F, d), 0.1, [6, d, F], synth.F32)
    index = rng.permutation(T).astype(np.int32) if gather else None
    src = x[:n]
    if gather:
        index[0], index[n // 2] = -1, T + 7                                # a bad row number reads row 0
        src = x[np.where((index >= 0) & (index < T), index, 0)][:n]
    y = torch.full((T, d), 7.0, device="cuda")
    moe.moe_expert_ffn(to_dev(x), to_dev(w1), to_dev(w2), to_dev(so), to_dev(se),
                       torch.tensor([len(rows)], dtype=torch.int32, device="cuda"), E, F, out=y, row_index=to_dev(index))
    got = to_host(y)
    assert (got[n:] == 7.0).all()
    e_of = np.repeat(se, rows)
    a, b1, b2 = f64(src), f64(w1), f64(w2)
    u = 2.0 ** -24
    for e in np.unique(e_of):
        r = e_of == e
        h = np.maximum(a[r] @ b1[e], 0.0)
        # sums in binary32 in any order: the first product's error carried through |W2|, and the second's own
        bound = (d + 2) * u * (np.abs(a[r]) @ np.abs(b1[e])) @ np.abs(b2[e]) + (F + 2) * u * (np.abs(h) @ np.abs(b2[e]))
        assert (np.abs(got[:n][r] - h @ b2[e]) <= bound + 1e-30).all()
