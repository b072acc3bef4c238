"""Sequences that fill a layer's row blocks and recurrence steps in part: every number of blocks per wavefront and of steps per chunk, row-major
embeddings and fragments, and batches whose sequences lie on several XCDs.  Against the oracle, and against the same sequences one by
one (the order of every sum is a sequence's own in the one-kernel form: the same bits)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,n_in,n_h,layers", [
    (3, 288, 64, 128, 2),         # nine blocks: one wavefront with two, five steps
    (9, 384, 128, 128, 2),        # the last length of six steps
    (5, 385, 128, 256, 2),        # the first of eight
    (3, 544, 128, 128, 2),        # 17 blocks: one wavefront with three
    (5, 640, 512, 128, 2),        # the last of ten steps; embeddings too wide beside the states for an image
    (3, 641, 64, 128, 2),         # the first of twelve
    (2, 768, 128, 128, 2),        # three blocks for everybody, the last of twelve steps
    (6, 769, 128, 256, 2),        # one wavefront with four, fourteen steps
    (3, 896, 512, 256, 2),        # embeddings as an image, the last of fourteen steps
    (3, 897, 256, 128, 2),        # sixteen; the highway from row-major rows
    (9, 23, 448, 256, 12),        # channel blocks dealt to the XCDs: many layers,
    (5, 33, 384, 1024, 2),        # wide ones
    (3, 300, 256, 1024, 3),       # and two row blocks
])
def test_sru_ragged(B, L, n_in, n_h, layers):
    import paper_2605_11537_amd as moe
    s = synth.sru_inputs(B, L, n_in, n_h, layers, 128, synth.BF16, 7000 + L, bias_std=0.2)
    w = moe.SruWeights([to_dev(a) for a in s["w_cat"]], [to_dev(a) for a in s["b_f"]], [to_dev(a) for a in s["b_r"]],
                       to_dev(s["w_head"]), to_dev(s["b_head"]))
    ref = oracle.sru(s["emb"], s["w_cat"], s["b_f"], s["b_r"], s["w_head"], s["b_head"])
    emb = to_dev(s["emb"])
    pred, logits = moe.sru_predict(emb, w, want_logits=True)
    lg, want = to_host(logits), ref["logits"].reshape(B * L, -1)
    assert np.abs(lg - want).max() <= 5e-3 * np.abs(want).max()      # states in bf16 between layers; the bound of the predictor tests
    assert (to_host(pred) == lg.argmax(axis=1)).all()
    # (one sequence of wide embeddings takes two kernels, which compose the chunks in another order)
    for b in range(B if n_in < 512 else 0):
        _, alone = moe.sru_predict(emb[b:b + 1].contiguous(), w, want_logits=True)
        assert torch.equal(alone, logits[b * L:(b + 1) * L]), b
