"""The one-kernel SRU layer at the edges of its variants: sequences around 256, 512 and 1024 positions, blocks of 32
positions part filled, the shortest sequences whose states are handed on as fragments and those that are not, first-layer
widths with and without room for their weights in LDS, one layer (nothing handed on) and several."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,n_in,n_h,layers", [
    (2, 7, 128, 128, 3),          # too short for the fragment images
    (3, 32, 64, 128, 2),          # seven wavefronts without rows, one chunk of k, one recurrence step
    (2, 64, 128, 128, 2),         # one step, two chunks
    (2, 65, 192, 128, 2),         # two steps, three chunks
    (1, 128, 320, 128, 2),        # two steps, four wavefronts with rows
    (2, 129, 256, 128, 2),        # three steps
    (1, 300, 64, 128, 2),         # two row blocks per wavefront, few weights
    (3, 8, 128, 256, 3),          # the shortest with them
    (1, 33, 256, 256, 2),         # one position in the last block; highway input from row-major and from fragments
    (2, 256, 64, 128, 2),         # the last length of one row block per wavefront
    (8, 257, 320, 128, 2),        # two row blocks, whole sequences per XCD
    (1, 512, 832, 256, 2),        # first layer too wide for its weights in LDS
    (2, 513, 768, 128, 2),        # four row blocks; embeddings too wide beside the states for an image of their own
    (2, 777, 768, 256, 3),        # embeddings packed first, their image overwritten by the second layer
    (1, 1024, 832, 256, 1),       # the same without room for the weights in LDS, one layer
    (2, 200, 128, 384, 2),        # fragments with weights too wide for LDS, one row block per wavefront
    (1, 400, 128, 384, 2),        # fragments of more than 256 channels whose weights fit, two row blocks
    (1, 400, 128, 896, 2),        # and whose weights do not
    (1, 288, 128, 896, 2),        # the same with wavefronts that have one row block and one that has two
    (2, 288, 128, 768, 2),        # the widest whose weights fit, likewise
    (1, 1024, 128, 384, 3),       # the longest; later layers too wide for their weights in LDS
    (1, 1025, 128, 128, 2),       # the two-kernel form
    (1, 600, 1024, 256, 2),       # the two-kernel form in front of one kernel: its states as fragments, the last layer's row-major
    (2, 513, 1024, 128, 3),       # the same with a layer in between
    (3, 520, 64, 1024, 2),        # one kernel in front of the two-kernel form
    (1, 513, 2048, 128, 1),       # the two-kernel form alone, under 1024 positions
])
def test_sru_layer_variants(B, L, n_in, n_h, layers):
    import paper_2605_11537_amd as moe
    s = synth.sru_inputs(B, L, n_in, n_h, layers, 128, synth.BF16, 4000 + L, bias_std=0.2)
    w = moe.SruWeights([to_dev(a) for a in s["w_cat"]], [to_dev(a) for a in s["b_f"]], [to_dev(a) for a in s["b_r"]],
                       to_dev(s["w_head"]), to_dev(s["b_head"]))
    ref = oracle.sru(s["emb"], s["w_cat"], s["b_f"], s["b_r"], s["w_head"], s["b_head"])
    # workspace contents must not matter
    import ctypes
    need = moe.lib().sru_predict_workspace_bytes(ctypes.byref(w.c), B, L, moe.MOE_BF16)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    pred, logits = moe.sru_predict(to_dev(s["emb"]), w, want_logits=True, ws=ws)
    lg, want = to_host(logits), ref["logits"].reshape(B * L, -1)
    # states are stored in bf16 between layers on both sides; the bound of the predictor tests
    assert np.abs(lg - want).max() <= 5e-3 * np.abs(want).max()
    assert (to_host(pred) == lg.argmax(axis=1)).all()


@pytest.mark.parametrize("L", [40, 1030])                 # one kernel, two kernels
@pytest.mark.parametrize("bias", [-1.0, -50.0, -79.0, -82.0, -86.0, -200.0])
def test_sru_nearly_closed_gate(L, bias):
    """A state that is the reset gate alone (x' large, forget gate and highway closed): sigmoid(bias) in bf16, also where it is tiny."""
    import paper_2605_11537_amd as moe
    n_in, n_h, n_out = 64, 128, 8
    dev = dict(dtype=torch.bfloat16, device="cuda")
    w_cat = torch.zeros(n_in, 4 * n_h, **dev)
    w_cat[:, :n_h] = 1.0                                    # x' = 64: tanh(c) = 1
    shift = 2.0 ** round(min(-bias / np.log(2.0), 120.0))
    b_f = torch.full((n_h,), -300.0, device="cuda")
    b_r = torch.full((n_h,), bias, device="cuda")
    w = moe.SruWeights([w_cat], [b_f], [b_r], torch.full((n_h, n_out), shift, **dev))
    _, logits = moe.sru_predict(torch.ones(2, L, n_in, **dev), w, want_logits=True)
    lg = to_host(logits).astype(np.float64)
    if bias < -88.0:                                        # below every normal number
        assert (lg >= 0).all() and (lg <= n_h * 2.0 ** -126 * shift).all()
        return
    want = n_h * shift / (1.0 + np.exp(-bias))
    # half an ulp of the stored state, a few of the hardware's exponential (whose argument is rounded to 2^-24 of itself)
    assert (np.abs(lg / want - 1) <= 2.0 ** -8 + abs(bias) * 2.0 ** -23).all()


@pytest.mark.parametrize("n_out,shift", [(64, 1), (104, 1), (104, 2), (512, 1), (512, 4), (1024, 3)])
def test_sru_head_at_any_address(n_out, shift):
    """A plain head matrix that starts in the middle of a 16-byte piece: columns are loaded as far as it is aligned."""
    import paper_2605_11537_amd as moe
    B, L, n_in, n_h = 2, 33, 64, 128
    s = synth.sru_inputs(B, L, n_in, n_h, 1, n_out, synth.BF16, 61 + n_out, bias_std=0.2)
    head = to_dev(s["w_head"])
    moved = torch.zeros(head.numel() + shift, dtype=head.dtype, device="cuda")[shift:].view(n_h, n_out)
    moved.copy_(head)
    assert moved.data_ptr() % 16 == 2 * shift and moved.is_contiguous()
    lg = []
    for w_head in (head, moved):
        w = moe.SruWeights([to_dev(a) for a in s["w_cat"]], [to_dev(a) for a in s["b_f"]], [to_dev(a) for a in s["b_r"]], w_head,
                           to_dev(s["b_head"]))
        pred, logits = moe.sru_predict(to_dev(s["emb"]), w, want_logits=True)
        lg.append(to_host(logits).astype(np.float64))
        assert (to_host(pred) == lg[-1].argmax(axis=1)).all()
    # the same products of bf16 values, summed in binary32 in another order
    assert np.abs(lg[0] - lg[1]).max() <= (n_h + 2) * 2.0 ** -22 * np.abs(lg[0]).max()


@pytest.mark.parametrize("B,L,n_in,n_h,layers", [
    (2, 7, 128, 128, 2),               # row-major states
    (3, 8, 128, 256, 1),               # the first layer writes the images itself; one part-filled block
    (2, 65, 128, 128, 2),              # a second score per lane, positions in the last group of 16
    (1, 257, 128, 256, 2),             # eight scores per lane
    (8, 513, 128, 128, 1),             # sixteen, the second half of the packed states
    (1, 1000, 128, 256, 2),
    (1, 600, 1024, 256, 2),       # after a first layer in two kernels
    (1, 600, 2048, 128, 1),       # whose form does not go in front of the attention
])
def test_attention_variants(B, L, n_in, n_h, layers):
    import ctypes
    import paper_2605_11537_amd as moe
    s = synth.sru_inputs(B, L, n_in, n_h, layers, 128, synth.BF16, 5000 + L, bias_std=0.1)
    w = moe.SruWeights([to_dev(a) for a in s["w_cat"]], [to_dev(a) for a in s["b_f"]], [to_dev(a) for a in s["b_r"]],
                       to_dev(s["w_head"]), to_dev(s["b_head"]), attention=True)
    ref = oracle.sru_attention(s["emb"], s["w_cat"], s["b_f"], s["b_r"], s["w_head"], s["b_head"])
    need = moe.lib().sru_predict_workspace_bytes(ctypes.byref(w.c), B, L, moe.MOE_BF16)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")     # whatever the images' padding holds: NaN here
    pred, logits = moe.sru_predict(to_dev(s["emb"]), w, want_logits=True, ws=ws)
    lg, want = to_host(logits), ref["logits"].reshape(B * L, -1)
    assert np.abs(lg - want).max() <= 5e-3 * np.abs(want).max()          # the bound of the predictor tests
    assert (to_host(pred) == lg.argmax(axis=1)).all()
