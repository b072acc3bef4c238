"""The expert products on slot tables and row numbers that are not what they should be, on every kernel that takes them: rows past
max_rows, entries past n_slots, ids that are no expert's, row numbers out of range.  Those rows are left alone (or, for the last, get
some value), everything else is computed."""
import numpy as np
import pytest
import torch

import oracle
import synth
from ffn_shapes import BAD_ROWS, BAD_TABLES
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
    d, F, S = 128, 1024, len(rows)
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


# every kernel: its shape, and what it does to the rows per slot
KERNELS = [pytest.param(synth.F32 if name.startswith("f32") else synth.BF16, *shape, id=name.replace(" ", "-")) for name, *shape in BAD_TABLES]


def _run(dtype, d, F, E, rows, se, used, schedule, index=None, n_src=None):
    """-> (y, oracle's y for the rows of each slot under its own id) with y preset to 7."""
    import paper_2605_11537_amd as moe
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    T = int(so[-1])
    x = synth.normal_tensor((n_src or T, d), 1.0, [94, d, T], dtype)
    # weights of six experts, the same ones again for the rest
    w1 = np.resize(synth.normal_tensor((min(E, 6), d, F), 0.05, [95, d, F], dtype), (E, d, F))
    w2 = np.resize(synth.normal_tensor((min(E, 6), F, d), 0.05, [96, d, F], dtype), (E, F, d))
    good = (se >= 0) & (se < E)
    src = x if index is None else np.ascontiguousarray(x[np.clip(index, 0, len(x) - 1)])
    ref = f64(oracle.ffn(src, w1, w2, so, np.where(good, se, 0).astype(np.int32), len(rows)))
    pack = (lambda w: w) if dtype == synth.F32 else moe.moe_pack_weights
    t = torch.float32 if dtype == synth.F32 else torch.bfloat16
    y = torch.full((T, d), 7.0, dtype=t, device="cuda")
    n_slots = torch.tensor([used], dtype=torch.int32, device="cuda")
    if index is None:
        moe.moe_expert_ffn(to_dev(x), pack(to_dev(w1)), pack(to_dev(w2)), to_dev(so), to_dev(se), n_slots, E, F,
                           schedule=schedule, out=y)
    else:
        moe.moe_expert_ffn_rows(to_dev(x), to_dev(index), T, pack(to_dev(w1)), pack(to_dev(w2)), to_dev(so), to_dev(se), n_slots,
                                E, F, schedule=schedule, out=y)
    return f64(to_host(y)), ref, np.repeat(np.arange(len(rows)), rows)


def _close(got, ref, dtype):
    if dtype == synth.F32:                      # d and F roundings of binary32 sums, far inside
        return np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    return (np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-3 * np.abs(ref).max()).all()


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("dtype,d,F,scale,empty,experts", KERNELS)
def test_slots_that_are_none(dtype, d, F, scale, empty, experts, schedule):
    E = max(6, experts)
    rows = BAD_ROWS[0]
    se = [0, E, 0, 2, 2, -1, 4, 4, 5]           # ids that are no expert's, one between two slots of an expert
    used = 7                                    # the second slot of expert 4 and expert 5's are not slots
    rows, se = [r * scale for r in rows] + [0] * empty, np.array(se + [5] * empty, np.int32)
    got, ref, slot = _run(dtype, d, F, E, rows, se, used, schedule)
    on = (slot < used) & (se[slot] >= 0) & (se[slot] < E)
    assert (got[~on] == 7.0).all()
    assert _close(got[on], ref[on], dtype)


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("dtype,d,F,scale,empty,experts", KERNELS)
def test_row_numbers_out_of_range(dtype, d, F, scale, empty, experts, schedule):
    E = max(4, experts)
    rows = [r * scale for r in BAD_ROWS[1]] + [0] * empty
    se = np.array([0, 1, 2, 3] + [3] * empty, np.int32)
    T = sum(rows)
    n_src = T // 2 + 1
    rng = np.random.default_rng(T)
    index = rng.integers(0, n_src, T).astype(np.int32)
    bad = rng.random(T) < 0.2
    bad[0] = bad[-1] = True
    index[bad] = rng.choice([-1, -2 ** 31, n_src, 2 ** 31 - 1], bad.sum())
    got, ref, _ = _run(dtype, d, F, E, rows, se, len(rows), schedule, index, n_src)
    assert np.isfinite(got).all()
    assert _close(got[~bad], ref[~bad], dtype)


# the kernels that cut an expert's rows into tiles themselves (the LDS tiles in the slot schedule only)
@pytest.mark.parametrize("dtype,d,F,scale,empty,experts,schedule", [
    pytest.param(*k.values, schedule, id=f"{k.id}-{schedule}") for k in KERNELS for schedule in (0, 1)
    if k.id in ("f32-short", "f32-64-rows", "f32-staged") or k.id == "lds" and schedule == 0])
@pytest.mark.parametrize("slots", [9, 300])          # a slot per thread of the search, and two
def test_slots_that_begin_before_the_rows(dtype, d, F, scale, empty, experts, schedule, slots):
    """Such a slot is none, however far before (its tiles are not walked one by one up to the first row)."""
    import paper_2605_11537_amd as moe
    E, n = 9, 40 * scale
    rows = [n // 2, n // 2] + [0] * (slots - 2)
    so = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    se = np.minimum(np.arange(slots), E - 1).astype(np.int32)
    so[0] = -2 ** 30                                 # slot 0 runs from there to the middle
    # the sizes that the kernels want: many rows per slot and no 256 x 256 tiles for the LDS tiles, 128 rows per expert for 64-row tiles
    T, F = (65 * slots + 1, 640) if dtype == synth.BF16 else (n if scale == 1 else 1200, F)
    x = synth.normal_tensor((T, d), 1.0, [97, d], dtype)
    w1, w2 = synth.normal_tensor((E, d, F), 0.05, [98, d], dtype), synth.normal_tensor((E, F, d), 0.05, [99, d], dtype)
    ref = f64(oracle.ffn(x, w1, w2, np.array([0, n // 2, n], np.int32), np.array([0, 1], np.int32), 2))
    pack = (lambda w: w) if dtype == synth.F32 else moe.moe_pack_weights
    y = torch.full((T, d), 7.0, dtype=torch.float32 if dtype == synth.F32 else torch.bfloat16, device="cuda")
    moe.moe_expert_ffn(to_dev(x), pack(to_dev(w1)), pack(to_dev(w2)), to_dev(so), to_dev(se),
                       torch.tensor([slots], dtype=torch.int32, device="cuda"), E, F, schedule=schedule, out=y)
    got = f64(to_host(y))
    assert (got[: n // 2] == 7.0).all() and (got[n:] == 7.0).all()
    assert _close(got[n // 2: n], ref[n // 2: n], dtype)
