"""moe_dispatch on both sides of the batch that one workgroup takes (2048 entries, 256 experts): every table against its definition, for replica
counts of every kind -- none, some, zero and negative, past the slot tables, past 31 bits in sum -- and entries of a top-k layer."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tables(ids, replicas, E, C, max_slots):
    """As the header defines them."""
    T = len(ids)
    counts = np.bincount(ids[(ids >= 0) & (ids < E)], minlength=E)
    r = np.maximum(replicas.astype(np.int64), 1)
    kept = np.minimum(counts, r * C)
    off = np.concatenate([[0], np.cumsum(kept)])
    inv, perm, seen = np.full(T, -1), np.full(T, -1), np.zeros(E, np.int64)
    for s, e in enumerate(ids):
        if not 0 <= e < E:
            continue
        if seen[e] < kept[e]:
            inv[s] = off[e] + seen[e]
            perm[inv[s]] = s
        seen[e] += 1
    slots = []
    for e in range(E):
        if len(slots) > max_slots:
            break
        j = np.arange(min(r[e], max_slots + 1))
        slots += list(off[e] + j * (kept[e] // r[e]) + np.minimum(j, kept[e] % r[e]))
    slots = (slots + [off[E]] * (max_slots + 1))[: max_slots + 1]
    return dict(counts=counts, kept=kept, expert_offset=off, slot_offset=np.array(slots), perm=perm, inv=inv)


@pytest.mark.parametrize("E", [1, 2, 63, 64, 200, 256, 257])
@pytest.mark.parametrize("T", [0, 1, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049])
def test_tables(T, E):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(100 * E + T)
    ids = rng.choice(E, T, p=np.arange(1, E + 1) ** -1.0 / np.sum(np.arange(1, E + 1) ** -1.0)).astype(np.int32)
    C, max_slots = max(1, T // E), E + max(2, E // 4)
    one = np.ones(E, np.int64)
    some, odd, huge = one.copy(), rng.integers(-3, 4, E), one.copy()
    some[rng.integers(0, E, max(1, E // 4))] += 1
    huge[rng.integers(0, E, 2)] = 2 ** 31 - 1
    for replicas in (None, some, odd, huge, one * (max_slots + 5)):
        rep = None if replicas is None else torch.from_numpy(replicas.astype(np.int32)).cuda()
        poison = lambda n: torch.full((n,), -77, dtype=torch.int32, device="cuda")  # noqa: E731
        out = dict(counts=poison(E), kept=poison(E), expert_offset=poison(E + 1), slot_offset=poison(max_slots + 1), perm=poison(T),
                   inv=poison(T), x_perm=None)
        moe.moe_dispatch(None, torch.from_numpy(ids).cuda(), rep, E, C, max_slots, out=out, shape=(T, 64), dtype=torch.float32)
        want = _tables(ids, one if replicas is None else replicas, E, C, max_slots)
        for k, v in want.items():
            assert np.array_equal(out[k].cpu().numpy(), v), (k, T, E)


@pytest.mark.parametrize("T", [1279, 1280, 1281, 1537, 2048])          # lanes of one id one after another, and by a ballot
@pytest.mark.parametrize("E,share", [(1, 1.0), (2, 0.5), (3, 0.9), (16, 0.8), (64, 0.0), (256, 1.0)])
def test_ids_that_lanes_share(T, E, share):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(T + E)
    ids = rng.integers(0, E, T).astype(np.int32)
    ids[rng.random(T) < share] = E - 1
    C = max(1, T // (2 * E))
    d = moe.moe_dispatch(torch.randn(T, 8, device="cuda"), torch.from_numpy(ids).cuda(), None, E, C, E)
    for name, v in _tables(ids, np.ones(E, np.int64), E, C, E).items():
        assert np.array_equal(d[name].cpu().numpy(), v), name


@pytest.mark.parametrize("T,k,E", [(682, 3, 64), (683, 3, 64), (100, 2, 256), (40, 8, 10)])     # 2046 and 2049 entries
def test_topk_rows(T, k, E):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(T)
    ids = np.stack([rng.permutation(E)[:k] for _ in range(T)], 1).astype(np.int32)
    x = torch.randn(T, 64, device="cuda")
    C = max(1, k * T // (2 * E))
    d = moe.moe_dispatch_topk(x, torch.from_numpy(ids).cuda(), None, E, C, E)
    want = _tables(ids.reshape(-1), np.ones(E, np.int64), E, C, E)
    for name, v in want.items():
        assert np.array_equal(d[name].cpu().numpy().reshape(-1), v), name
    K = want["expert_offset"][-1]
    row = d["row_token"].cpu().numpy()
    assert np.array_equal(row[:K], want["perm"][:K] % T) and (row[K:] == -1).all()
    assert torch.equal(d["x_perm"][:K], x[torch.from_numpy(want["perm"][:K] % T).cuda()])
