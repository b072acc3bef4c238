"""The hand-out of the slots that the floors of the plan leave, several per step, and the dispatch tables made beside it, against the oracle: equal
loads (ties by id), loads that binary32 cannot tell apart, one expert far ahead (several slots in a row), more experts above the bar than slots,
every size class of the allocating wavefront, no slot and one, plan and dispatch apart and in one call, one block of tokens to many."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _ids(kind, T, E, rng):
    if kind == "equal":
        return np.arange(T) % E
    if kind == "close":                      # loads that differ by a few in a hundred thousand and more
        n = T // E + rng.integers(-2, 3, E)
        return np.repeat(np.arange(E), np.maximum(n, 0))[:T] if n.sum() >= T else np.concatenate(
            [np.repeat(np.arange(E), np.maximum(n, 0)), np.full(T - n.sum(), E - 1)])
    if kind == "one":
        return np.where(rng.random(T) < 0.7, E // 2, rng.integers(0, E, T))
    w = np.arange(1, E + 1.0) ** -{"zipf": 1.0, "steep": 2.0}[kind]
    return rng.permutation(E)[rng.choice(E, T, p=w / w.sum())]


@pytest.mark.parametrize("kind", ["equal", "close", "one", "zipf", "steep"])
@pytest.mark.parametrize("T,E,R,C", [
    (500, 5, 3, 7), (4096, 128, 16, 40), (8192, 256, 200, 9), (8193, 60, 31, 30), (12288, 128, 16, 120), (20000, 64, 100, 50),
    (30000, 256, 64, 70), (9000, 500, 90, 11), (17000, 1024, 333, 10),
    (4000, 128, 0, 5), (3000, 200, 1, 5), (5000, 600, 1, 4), (3000000, 7, 3, 1000), (3000000, 12, 40, 20000), (6000000, 300, 500, 3000),
])
def test_plan_and_dispatch(T, E, R, C, kind):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(T + E)
    ids = _ids(kind, T, E, rng).astype(np.int32)
    other = np.roll(ids, 3)[: T // 2].copy()
    for plan_ids in (ids, other):
        ref = oracle.plan(plan_ids, E, R, C)
        dev = to_dev(ids)
        same = dev if plan_ids is ids else to_dev(plan_ids)
        pl, dp = moe.moe_plan_dispatch(same, dev, E, R, C)
        alone = moe.replica_plan(same, E, R, C)
        apart = moe.moe_dispatch(None, dev, alone["replicas"], E, C, E + R, shape=(T, 8), dtype=torch.float32)
        for got in (pl, alone):
            assert (to_host(got["replicas"]) == ref["replicas"]).all() and (to_host(got["plan_counts"]) == ref["counts"]).all()
            assert (to_host(got["slot_base"]) == ref["slot_base"]).all() and int(got["n_slots"][0]) == ref["n_slots"]
            assert (to_host(got["slot_expert"]) == ref["slot_expert"]).all()
        counts = np.bincount(ids, minlength=E)
        kept = np.minimum(counts, ref["replicas"].astype(np.int64) * C)
        first = np.concatenate([[0], np.cumsum(kept)])
        order = np.argsort(ids, kind="stable")
        rank = np.empty(T, np.int64)
        rank[order] = np.arange(T) - np.repeat(np.concatenate([[0], np.cumsum(counts)[:-1]]), counts)
        inv = np.where(rank < kept[ids], first[ids] + rank, -1)
        perm = np.full(T, -1, np.int64)
        perm[inv[inv >= 0]] = np.nonzero(inv >= 0)[0]
        slots = [first[-1]] * (E + R + 1)
        for e in range(E):
            q, rem = divmod(int(kept[e]), int(ref["replicas"][e]))
            for j in range(ref["replicas"][e]):
                slots[ref["slot_base"][e] + j] = first[e] + j * q + min(j, rem)
        for got in (dp, apart):
            for key, want in (("counts", counts), ("kept", kept), ("expert_offset", first), ("inv", inv), ("perm", perm),
                              ("slot_offset", slots)):
                assert (to_host(got[key]) == np.asarray(want)).all(), key


@pytest.mark.parametrize("replicas,max_slots", [
    ([2**31 - 1, 1, 1], 3),                         # "as many as it takes"
    ([2, 2**31 - 1, 5, 2**31 - 1], 9),              # their sum does not fit an int
    ([1, 70, 2**31 - 64, 1], 200),
    ([1] * 70 + [2**31 - 1] + [3] * 5, 90),         # past the first wavefront of experts
    ([3, 4, 2], 9),
])
def test_replicas_beyond_the_slot_table(replicas, max_slots):
    """Replica counts of a caller's own, however large: every slot that the table holds, nothing behind it."""
    import paper_2605_11537_amd as moe
    E, C, T = len(replicas), 3, 1500
    rng = np.random.default_rng(E)
    ids = rng.integers(0, E, T).astype(np.int32)
    room = to_dev(np.full(max_slots + 1 + 64, -7, np.int32))
    i32 = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")  # noqa: E731
    out = dict(counts=i32(E), kept=i32(E), expert_offset=i32(E + 1), slot_offset=room[: max_slots + 1], perm=i32(T), inv=i32(T), x_perm=None)
    moe.moe_dispatch(None, to_dev(ids), to_dev(np.array(replicas, np.int32)), E, C, max_slots, out=out, shape=(T, 8), dtype=torch.float32)
    kept = np.minimum(np.bincount(ids, minlength=E), np.array(replicas, np.int64) * C)
    first = np.concatenate([[0], np.cumsum(kept)])
    slots = []
    for e in range(E):
        q, rem = divmod(int(kept[e]), replicas[e])
        slots += [first[e] + j * q + min(j, rem) for j in range(min(replicas[e], max_slots + 1))]
    slots = (slots + [first[-1]] * (max_slots + 1))[: max_slots + 1]
    assert (to_host(out["kept"]) == kept).all() and (to_host(out["expert_offset"]) == first).all()
    assert (to_host(room) == np.array(slots + [-7] * 64)).all()


@pytest.mark.parametrize("E", [3, 40, 128, 200, 700])
def test_random_plans(E):
    """Plans of random sizes, loads and capacities, in both policies: few ids (many equal loads) to many (loads close together)."""
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(E)
    for i in range(60):
        T = int(np.exp(rng.uniform(np.log(E), np.log(200000 if i % 6 == 0 else 6000))))
        w = rng.pareto(rng.uniform(0.5, 4.0), E) + rng.choice([0.0, 0.2, 5.0, 500.0])
        ids = rng.choice(E, T, p=w / w.sum()).astype(np.int32)
        R, C, policy = int(rng.integers(0, 2 * E)), max(1, int(T / E * rng.uniform(0.1, 2.0))), int(i % 4 == 3)
        ref, got = oracle.plan(ids, E, R, C, policy), moe.replica_plan(to_dev(ids), E, R, C, policy)
        assert (to_host(got["replicas"]) == ref["replicas"]).all(), (i, T, R, C, policy)
        assert (to_host(got["slot_expert"]) == ref["slot_expert"]).all() and int(got["n_slots"][0]) == ref["n_slots"]
