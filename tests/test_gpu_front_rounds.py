"""moe_plan_dispatch at the edges of its one-workgroup kernels: they are built for 2048, 4096 and 8192 ids, for up to 128 and up to 256 experts, and for
plan ids that are the routed ids or others.  Whole numbers: equal to the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [128, 129])
@pytest.mark.parametrize("T,n_plan", [(2048, 2048), (2049, 2049), (4096, 4096), (4097, 4097), (2048, 5), (5, 2049), (2049, 2048), (1000, 4097),
                                      (4097, 4000), (8192, 8191)])
def test_edges(T, n_plan, E):
    import paper_2605_11537_amd as moe
    rng = np.random.default_rng(T + n_plan)
    ids, other = (rng.choice(E, n, p=synth.zipf_weights(E, 1.1)).astype(np.int32) for n in (T, n_plan))
    pids = ids if n_plan == T else other
    dev = to_dev(ids)
    R, C = E // 8, max(1, T // E)
    want = oracle.plan(pids, E, R, C, 0)
    rows = oracle.dispatch(np.zeros((T, 4), np.float32), ids, want["replicas"], E, C, E + R)
    for dev_pids in ([dev] if n_plan == T else []) + [to_dev(pids)]:
        plan, disp = moe.moe_plan_dispatch(dev_pids, dev, E, R, C, 0)
        for name in ("replicas", "slot_base", "slot_expert"):
            assert (to_host(plan[name]) == want[name]).all(), name
        for name in ("counts", "kept", "expert_offset", "slot_offset", "perm", "inv"):
            assert (to_host(disp[name]) == rows[name]).all(), name
