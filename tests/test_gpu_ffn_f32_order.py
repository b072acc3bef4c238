"""The binary32 expert products sum a row in one order of k, whatever kernel takes them: both schedules and every batch size give the same bits."""
import numpy as np
import pytest
import torch

import oracle  # noqa: F401  (built before the GPU is touched)
import synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F", [
    (64, 256),               # short k, then k = 256 with tiles of 32 columns for small batches
    (256, 1024),
    (512, 384),              # dealt in pairs of steps, three to a wavefront
    (320, 448),              # quarters: no whole number of pairs
    (1024, 256),
])
def test_schedules_and_batch_sizes_give_the_same_bits(d, F):
    import paper_2605_11537_amd as moe
    E, rows = 4, [37, 300, 1, 70]                                    # small batch: the first 20 rows of every expert
    w1, w2 = (to_dev(synth.normal_tensor(s, 0.1, [k, d, F], synth.F32)) for k, s in ((1, (E, d, F)), (2, (E, F, d))))
    x = torch.from_numpy(synth.normal_tensor((sum(rows), d), 1.0, [3, d, F], synth.F32)).cuda()

    def run(xs, counts, schedule, copies=1):
        # copies: every expert's rows that many times, one after another
        so = to_dev(np.concatenate([[0], np.cumsum([c * copies for c in counts])]).astype(np.int32))
        parts = [p.repeat(copies, 1) for p in torch.split(xs, counts)]
        y = moe.moe_expert_ffn(torch.cat(parts).contiguous(), w1, w2, so, to_dev(np.arange(E, dtype=np.int32)),
                               torch.tensor([E], dtype=torch.int32, device="cuda"), E, F, schedule=schedule)
        return [p[:c] for p, c in zip(torch.split(y, [c * copies for c in counts]), counts)]

    slots = run(x, rows, moe.SCHEDULE_SLOTS)
    few = [min(c, 20) for c in rows]
    first = torch.cat([p[:n] for p, n in zip(torch.split(x, rows), few)])
    for other, n in ((run(x, rows, moe.SCHEDULE_EXPERTS), rows), (run(x, rows, moe.SCHEDULE_SLOTS, 2), rows),
                     (run(x, rows, moe.SCHEDULE_SLOTS, 8), rows), (run(first, few, moe.SCHEDULE_SLOTS), few),
                     (run(first, few, moe.SCHEDULE_EXPERTS), few)):
        for e in range(E):
            assert torch.equal(other[e], slots[e][:n[e]]), f"expert {e}"
