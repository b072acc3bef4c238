"""The router on small batches: 16-token tiles and more wavefronts than four, at the ends of their ranges, with k that leaves wavefronts
without a step, ends inside a step, and takes several rounds."""
import pytest

import synth
from test_gpu_route_direct import test_route_direct as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,dtype,k", [
    (1, 8, 20, synth.F32, 1),                # one step for eight wavefronts; two columns per lane
    (17, 24, 36, synth.F32, 2),              # four columns; half a step at the end
    (4096, 136, 32, synth.F32, 1),           # the last tile count with 16 tokens
    (4097, 136, 32, synth.F32, 1),
    (33, 1040, 100, synth.F32, 3),           # two runs of four columns, several rounds
    (50, 2056, 128, synth.F32, 1),
    (40, 64, 22, synth.F32, 8),
    (8190, 16, 8, synth.F32, 1),             # 16 wavefronts, 32 tokens
    (1024, 1024, 16, synth.F32, 2),          # the last depths with 16 wavefronts, and the next
    (1025, 512, 3, synth.F32, 1),
    (1025, 520, 16, synth.F32, 1),
    (7, 1032, 16, synth.F32, 1),
    (1, 8, 8, synth.BF16, 1),
    (8192, 40, 32, synth.BF16, 3),
    (8193, 40, 32, synth.BF16, 1),
    (70, 1160, 64, synth.BF16, 2),
    (300, 24, 100, synth.BF16, 8),           # eight wavefronts
    (31, 2000, 120, synth.BF16, 1),
])
def test_route_few_tiles(T, d, E, dtype, k):
    check(T, d, E, dtype, k)
