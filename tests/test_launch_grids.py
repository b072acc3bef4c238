"""Launch sizes that the host computes for the worst case: enough workgroups for any slot tables, and within the launch limit
of 2^32 threads for every batch that fits the card.  The host functions are compiled from the library's headers; the deal of
tiles to the eight XCD ranges is done again in Python."""
import os
import subprocess

import numpy as np
import pytest

from gpu_util import few_rows

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SLOTS, EXPERTS = 0, 1

MAIN = """
#include "ffn_share.h"
#include <stdio.h>
int main()
{
    int a[6];
    while (scanf("%d %d %d %d %d %d", a, a + 1, a + 2, a + 3, a + 4, a + 5) == 6)
        printf("%d\\n", moe::share_grid(a[0], a[1], a[2], a[3], a[4], a[5]));
}
"""


def _compiled(tmp_path_factory, name, text):
    d = tmp_path_factory.mktemp(name)
    src, exe = str(d / "main.cpp"), str(d / "main")
    open(src, "w").write(text)
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1",
                           "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_11537_amd", "csrc"), src, "-o", exe])

    def ask(rows):
        text = "\n".join(" ".join(str(v) for v in r) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [[int(v) for v in line.split()] for line in out.splitlines()]
    return ask


@pytest.fixture(scope="module")
def share_grid(tmp_path_factory):
    return _compiled(tmp_path_factory, "share", MAIN)


def _most_units(rows_of_expert, bm, n_nt, schedule):
    """The most units one of the eight ranges of equal cost holds."""
    cost = []
    for n in rows_of_expert:
        if n <= 0:
            continue
        if schedule == EXPERTS:
            cost.append(3)
            continue
        left = n
        while left > 0:
            cost.append(3 + 2 * -(-min(left, bm) // 16))
            left -= bm
    starts = np.concatenate([[0], np.cumsum(np.repeat(np.array(cost, np.int64), n_nt))])
    edges = starts[-1] * np.arange(9) // 8
    return int(np.diff(np.searchsorted(starts[:-1], edges)).max()) if len(cost) else 0


def test_grid_holds_every_range(share_grid):
    rng = np.random.default_rng(5)
    asked, want = [], []
    for _ in range(6000):
        # 128 rows: the LDS tiles, which take the slot schedule only; 32 columns: binary32 with few units
        bm, bn, n_nt = int(rng.choice([32, 64, 128])), int(rng.choice([32, 64, 128, 256])), int(rng.integers(1, 9))
        schedule = int(rng.integers(0, 2)) if bm < 128 else SLOTS
        S = int(rng.integers(1, 60))
        kind = rng.integers(0, 4)
        rows = (rng.integers(0, 3, S) if kind == 0 else rng.integers(0, 130, S) if kind == 1
                else (rng.pareto(1.0, S) * 20).astype(int) % 3000 if kind == 2 else np.eye(S, dtype=int)[0] * 2000)
        expert = np.sort(rng.integers(0, S, S))                      # some experts own several slots
        per_expert = np.bincount(expert, weights=rows, minlength=S).astype(int)
        asked.append([bm, bn, max(1, int(rows.sum())), S, schedule, bn * n_nt])
        want.append(_most_units(per_expert, bm, n_nt, schedule))
    for a, w, (got,) in zip(asked, want, share_grid(asked)):
        assert got % 8 == 0 and got // 8 >= w, (a, w, got)


def test_long_batches_fit_a_launch(share_grid):
    """A row tile of 64 rows needs one workgroup per column tile; up to the slots' own share no batch gets many more, so that the
    launch limit is reached where the hidden rows alone fill the card (256 GB at T * N = 6.4e10)."""
    asked = [[64, 64, T, S, schedule, N] for T in (10 ** 5, 4 * 10 ** 6, 10 ** 7, 1.5e7, 3 * 10 ** 7)
             for S in (8, 256, 4096) for schedule in (SLOTS, EXPERTS) for N in (64, 1024, 2048, 4096) if T * N <= 6.2e10]
    asked = [[int(v) for v in a] for a in asked]
    for a, (got,) in zip(asked, share_grid(asked)):
        T, S, N = a[2], a[3], a[5]
        assert 0 < got <= (T // 64 + 8 * S + 8) * (N // 64) + 64, (a, got)
        assert got * 256 < 2 ** 32, (a, got)


FORMS = """
#include "sru_forms.h"
#include <stdio.h>
int main()
{
    int a[6];
    while (scanf("%d %d %d %d %d %d", a, a + 1, a + 2, a + 3, a + 4, a + 5) == 6)
        printf("%d %d\\n", moe::sru_two_kernels(a[0], a[1], a[2], a[3], a[4], a[5]), moe::fus_packs_input(a[0], a[1], a[2], a[3]));
}
"""


def test_sru_forms(tmp_path_factory):
    """The form an SRU layer takes, where the two differ by 12 % and more in measurements (sequences, positions, widths, input as
    fragments, one kernel behind), and the forms that are the only ones."""
    ask = _compiled(tmp_path_factory, "forms", FORMS)
    one = [(5, 512, 2048, 1024, 0, 0), (64, 7, 768, 256, 0, 1), (8, 1024, 256, 256, 1, 0), (8, 1024, 256, 256, 0, 1),
           (16, 1024, 128, 128, 1, 1), (1, 1024, 256, 256, 1, 0), (32, 1024, 512, 512, 1, 0), (16, 1024, 768, 256, 0, 1),
           (5, 777, 768, 256, 0, 1), (64, 1024, 384, 384, 0, 0), (64, 1024, 768, 768, 0, 0), (24, 1024, 768, 768, 0, 0)]
    two = [(1, 1025, 64, 128, 0, 0), (16, 4096, 256, 256, 1, 0), (1, 600, 1024, 256, 0, 1), (5, 777, 1024, 1024, 1, 0),
           (1, 600, 2048, 256, 0, 1), (5, 777, 2048, 256, 0, 1), (5, 777, 768, 128, 0, 1), (1, 1024, 1024, 1024, 0, 0),
           (64, 600, 1024, 1024, 0, 0), (64, 600, 2048, 512, 0, 0)]
    assert [r[0] for r in ask(one)] == [0] * len(one)
    assert [r[0] for r in ask(two)] == [1] * len(two)
    # an image of the embeddings only beside the states' in the room of the projections (16 bytes per state and channel)
    for B, L, K, n_h in [(16, 1024, 768, 256), (2, 513, 768, 128), (2, 513, 512, 128), (1, 1024, 1792, 256), (1, 1024, 1856, 256)]:
        (_, packs), = ask([(B, L, K, n_h, 0, 0)])
        assert packs == (2 * B * (-(-L // 32) * 32) * (K + n_h) <= 16 * B * L * n_h)


ROWS = """
#include "row_groups.h"
#include <stdio.h>
int main()
{
    int a[2];
    while (scanf("%d %d", a, a + 1) == 2) {
        const dim3 g = moe::rows_grid(a[0], a[1]);
        printf("%u %u\\n", g.x, g.y);
    }
}
"""


def test_rows_grid(tmp_path_factory):
    """The grid of the combine kernels stays within the limit per dimension and reaches the last row."""
    ask = _compiled(tmp_path_factory, "rows_grid", ROWS)
    asked = [[T, lg] for T in (1, 7, 64, 65536, 2 ** 22 + 1, 2 ** 27 - 1, 2 ** 27 + 5, 2 ** 31 - 1) for lg in (0, 3, 5, 8)]
    for (T, lg), (gx, gy) in zip(asked, ask(asked)):
        threads = gx * gy * 256
        assert gx * 256 < 2 ** 32 and gy < 2 ** 16 and gx * gy * (256 >> lg) < 2 ** 32
        assert T << lg <= threads < (T << lg) + (gx + 1) * 256 + 256


LANES = """
#include "row_groups.h"
#include <stdio.h>
int main()
{
    int a[3];
    while (scanf("%d %d %d", a, a + 1, a + 2) == 3) {
        const int lg = a[2] ? moe::combine_topk_lanes(a[0], a[1]) : moe::combine_lanes(a[0], a[1]);
        const dim3 g = moe::rows_grid(a[0], lg < 0 ? 5 : lg);
        printf("%d %u %u\\n", lg, g.x, g.y);
    }
}
"""


def test_row_groups(tmp_path_factory):
    """Lanes per row of the combine kernels: none idle on short rows, and a grid within the limit that reaches the last row."""
    ask = _compiled(tmp_path_factory, "lanes", LANES)
    asked = [[T, vec, topk] for T in (1, 7, 64, 2048, 2049, 4097, 65536, 2 ** 22 + 1, 2 ** 27 + 5, 2 ** 31 - 1)
             for vec in (1, 2, 3, 8, 9, 31, 32, 33, 96, 97, 255, 256, 512, 1025) for topk in (0, 1)]
    for (T, vec, topk), (lg, gx, gy) in zip(asked, ask(asked)):
        if T * vec * 16 > 2 ** 39:                       # past any card
            continue
        lanes = 1 << (5 if lg < 0 else lg)
        if vec <= 32:
            assert lg >= 0 and vec <= lanes < 2 * vec, (T, vec, lg)
        assert lanes <= 1024 and (lanes <= 256 or T <= 2048 or vec >= 256)
        assert gx * 256 < 2 ** 32 and gy < 2 ** 16
        threads = gx * gy * 256
        assert T * lanes <= threads < T * lanes + (gx + 1) * 256 + 256 and gx * gy * max(1, 256 // lanes) < 2 ** 32


FEW = """
#include "ffn_few_rows.h"
#include <stdio.h>
int main()
{
    int a[5];
    while (scanf("%d %d %d %d %d", a, a + 1, a + 2, a + 3, a + 4) == 5)
        printf("%d %d\\n", moe::ffn_few_rows(a[0], a[1], a[2], a[3]), moe::few_rows_grid(a[0], a[1], a[4], a[3]));
}
"""


def test_few_rows(tmp_path_factory):
    """Which products the kernel for few rows takes, and how many workgroups look for work: never more than are resident, nor, with one
    unit per expert that has rows, more than that many experts have column tiles."""
    ask = _compiled(tmp_path_factory, "few", FEW)
    asked = [[rows, slots, K, N, schedule] for rows in (1, 8, 37, 72, 73, 144, 500, 2048, 32768) for slots in (1, 8, 36, 144, 288, 1024)
             for K in (128, 768, 1024, 3072) for N in (128, 256, 3072) for schedule in (SLOTS, EXPERTS) if rows <= 64 * slots]
    for (rows, slots, K, N, schedule), (takes, grid) in zip(asked, ask(asked)):
        assert takes == few_rows(rows, slots, K, N)
        units = (min(rows, slots) + (rows // 32 if schedule == SLOTS else 0)) * (N // 32)
        assert grid == min(-(-units // 8) * 8, 256 * (3 if schedule == SLOTS else 2))


F32 = """
#include "ffn_f32.h"
#include <stdio.h>
int main()
{
    int a[7];
    while (scanf("%d %d %d %d %d %d %d", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6) == 7)
        printf("%d %d %d\\n", moe::f32_depth(a[4]), moe::f32_rows(a[1], a[6]), moe::f32_grid(a[0], a[1], a[2], a[3], a[4], a[5]));
}
"""


def test_f32_grid(share_grid, tmp_path_factory):
    """binary32 products: a workgroup per unit from k = 320 on, at most a few per compute unit below."""
    ask = _compiled(tmp_path_factory, "f32", F32)
    asked = [[bm, rows, slots, schedule, K, N, E] for bm in (0, 32, 64) for rows in (1, 100, 16384) for slots in (1, 40, 600)
             for schedule in (SLOTS, EXPERTS) for K in (64, 192, 256, 320, 2048) for N in (64, 2048) for E in (8, 128)]
    each = share_grid([[a[0] or 32, 64, a[1], a[2], a[3], a[5]] for a in asked])
    for (bm, rows, slots, schedule, K, N, E), (all_,), (depth, height, grid) in zip(asked, each, ask(asked)):
        assert depth == (1 if K < 256 else 4) and height == (64 if rows >= 128 * E else 32)
        assert grid == (all_ if K > 256 else min(all_, 256 * {0: 4, 32: 6, 64: 4}[bm])) and grid % 8 == 0
