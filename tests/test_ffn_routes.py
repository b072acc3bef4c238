"""Which kernel the expert products of a shape take, asked of the library's rules compiled for the host: every shape that a GPU test brings for one
kernel takes that one."""
import pytest

from ffn_shapes import BAD_ROWS, BAD_TABLES, FFN_KERNEL, FFN_SHAPES
from test_launch_grids import EXPERTS, SLOTS, _compiled

RULES = """
#include "ffn_rules.h"
#include "ffn_f32.h"
#include <stdio.h>
int main()
{
    int r, s, E, d, F, sched;
    while (scanf("%d %d %d %d %d %d", &r, &s, &E, &d, &F, &sched) == 6) {
        const moe::FfnRoute b = moe::ffn_route(r, s, E, d, F, sched);
        const int bm = moe::f32_rows(r, E);
        printf("%d %d %d %d %d %d %d %d %d\\n", (int)b.kernel, b.list, b.few_rows[0], b.few_rows[1], bm,
               moe::f32_narrow(r, s, E, sched, d, F), moe::f32_narrow(r, s, E, sched, F, d),
               moe::f32_staged(bm, r, s, E, sched, d, F), moe::f32_staged(bm, r, s, E, sched, F, d));
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    ask = _compiled(tmp_path_factory, "rules", RULES)

    def of(rows, slots, E, d, F, schedule=SLOTS):
        (kernel, listed, few1, few2, bm, narrow1, narrow2, staged1, staged2), = ask([[rows, slots, E, d, F, schedule]])
        bf16 = {0: "columns listed" if listed else "few rows" if few1 and few2 else "columns", 1: "dense", 2: "lds"}[kernel]
        return bf16, dict(bm=bm, narrow=(narrow1, narrow2), staged=(staged1, staged2), few=(few1, few2))
    return of


@pytest.mark.parametrize("name", list(FFN_SHAPES))
def test_shapes_take_their_kernel(rules, name):
    E, d, F, rows, experts, behind = FFN_SHAPES[name]
    assert len(rows) == len(experts) and max(experts) < E
    assert rules(sum(rows) + behind, len(rows), E, d, F)[0] == FFN_KERNEL[name]
    assert rules(sum(rows) + behind, len(rows), E, d, F, EXPERTS)[0].startswith("columns")


@pytest.mark.parametrize("name,d,F,scale,empty,experts", BAD_TABLES)
@pytest.mark.parametrize("rows", BAD_ROWS)
def test_bad_tables_take_their_kernel(rules, name, d, F, scale, empty, experts, rows):
    n, slots, E = sum(rows) * scale, len(rows) + empty, max(experts, 6 if len(rows) == 9 else 4)
    bf16, f32 = rules(n, slots, E, d, F)
    if not name.startswith("f32"):
        assert bf16 == name
    elif name == "f32 short":
        assert f32["bm"] == 32 and f32["narrow"] == f32["staged"] == (0, 0)
    elif name == "f32 64 rows":
        assert f32["bm"] == 64 and f32["staged"] == (0, 0)
    elif name == "f32 staged":
        assert f32["bm"] == 64 and f32["staged"] == (1, 1)
    else:
        assert f32["narrow"] == (1, 1)


def test_f32_staged_shapes(rules):
    """The shapes of the staged tests: narrow, staged on 32 and on 64 rows, and neither."""
    from test_gpu_ffn_f32_staged import SHAPES
    for (d, F, E, rows, _, _), (bm, narrow, staged) in SHAPES:
        _, f32 = rules(sum(rows) + 3, len(rows), E, d, F)
        assert (f32["bm"], f32["narrow"], f32["staged"]) == (bm, narrow, staged), (d, F, rows)


def test_lds_shapes(rules):
    from test_gpu_ffn_lds_tile import SHAPES
    for d, F, E, rows, *_ in SHAPES:
        assert rules(sum(rows) + 3, len(rows), E, d, F)[0] == "lds", (d, F, rows)
