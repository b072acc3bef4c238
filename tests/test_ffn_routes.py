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
        printf("%d %d %d %d %d %d %d %d %d %d %d %d %d\\n", (int)b.kernel, b.list, b.few_rows[0], b.few_rows[1], bm,
               moe::f32_narrow(r, s, E, sched, d, F), moe::f32_narrow(r, s, E, sched, F, d),
               moe::f32_staged(bm, r, s, E, sched, d, F), moe::f32_staged(bm, r, s, E, sched, F, d), moe::f32_depth(F), moe::f32_several(F),
               moe::ffn_output_pays(r, s, E, d, F, MOE_F32, sched), moe::ffn_output_pays(r, s, E, d, F, MOE_BF16, sched));
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    ask = _compiled(tmp_path_factory, "rules", RULES)

    def of(rows, slots, E, d, F, schedule=SLOTS):
        (kernel, listed, few1, few2, bm, narrow1, narrow2, staged1, staged2, depth2, several2, out32, out16), = ask(
            [[rows, slots, E, d, F, schedule]])
        bf16 = {0: "columns listed" if listed else "few rows" if few1 and few2 else "columns", 1: "dense", 2: "lds"}[kernel]
        second = ("32 columns" if narrow2 else "32 rows, short k" if depth2 == 1 else f"{bm} rows, staged" if staged2
                  else f"{bm} rows, several units" if several2 else f"{bm} rows")
        return bf16, dict(bm=bm, narrow=(narrow1, narrow2), staged=(staged1, staged2), few=(few1, few2), second=second, output=(out32, out16))
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


def test_layer_output_cases(rules):
    """The layers of the output tests: the second product's kernel, and whether it makes the output; every kernel that can is there."""
    from test_gpu_layer_output import CASES
    made = set()
    for (name, T, d, F, E, R, _), kernel, makes in CASES:
        bf16, more = rules(T, E + R, E, d, F)
        takes = more["second"] if name == "f32" else "few rows" if more["few"][1] else bf16
        assert takes == kernel and more["output"][name == "bf16"] == makes, (name, T, d, F, E, R, takes, more["output"])
        assert rules(T, E + R, E, d, F, EXPERTS)[1]["output"] == (0, 0)
        if makes:
            made.add((name, kernel))
    assert made == {("f32", k) for k in ("32 columns", "32 rows, short k", "32 rows, staged", "64 rows, staged", "32 rows, several units",
                                         "64 rows, several units", "32 rows", "64 rows")} | {("bf16", "columns"), ("bf16", "columns listed")}


APART = """
#include "ffn_rules.h"
#include <stdio.h>
int main()
{
    // a layer whose buffers stand one after another, and an output at a byte of that row
    int T, d, F, E, budget, f32, which;
    long long shift;
    while (scanf("%d %d %d %d %d %d %d %lld", &T, &d, &F, &E, &budget, &f32, &which, &shift) == 8) {
        const size_t esz = f32 ? 4 : 2, slots = E + budget, ws = (size_t)T * F * esz + 4096;
        const size_t bytes[] = {ws, (size_t)E * F * d * esz, (size_t)T * 4, (slots + 1) * 4, slots * 4, 4, (size_t)T * 4, (size_t)E * F * d * esz};
        char *at[8], *next = (char *)(1ull << 40);
        for (int i = 0; i < 8; ++i) {
            at[i] = next;
            next += bytes[i] + 2 * (size_t)T * d * esz;
        }
        moe_layer_args a = {};
        a.T = T, a.d = d, a.F = F, a.E = E, a.budget = budget, a.dtype = f32 ? MOE_F32 : MOE_BF16;
        a.ffn_ws = at[0], a.w2 = at[1], a.perm = (int32_t *)at[2], a.slot_offset = (int32_t *)at[3], a.slot_expert = (int32_t *)at[4];
        a.n_slots = (int32_t *)at[5], a.replicas = (int32_t *)at[6], a.w1 = at[7];
        // shift < 0: that many bytes of the output in front of the buffer; >= 0: the output begins there, from its end if beyond 1 << 40
        a.out = at[which] + (shift >= 1ll << 40 ? (long long)bytes[which] + (shift - (1ll << 41)) : shift);
        a.ffn_ws_bytes = 1ull << 60;
        printf("%d\\n", moe::ffn_output_apart(&a, (int)slots, ws));
    }
}
"""


@pytest.mark.parametrize("T,d,F,E,budget,f32", [(64, 64, 256, 8, 2, 1), (1500, 128, 128, 64, 0, 0), (1, 128, 64, 1, 0, 1)])
def test_an_output_in_the_second_product_s_operands(tmp_path_factory, T, d, F, E, budget, f32):
    """Workspace, second weights, the permutation and the slot tables: an output that meets one of them by a byte is not made by the product."""
    ask = _compiled(tmp_path_factory, "apart", APART)
    end, out = 1 << 41, T * d * (4 if f32 else 2)
    for which in range(8):
        read = which < 6                                 # the others are free: replica counts, first weights
        at = [0, -out + 1, -1, end - 1, -out, end]
        got = [v for v, in ask([[T, d, F, E, budget, f32, which, a] for a in at])]
        assert got == [int(not read)] * 4 + [1, 1], (which, got)
