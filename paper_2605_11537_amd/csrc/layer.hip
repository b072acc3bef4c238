// moe_layer_forward: the four calls of a layer in turn on one stream, the last two as one where the second product can make the output
// (ffn_makes_output).  The results are those of the calls; what it saves is four crossings of a foreign-function boundary (a Python program
// issues a layer in 15 instead of 29 us, which bounded small layers) and there a launch.
#include "route.h"

static_assert(sizeof(moe_layer_args) == 28 * 8 + 16 * 4, "no padding: callers pack it field by field");

extern "C" int moe_layer_forward(const moe_layer_args *a, void *stream)
{
    MOE_REQUIRE(a, MOE_ERR_INVALID_ARG, "moe_layer_forward: null arguments");
    MOE_REQUIRE(a->top_k >= 0 && a->top_k <= MOE_MAX_TOPK && a->T >= 0, MOE_ERR_INVALID_ARG,
                "moe_layer_forward: T=%d top_k=%d out of range", a->T, a->top_k);
    const int k = a->top_k > 0 ? a->top_k : 1;
    MOE_REQUIRE((long long)a->T * k <= 0x7fffffffLL, MOE_ERR_INVALID_ARG, "moe_layer_forward: T*k=%lld does not fit 31 bits",
                (long long)a->T * k);
    const int n = a->T * k, max_slots = a->E + a->budget;
    int rc = a->top_k > 0 ? moe_route_topk(a->x, a->w_router, a->router_layout, a->b_router, a->T, a->d, a->router_E, a->dtype, k,
                                           a->renormalize, a->expert_idx, a->expert_prob, nullptr, a->route_ws, a->route_ws_bytes,
                                           stream)
                          : moe_route(a->x, a->w_router, a->router_layout, a->b_router, a->T, a->d, a->router_E, a->dtype,
                                      a->expert_idx, a->expert_prob, nullptr, a->route_ws, a->route_ws_bytes, stream);
    if (rc != MOE_OK) return rc;
    rc = moe_plan_dispatch(a->plan_idx ? a->plan_idx : a->expert_idx, a->plan_idx ? a->n_plan : n, a->expert_idx, a->T, k, a->E, a->budget,
                           a->slot_capacity, a->policy, a->plan_counts, a->replicas, a->slot_base, a->slot_expert, a->n_slots,
                           a->counts, a->kept, a->expert_offset, a->slot_offset, a->perm, a->inv, a->row_token, a->front_ws,
                           a->front_ws_bytes, stream);
    if (rc != MOE_OK) return rc;
    // (arguments that moe_combine refuses go step by step: the products are enqueued in front of the error)
    if (a->top_k == 0 && moe::ffn_makes_output(a, max_slots) &&
        moe::combine_check(a->y_perm, a->x, a->inv, a->expert_prob, a->T, a->d, a->dtype, a->residual, a->out) == MOE_OK)
        return moe::ffn_layer(a, max_slots, stream);
    rc = a->top_k > 0 ? moe_expert_ffn_rows(a->x, a->T, a->row_token, a->w1, a->w2, a->weight_layout, a->slot_offset, a->slot_expert,
                                            a->n_slots, n, max_slots, a->E, a->d, a->F, a->dtype, a->schedule, a->y_perm, a->ffn_ws,
                                            a->ffn_ws_bytes, stream)
                      : moe_expert_ffn(a->x, a->perm, a->w1, a->w2, a->weight_layout, a->slot_offset, a->slot_expert, a->n_slots, a->T,
                                       max_slots, a->E, a->d, a->F, a->dtype, a->schedule, a->y_perm, a->ffn_ws, a->ffn_ws_bytes,
                                       stream);
    if (rc != MOE_OK) return rc;
    return a->top_k > 0 ? moe_combine_topk(a->y_perm, a->x, a->inv, a->expert_prob, a->T, k, a->d, a->dtype, a->residual, a->out, stream)
                        : moe_combine(a->y_perm, a->x, a->inv, a->expert_prob, a->T, a->d, a->dtype, a->residual, a->out, stream);
}
