// cs_run_layers: one iteration's layers with the safepoints of layer-wise preemption between them
// (paper Sec. 4.3, Alg. 1).  Host code only.
#include <algorithm>
#include "cs_plan.h"

using namespace cs;

// Between two safepoints the batch cannot change and the caller has all layers' inputs in place, so up
// to this many layers go into one append launch, and into one attention launch where the workspace
// holds the partial results of all of them.  A small step's layer is mostly start-up, tail and the
// gaps between its launches.  Every layer is cut as in a launch of its own, so its results are, bit for
// bit, those of cs_kv_append + cs_paged_attention_mixed, whatever shares its launch.
constexpr int32_t kLayersPerLaunch = 4;

// Whether the layers' tensors can be worked on in any order: every layer has an output of its own,
// which is no other layer's input (a caller may hand one buffer to all layers, or chain them), and all
// are aligned as the single calls ask.  (Only then; otherwise layer after layer.)
static bool layers_are_apart(const cs_batch& b, int32_t layers, const void* q, const void* k_new, const void* v_new, const void* out,
                             int64_t q_stride, int64_t kv_stride, int32_t Hq, int32_t Hkv, int32_t D) {
    const int64_t q_elems = (int64_t)b.num_tokens * Hq * D, kv_elems = (int64_t)b.num_tokens * Hkv * D;
    if (((uintptr_t)q | (uintptr_t)out | (uintptr_t)k_new | (uintptr_t)v_new) & 15 || (q_stride | kv_stride) & 7) return false;
    if (q_stride < q_elems) return false;
    auto end = [&](const void* p, int64_t stride, int64_t elems) { return (uintptr_t)p + 2 * ((layers - 1) * stride + elems); };
    auto clear_of_out = [&](const void* p, int64_t stride, int64_t elems) {
        return end(p, stride, elems) <= (uintptr_t)out || end(out, q_stride, q_elems) <= (uintptr_t)p;
    };
    return (q == out || clear_of_out(q, q_stride, q_elems)) && clear_of_out(k_new, kv_stride, kv_elems) &&
           clear_of_out(v_new, kv_stride, kv_elems);
}

// Attention of layers [l, l + n) in one launch; the workspace holds what it needs
// (workspace_for_layers), and its pointer has been checked if that is anything: several layers need
// memory only where one does.
static int attention_of_layers(const cs_kv_pool& pool, int32_t l, int32_t n, const cs_batch& b, const void* q, void* out,
                               int64_t q_stride, int32_t Hq, float scale, void* workspace, hipStream_t st, bool f16) {
    const Plans& plans = plans_for(&b, Hq, pool.num_kv_heads, pool.head_dim, n);
    const LayerSpan span = {n, pool.layer_stride, q_stride, 0};
    void* prefill_ws = (char*)workspace + plans.decode_bytes;
    if (plans.f.arrangement != 0) {
        int rc = launch_mixed_layers(pool, l, span, b, plans.d, plans.p, q, out, Hq, scale, workspace, prefill_ws, st, f16,
                                     plans.f.prio, plans.f.arrangement == 2 ? plans.f.persistent_wgs : 0);
        if (rc == CS_OK && plans.p.max_ranges > 1 && !plans.p.merges_in_place)
            rc = launch_prefill_merge(pool, span, b, plans.p, out, Hq, prefill_ws, st, f16);
        if (rc || plans.d.num_multi == 0 || plans.d.merges_in_place) return rc;
        return launch_decode_layers(pool, l, span, b, plans.d, q, out, Hq, scale, workspace, st, f16, true);
    }
    if (plans.d.num_prefill > 0) {
        const int rc = launch_prefill_layers(pool, l, span, b, plans.p, q, out, Hq, scale, prefill_ws, st, f16);
        if (rc) return rc;
    }
    return launch_decode_layers(pool, l, span, b, plans.d, q, out, Hq, scale, workspace, st, f16, false);
}

static int run_layers(const cs_kv_pool* pool, int32_t l0, int32_t l1, const cs_batch* batch,
                      const void* q, const void* k_new, const void* v_new, void* out,
                      int64_t q_stride, int64_t kv_stride, int32_t Hq, float scale,
                      void* workspace, size_t workspace_bytes, const cs_safepoint* sp,
                      int32_t* preempted_before_layer, void* stream, bool f16) {
    if (preempted_before_layer) *preempted_before_layer = -1;
    int rc = validate_pool(pool);
    if (rc) return rc;
    if (l0 < 0 || l1 < l0 || l1 > pool->num_layers || q_stride < 0 || kv_stride < 0) return CS_ERR_INVALID_ARG;
    rc = validate_batch(pool, batch);
    if (rc) return rc;
    if (sp && (sp->check_every <= 0 || sp->num_online_seqs < 0 || sp->num_online_seqs > batch->num_seqs))
        return CS_ERR_INVALID_ARG;
    // Everything that can refuse the iteration is checked before its first layer is enqueued.  The
    // workspace must hold the full batch's plan AND the online prefix's: fewer sequences are cut
    // finer (more partials), so the prefix can need more than the whole.
    if (l1 > l0 && batch->num_tokens > 0) {
        rc = attention_shape_ok(Hq, pool->num_kv_heads, pool->head_dim);
        if (rc) return rc;
        if (!q || !out || !k_new || !v_new) return CS_ERR_INVALID_ARG;
        if (!(scale > 0.f) || scale > 3.0e38f) return CS_ERR_INVALID_ARG;
        const size_t need = cs_run_layers_workspace_bytes(batch, sp ? sp->num_online_seqs : 0, Hq, pool->num_kv_heads,
                                                          pool->head_dim);
        if (need > 0 && (!workspace || ((uintptr_t)workspace & 15))) return CS_ERR_INVALID_ARG;
        if (workspace_bytes < need) return CS_ERR_WORKSPACE_TOO_SMALL;
    }
    cs_batch cur = *batch;
    bool preempted = false;
    const bool apart = l1 > l0 && batch->num_tokens > 0 &&
                       layers_are_apart(*batch, l1 - l0, q, k_new, v_new, out, q_stride, kv_stride, Hq, pool->num_kv_heads,
                                        pool->head_dim);
    for (int32_t l = l0; l < l1;) {
        if (sp && !preempted && (l - l0) % sp->check_every == 0) {
            // safepoint: between two layers nothing of the iteration is half done
            if (sp->sync_at_safepoint) {
                const hipError_t e = hipStreamSynchronize((hipStream_t)stream);
                if (e != hipSuccess) return hip_failed(e, "safepoint synchronise");
            }
            bool raise = sp->flag && *sp->flag != 0;
            if (!raise && sp->poll) raise = sp->poll(sp->poll_arg) != 0;
            if (raise) {
                // drop the offline tail: same arrays, fewer sequences
                preempted = true;
                cur = online_prefix(*batch, sp->num_online_seqs);
                if (preempted_before_layer) *preempted_before_layer = l;
            }
        }
        auto q_of = [&](const void* base, int32_t layer) { return (uint16_t*)base + (int64_t)(layer - l0) * q_stride; };
        auto kv_of = [&](const void* base, int32_t layer) { return (const uint16_t*)base + (int64_t)(layer - l0) * kv_stride; };
        int32_t n = apart ? std::min(kLayersPerLaunch, l1 - l) : 1;
        if (sp && !preempted) n = std::min(n, sp->check_every - (l - l0) % sp->check_every);
        if (n > 1 && cur.num_tokens == 0) {                // no online work left
            l += n;
            continue;
        }
        if (n > 1) {
            const LayerSpan span = {n, pool->layer_stride, q_stride, kv_stride};
            rc = launch_append_layers(*pool, l, span, cur, kv_of(k_new, l), kv_of(v_new, l), (hipStream_t)stream);
        } else {
            rc = cs_kv_append(pool, l, &cur, kv_of(k_new, l), kv_of(v_new, l), stream);
        }
        if (rc) return rc;
        // their attention, as many of them at a time as the workspace has room for
        for (const int32_t end = l + n; l < end; l += n) {
            n = end - l;
            while (n > 1 && workspace_for_layers(&cur, Hq, pool->num_kv_heads, pool->head_dim, n) > workspace_bytes) --n;
            rc = n > 1 ? attention_of_layers(*pool, l, n, cur, q_of(q, l), q_of(out, l), q_stride, Hq, scale, workspace, (hipStream_t)stream, f16)
                       : attention_mixed(pool, l, &cur, q_of(q, l), q_of(out, l), Hq, scale, workspace, workspace_bytes, stream, f16);
            if (rc) return rc;
        }
    }
    return CS_OK;
}

extern "C" {

int cs_run_layers(const cs_kv_pool* pool, int32_t l0, int32_t l1, const cs_batch* batch,
                  const void* q, const void* k_new, const void* v_new, void* out,
                  int64_t q_stride, int64_t kv_stride, int32_t Hq, float scale,
                  void* workspace, size_t workspace_bytes, const cs_safepoint* sp,
                  int32_t* preempted_before_layer, void* stream) {
    return run_layers(pool, l0, l1, batch, q, k_new, v_new, out, q_stride, kv_stride, Hq, scale, workspace,
                      workspace_bytes, sp, preempted_before_layer, stream, false);
}

int cs_run_layers_f16(const cs_kv_pool* pool, int32_t l0, int32_t l1, const cs_batch* batch,
                      const void* q, const void* k_new, const void* v_new, void* out,
                      int64_t q_stride, int64_t kv_stride, int32_t Hq, float scale,
                      void* workspace, size_t workspace_bytes, const cs_safepoint* sp,
                      int32_t* preempted_before_layer, void* stream) {
    return run_layers(pool, l0, l1, batch, q, k_new, v_new, out, q_stride, kv_stride, Hq, scale, workspace,
                      workspace_bytes, sp, preempted_before_layer, stream, true);
}

}  // extern "C"
