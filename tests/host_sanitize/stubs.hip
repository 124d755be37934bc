// Stand-ins for the kernel launchers, so that the kernel-free host part of the library (argument
// checks, launch planning, the iteration over layers, the page map) links without any device code.
// Most of the driver's calls return before a launch: reaching one of these is a test failure then.
// For the iterations that do launch, the driver opens a LaunchWindow, and every launch is held
// against the workspace that the caller brought.
#include <cstdio>
#include <cstdlib>
#include "cs_common.h"
#include "launch_window.h"

LaunchWindow g_window;

namespace cs {

[[noreturn]] static void fail(const char* what) {
    std::fprintf(stderr, "kernel launcher %s\n", what);
    std::abort();
}

static void used(const char* what, const void* ws, size_t bytes) {
    if (!g_window.open) { std::fprintf(stderr, "host-only test reached: %s\n", what); fail("reached outside a window"); }
    if (bytes == 0) return;
    const uintptr_t p = (uintptr_t)ws, w = (uintptr_t)g_window.workspace;
    if (w == 0 || (w & 15)) fail("given scratch work without a usable workspace");
    if ((p & 15) || p < w || p + bytes > w + g_window.bytes) fail("given scratch work outside the workspace");
}

int launch_append(const cs_kv_pool&, int32_t, const cs_batch&, const void*, const void*, hipStream_t) {
    used("append", nullptr, 0);
    ++g_window.layers_appended;
    return CS_OK;
}
int launch_append_layers(const cs_kv_pool&, int32_t, const LayerSpan& span, const cs_batch&, const void*, const void*, hipStream_t) {
    used("append of layers", nullptr, 0);
    g_window.layers_appended += span.n;
    return CS_OK;
}
int launch_page_copy(const cs_kv_pool&, int32_t, int32_t, const int32_t*, int32_t, void*, bool, hipStream_t, bool) { fail("reached: page copy"); }
int launch_token_copy(const cs_kv_pool&, int32_t, int32_t, const int32_t*, int32_t, void*, bool, hipStream_t) { fail("reached: token copy"); }
int launch_plain_copy(void*, const void*, size_t, hipStream_t) { fail("reached: plain copy"); }

int launch_decode_layers(const cs_kv_pool& pool, int32_t, const LayerSpan& span, const cs_batch&, const DecodePlan& plan, const void*, void*,
                         int32_t Hq, float, void* ws, hipStream_t, bool, bool merge_only) {
    used("decode", ws, decode_workspace(plan, Hq, pool.num_kv_heads, pool.head_dim, span.n).total);
    if (plan.num_decode > 0 && !merge_only) g_window.layers_decoded += span.n;
    return CS_OK;
}
int launch_prefill_layers(const cs_kv_pool&, int32_t, const LayerSpan& span, const cs_batch&, const PrefillPlan& plan, const void*, void*,
                          int32_t, float, void* ws, hipStream_t, bool) {
    used("prefill", ws, plan.bytes);
    g_window.layers_prefilled += span.n;
    return CS_OK;
}
int launch_mixed_layers(const cs_kv_pool& pool, int32_t, const LayerSpan& span, const cs_batch&, const DecodePlan& dplan,
                        const PrefillPlan& pplan, const void*, void*, int32_t Hq, float, void* decode_ws, void* prefill_ws, hipStream_t, bool,
                        int32_t, int32_t) {
    used("mixed: decode side", decode_ws, decode_workspace(dplan, Hq, pool.num_kv_heads, pool.head_dim, span.n).total);
    used("mixed: tiles", prefill_ws, pplan.bytes);
    g_window.layers_decoded += span.n;
    g_window.layers_prefilled += span.n;
    return CS_OK;
}

int launch_prefill_merge(const cs_kv_pool&, const LayerSpan&, const cs_batch&, const PrefillPlan& plan, void*, int32_t, void* ws, hipStream_t, bool) {
    used("prefill merge", ws, plan.bytes);
    if (plan.max_ranges <= 1 || plan.merges_in_place) fail("given a merge that nobody needs");
    return CS_OK;
}

int launch_decode(const cs_kv_pool& pool, int32_t layer, const cs_batch& b, const DecodePlan& plan, const void* q, void* out, int32_t Hq,
                  float scale, void* ws, hipStream_t st, bool f16, bool merge_only) {
    return launch_decode_layers(pool, layer, LayerSpan{1, 0, 0, 0}, b, plan, q, out, Hq, scale, ws, st, f16, merge_only);
}
int launch_prefill(const cs_kv_pool& pool, int32_t layer, const cs_batch& b, const PrefillPlan& plan, const void* q, void* out, int32_t Hq,
                   float scale, void* ws, hipStream_t st, bool f16) {
    return launch_prefill_layers(pool, layer, LayerSpan{1, 0, 0, 0}, b, plan, q, out, Hq, scale, ws, st, f16);
}
int launch_mixed(const cs_kv_pool& pool, int32_t layer, const cs_batch& b, const DecodePlan& dplan, const PrefillPlan& pplan, const void* q,
                 void* out, int32_t Hq, float scale, void* decode_ws, void* prefill_ws, hipStream_t st, bool f16, int32_t prio, int32_t wgs) {
    return launch_mixed_layers(pool, layer, LayerSpan{1, 0, 0, 0}, b, dplan, pplan, q, out, Hq, scale, decode_ws, prefill_ws, st, f16, prio, wgs);
}

}  // namespace cs
