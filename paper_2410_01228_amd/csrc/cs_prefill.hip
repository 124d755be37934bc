// Kernels, launch plan and launcher of the prefill-chunk path (the workgroup's work itself is
// in cs_prefill_impl.h, shared with the fused mixed-batch kernel).
#include "cs_prefill_impl.h"

namespace cs {

// grid.x = slots * Hkv, kv head fastest (the slots from base_slot on: no sequence before it has a
// chunk); grid.y = key ranges; grid.z = layers
template <int D, class E, int PS, bool kMayCut>
__global__ __launch_bounds__(kPrefillThreads, 2) void prefill_kernel(
    const uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t G, int32_t S,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ q, uint16_t* __restrict__ out, float scale_log2e,
    int32_t range_steps, int32_t base_slot, float* __restrict__ part, uint64_t launch, int32_t n_ordered, const SlotOrder order,
    int32_t backwards, int64_t next_layer, int64_t next_q, int64_t next_part)
{
    __shared__ PrefillLds<D> lds;
    const int32_t pos = blockIdx.x / Hkv;
    const int32_t g = blockIdx.x - pos * Hkv;
    const int32_t b = n_ordered > 0 ? (int32_t)order.slot[pos]
                                    : base_slot + (backwards ? (int32_t)(gridDim.x / Hkv) - 1 - pos : pos);
    // (with key ranges the grid has no order table: cut position = slot position)
    prefill_tile<D, E, 1, PS, false, kMayCut>(lds, layer_base + blockIdx.z * next_layer, page_stride, num_pages, Hkv, G, S, block_tables, max_blocks, ctx_lens, cu_q_lens,
                       q + blockIdx.z * next_q, out + blockIdx.z * next_q, scale_log2e, range_steps,
                       partials_of<D>(part + blockIdx.z * next_part, b - base_slot, Hkv, g, gridDim.y), launch, g, b,
                       blockIdx.y);
}

// (plan_prefill, the host plan of the key-range split and the tile order, is in cs_api.hip with
// the other launch planning.)

template <class E>
static int launch_prefill_as(const cs_kv_pool& pool, int32_t layer, const LayerSpan& span, const cs_batch& b, const PrefillPlan& plan,
                             const void* q, void* out, int32_t Hq, float scale, void* workspace, hipStream_t st)
{
    const int32_t Hkv = pool.num_kv_heads, D = pool.head_dim, G = Hq / Hkv;
    const uint16_t* layer_base = (const uint16_t*)pool.base + (int64_t)layer * pool.layer_stride;
    const float scale_log2e = scale * 1.4426950408889634f;
    if ((int64_t)plan.num_slots * Hkv > 2147483647ll || plan.max_ranges > 65535) return CS_ERR_UNSUPPORTED;
    const uint32_t slots = plan.n_ordered > 0 ? (uint32_t)plan.n_ordered : (uint32_t)plan.num_slots;
    dim3 grid((uint32_t)Hkv * slots, (uint32_t)plan.max_ranges, (uint32_t)span.n);
    const int64_t next_part = (int64_t)(plan.bytes / sizeof(float)) / span.n;
    float* part = (float*)workspace;
#define CS_LAUNCH_PREFILL_C(DD, PS, CUT)                                                                            \
    hipLaunchKernelGGL((prefill_kernel<DD, E, PS, CUT>), grid, dim3(kPrefillThreads), 0, st, layer_base, pool.page_stride, \
                       pool.num_pages, Hkv, G, b.num_seqs, b.block_tables, b.max_blocks_per_seq,                   \
                       b.ctx_lens, b.cu_q_lens, (const uint16_t*)q, (uint16_t*)out, scale_log2e,                   \
                       plan.range_steps, plan.base_slot, part, next_launch_number(), plan.n_ordered, plan.order, (int32_t)plan.backwards, \
                       span.pool, span.q, next_part);
#define CS_LAUNCH_PREFILL(DD, PS)                                                                                   \
    if (plan.max_ranges > 1) { CS_LAUNCH_PREFILL_C(DD, PS, true) } else { CS_LAUNCH_PREFILL_C(DD, PS, false) }
    if (pool.page_size == 16) { if (D == 128) { CS_LAUNCH_PREFILL(128, 16) } else { CS_LAUNCH_PREFILL(64, 16) } }
    else                      { if (D == 128) { CS_LAUNCH_PREFILL(128, 8) } else { CS_LAUNCH_PREFILL(64, 8) } }
#undef CS_LAUNCH_PREFILL
#undef CS_LAUNCH_PREFILL_C
    return check_launch("prefill kernels");
}

int launch_prefill_layers(const cs_kv_pool& pool, int32_t layer, const LayerSpan& span, const cs_batch& b, const PrefillPlan& plan,
                          const void* q, void* out, int32_t Hq, float scale, void* workspace, hipStream_t st, bool f16)
{
    return f16 ? launch_prefill_as<F16>(pool, layer, span, b, plan, q, out, Hq, scale, workspace, st)
               : launch_prefill_as<Bf16>(pool, layer, span, b, plan, q, out, Hq, scale, workspace, st);
}

int launch_prefill(const cs_kv_pool& pool, int32_t layer, const cs_batch& b, const PrefillPlan& plan,
                   const void* q, void* out, int32_t Hq, float scale, void* workspace, hipStream_t st, bool f16)
{
    return launch_prefill_layers(pool, layer, LayerSpan{1, 0, 0, 0}, b, plan, q, out, Hq, scale, workspace, st, f16);
}

}  // namespace cs
