// Kernels and launcher of the decode path (the workgroup's work itself is in
// cs_decode_impl.h, shared with the fused mixed-batch kernel).
#include "cs_decode_impl.h"

namespace cs {

constexpr int kPlanThreads = 1024;

__global__ __launch_bounds__(kPlanThreads) void decode_plan_kernel(
    int32_t S, const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    int32_t split_tokens, int32_t total_items, DecodeItem* __restrict__ items)
{
    // total_items is what the host planned from its copies of the lengths; it bounds every write
    // here should the device arrays disagree with those copies
    __shared__ int32_t sh_items[kPlanThreads];
    const int tid = threadIdx.x;
    const int32_t per = (S + kPlanThreads - 1) / kPlanThreads;
    const int32_t s0 = min(S, tid * per), s1 = min(S, s0 + per);
    int32_t n_items = 0;
    for (int32_t s = s0; s < s1; ++s) {
        if (cu_q_lens[s + 1] - cu_q_lens[s] != 1) continue;
        n_items += decode_num_splits(ctx_lens[s] + 1, split_tokens);
    }
    sh_items[tid] = n_items;
    __syncthreads();
    for (int off = 1; off < kPlanThreads; off <<= 1) {           // inclusive scan
        const int32_t a = tid >= off ? sh_items[tid - off] : 0;
        __syncthreads();
        sh_items[tid] += a;
        __syncthreads();
    }
    int32_t item = sh_items[tid] - n_items;                                // exclusive
    for (int32_t s = s0; s < s1; ++s) {
        const int32_t t = cu_q_lens[s];
        if (cu_q_lens[s + 1] - t != 1) continue;
        const int32_t n = ctx_lens[s] + 1;
        const int32_t k = decode_num_splits(n, split_tokens);
        const int32_t chunk = decode_chunk_keys(n, k);
        for (int32_t i = 0; i < k; ++i) {
            DecodeItem it;
            it.seq = s; it.token = t; it.n_keys = n;
            it.key_begin = min(n, i * chunk);
            it.key_end = min(n, (i + 1) * chunk);
            it.n_splits = k; it.first_item = item; it.pad = 0;
            if (item + i < total_items) items[item + i] = it;
        }
        item += k;
    }
}

// grid = (items * Hkv, layers) workgroups, kv head fastest (the heads of one page are neighbours
// in memory, so neighbouring workgroups share DRAM pages and translations).
// kCut: a list in the arguments that holds pieces, which part.words may ask to merge in place.  (Launches
// without cuts run pages of 8 tokens 4% faster without that code: 137 sequences of 47-349 keys, 64/8 heads,
// 27.0 -> 26.1 us.  Cut lists that a kernel merges are faster with it: 64 of 1K-8K keys, 28/4 heads, the
// append included, 112.7 -> 109.4 us.)
template <int D, class Src, class E, int kAhead, int PS, bool kCut, Loads kLoads>
__device__ __forceinline__ void split_workgroup(
    const uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t G,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const Src& src,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ q, uint16_t* __restrict__ out,
    float scale_log2e, const DecodePartials& part, int64_t next_layer, int64_t next_q)
{
    __shared__ DecodeLds<D> lds;
    const int32_t item = blockIdx.x / Hkv, g = blockIdx.x - item * Hkv, n_items = gridDim.x / Hkv;
    const DecodePartials mine = part.of_layer(blockIdx.y, n_items, Hkv * G, Hkv, D);
    out += blockIdx.y * next_q;
    decode_item<D, Src, E, kAhead, PS, kLoads>(lds, layer_base + blockIdx.y * next_layer, page_stride, num_pages, Hkv, G, block_tables, max_blocks, src, ctx_lens,
                           cu_q_lens, q + blockIdx.y * next_q, out, scale_log2e, mine, item, g);
    if constexpr (kCut) {
        if (part.words) merge_in_place<D, E>(lds, mine, src, item, g, ctx_lens, cu_q_lens, Hkv, G, out);
    }
}

template <int D, class Src, class E, int kAhead, int PS, bool kCut>
__global__ __launch_bounds__(kDecodeThreads, 2) void decode_split_kernel(
    const uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t G,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const Src src,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ q, uint16_t* __restrict__ out,
    float scale_log2e, const DecodePartials part, int64_t next_layer, int64_t next_q)
{
    split_workgroup<D, Src, E, kAhead, PS, kCut, Loads::kSkipped>(layer_base, page_stride, num_pages, Hkv, G, block_tables, max_blocks, src, ctx_lens,
                                                        cu_q_lens, q, out, scale_log2e, part, next_layer, next_q);
}

// The same for launches that end with workgroups alone on their CUs (plan_decode_loads says which, and
// what it measured): bound there by one wavefront per SIMD waiting for its pages, so the loads are counted.
template <int D, class Src, class E, int kAhead, int PS, bool kCut>
__global__ __launch_bounds__(kDecodeThreads, 2) void decode_lone_kernel(
    const uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t G,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const Src src,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ q, uint16_t* __restrict__ out,
    float scale_log2e, const DecodePartials part, int64_t next_layer, int64_t next_q)
{
    split_workgroup<D, Src, E, kAhead, PS, kCut, Loads::kLone>(layer_base, page_stride, num_pages, Hkv, G, block_tables, max_blocks, src, ctx_lens,
                                                       cu_q_lens, q, out, scale_log2e, part, next_layer, next_q);
}

// Merge of the partials of the cut sequences where the workgroups do not do it themselves: grid as
// above; the workgroup of a cut sequence's first item merges it.
template <int D, class Src, class E>
__global__ __launch_bounds__(kDecodeThreads) void decode_merge_kernel(
    int32_t Hkv, int32_t G, const Src src, const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    uint16_t* __restrict__ out, const DecodePartials part, int64_t next_q)
{
    const int32_t n_items = gridDim.x / Hkv, item = blockIdx.x / Hkv, g = blockIdx.x - item * Hkv, Hq = Hkv * G;
    DecodeItem it;
    if (!fetch_item(src, item, ctx_lens, cu_q_lens, it) || it.n_splits == 1 || item != it.first_item) return;
    merge_pieces<D, E>(part.of_layer(blockIdx.y, n_items, Hq, Hkv, D), it.first_item, it.n_splits, Hq, g, G,
                       out + blockIdx.y * next_q + (int64_t)it.token * Hq * D);
}

template <class E>
static int launch_decode_as(const cs_kv_pool& pool, int32_t layer, const LayerSpan& span, const cs_batch& b, const DecodePlan& plan,
                            const void* q, void* out, int32_t Hq, float scale, void* workspace, hipStream_t st,
                            bool merge_only)
{
    if (plan.num_decode == 0) return CS_OK;
    const int32_t Hkv = pool.num_kv_heads, D = pool.head_dim, G = Hq / Hkv;
    const uint16_t* layer_base = (const uint16_t*)pool.base + (int64_t)layer * pool.layer_stride;
    const float scale_log2e = scale * 1.4426950408889634f;
    const DecodeWorkspace w = decode_workspace(plan, Hq, Hkv, D, span.n);
    char* ws = (char*)workspace;
    const bool cut = plan.num_multi > 0, in_place = cut && plan.merges_in_place && !merge_only;
    const DecodePartials part = {(float*)(ws + w.part_o), (float*)(ws + w.part_ml), in_place ? (uint64_t*)ws : nullptr,
                                 in_place ? next_launch_number() : 0};
    const uint32_t n_items = plan.in_args || cut ? plan.total_items : b.num_seqs;
    dim3 grid(n_items * (uint32_t)Hkv, (uint32_t)span.n);
#define CS_LAUNCH_DECODE_P(KERNEL, DD, SRC, src, AH, PS, CUT)                                                \
    hipLaunchKernelGGL((KERNEL<DD, SRC, E, AH, PS, CUT>), grid, dim3(kDecodeThreads), 0, st, layer_base, \
                       pool.page_stride, pool.num_pages, Hkv, G, b.block_tables, b.max_blocks_per_seq, \
                       src, b.ctx_lens, b.cu_q_lens, (const uint16_t*)q, (uint16_t*)out,               \
                       scale_log2e, part, span.pool, span.q);
#define CS_LAUNCH_DECODE_A(KERNEL, DD, SRC, src, AH, CUT)                                                    \
    if (pool.page_size == 16) { CS_LAUNCH_DECODE_P(KERNEL, DD, SRC, src, AH, 16, CUT) } else { CS_LAUNCH_DECODE_P(KERNEL, DD, SRC, src, AH, 8, CUT) }
#define CS_LAUNCH_DECODE(KERNEL, DD, SRC, src, CUT)                                                         \
    if (plan.pages_ahead == 2) { CS_LAUNCH_DECODE_A(KERNEL, DD, SRC, src, 2, CUT) } else { CS_LAUNCH_DECODE_A(KERNEL, DD, SRC, src, 1, CUT) }
#define CS_LAUNCH_DECODE_ARGS(DD, CUT)                                                                      \
    if (plan.counted_loads) { CS_LAUNCH_DECODE(decode_lone_kernel, DD, ItemsInArgs, plan.arg_items, CUT) } else { CS_LAUNCH_DECODE(decode_split_kernel, DD, ItemsInArgs, plan.arg_items, CUT) }
#define CS_LAUNCH_MERGE(DD, SRC, src)                                                                       \
    hipLaunchKernelGGL((decode_merge_kernel<DD, SRC, E>), grid, dim3(kDecodeThreads), 0, st, Hkv, G, src, b.ctx_lens, \
                       b.cu_q_lens, (uint16_t*)out, part, span.q);
    if (plan.in_args) {
        // (merge_only: the fused mixed-batch kernel has already done the items' work)
        if (!merge_only) {
            if (cut) {
                if (D == 128) { CS_LAUNCH_DECODE_ARGS(128, true) } else { CS_LAUNCH_DECODE_ARGS(64, true) }
            } else {
                if (D == 128) { CS_LAUNCH_DECODE_ARGS(128, false) } else { CS_LAUNCH_DECODE_ARGS(64, false) }
            }
        }
        if (cut && !in_place) {
            if (D == 128) { CS_LAUNCH_MERGE(128, ItemsInArgs, plan.arg_items) } else { CS_LAUNCH_MERGE(64, ItemsInArgs, plan.arg_items) }
        }
    } else if (!cut) {
        const ItemsIdentity src = {0};
        if (D == 128) { CS_LAUNCH_DECODE(decode_split_kernel, 128, ItemsIdentity, src, false) } else { CS_LAUNCH_DECODE(decode_split_kernel, 64, ItemsIdentity, src, false) }
    } else {
        DecodeItem* items = (DecodeItem*)(ws + w.items);
        hipLaunchKernelGGL(decode_plan_kernel, dim3(1), dim3(kPlanThreads), 0, st, b.num_seqs, b.ctx_lens,
                           b.cu_q_lens, plan.split_tokens, plan.total_items, items);
        const ItemsInMemory src = {items};
        if (D == 128) { CS_LAUNCH_DECODE(decode_split_kernel, 128, ItemsInMemory, src, false) } else { CS_LAUNCH_DECODE(decode_split_kernel, 64, ItemsInMemory, src, false) }
        if (D == 128) { CS_LAUNCH_MERGE(128, ItemsInMemory, src) } else { CS_LAUNCH_MERGE(64, ItemsInMemory, src) }
    }
#undef CS_LAUNCH_DECODE
#undef CS_LAUNCH_DECODE_ARGS
#undef CS_LAUNCH_DECODE_A
#undef CS_LAUNCH_DECODE_P
#undef CS_LAUNCH_MERGE
    return check_launch("decode kernels");
}

int launch_decode_layers(const cs_kv_pool& pool, int32_t layer, const LayerSpan& span, const cs_batch& b, const DecodePlan& plan,
                         const void* q, void* out, int32_t Hq, float scale, void* workspace, hipStream_t st, bool f16,
                         bool merge_only)
{
    return f16 ? launch_decode_as<F16>(pool, layer, span, b, plan, q, out, Hq, scale, workspace, st, merge_only)
               : launch_decode_as<Bf16>(pool, layer, span, b, plan, q, out, Hq, scale, workspace, st, merge_only);
}

int launch_decode(const cs_kv_pool& pool, int32_t layer, const cs_batch& b, const DecodePlan& plan,
                  const void* q, void* out, int32_t Hq, float scale, void* workspace, hipStream_t st, bool f16,
                  bool merge_only)
{
    return launch_decode_layers(pool, layer, LayerSpan{1, 0, 0, 0}, b, plan, q, out, Hq, scale, workspace, st, f16, merge_only);
}

}  // namespace cs
