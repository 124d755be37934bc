// Copy kernels: KV append into pages, checkpoint gather / restore of whole pages, and a
// plain copy used as the bandwidth ceiling.  All are HBM-bound streams of 16-byte lanes.
#include <algorithm>
#include "cs_common.h"

namespace cs {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------
// Whole-page copies (paper Sec. 5: gather scattered pages into one contiguous buffer;
// Sec. 4.4: bring them back on resume).  One (layer, page) is contiguous in the pool, so
// both directions are straight 16-byte-per-lane streams.  A workgroup is a single wavefront
// moving kChunkBytes (measured: many one-wavefront workgroups of 1 KiB sustain more HBM
// bandwidth on this part than fewer, fatter ones with several requests per lane in flight).
// ------------------------------------------------------------------------------------
constexpr int kCopyThreads = 64;
constexpr int kCopyUnroll = 1;                                   // 1 KiB per workgroup
constexpr int kChunkBytes = kCopyThreads * 16 * kCopyUnroll;

template <bool kToStaging>
__global__ __launch_bounds__(kCopyThreads) void page_copy_kernel(
    char* __restrict__ pool_base, int64_t layer_stride_b, int64_t page_stride_b,
    int32_t num_pages, int32_t layer_begin, const int32_t* __restrict__ ids,
    char* __restrict__ staging, int64_t stg_layer_stride_b, int64_t stg_page_stride_b,
    int32_t page_bytes, int32_t chunks_per_page)
{
    // grid.x = n * chunks_per_page (page-major), grid.y = layers
    const int32_t i = blockIdx.x / chunks_per_page;
    const int32_t c = blockIdx.x - i * chunks_per_page;
    const int32_t l = blockIdx.y;
    const int32_t id = ids[i];
    if (id < 0 || id >= num_pages) return;                       // never touch a bad page id
    char* p = pool_base + (int64_t)(layer_begin + l) * layer_stride_b + (int64_t)id * page_stride_b;
    char* s = staging + l * stg_layer_stride_b + i * stg_page_stride_b;
    const char* src = kToStaging ? p : s;
    char* dst = kToStaging ? s : p;
    const int32_t off0 = c * kChunkBytes + threadIdx.x * 16;
    u32x4 r[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const int32_t off = off0 + u * kCopyThreads * 16;
        if (off < page_bytes) r[u] = __builtin_nontemporal_load((const u32x4*)(src + off));
    }
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const int32_t off = off0 + u * kCopyThreads * 16;
        if (off < page_bytes) __builtin_nontemporal_store(r[u], (u32x4*)(dst + off));
    }
}

int launch_page_copy(const cs_kv_pool& pool, int32_t layer_begin, int32_t layer_end,
                     const int32_t* ids, int32_t n, void* staging, bool to_staging, hipStream_t st,
                     bool page_major)
{
    const int32_t layers = layer_end - layer_begin;
    if (n == 0 || layers == 0) return CS_OK;
    const int32_t page_bytes = (int32_t)pool_page_bytes(pool);
    const int32_t cpp = (page_bytes + kChunkBytes - 1) / kChunkBytes;
    dim3 grid((uint32_t)n * cpp, (uint32_t)layers);
    // staging[layer][page] (the default) or staging[page][layer] (one page's layers together)
    const int64_t stg_layer = page_major ? (int64_t)page_bytes : (int64_t)n * page_bytes;
    const int64_t stg_page = page_major ? (int64_t)layers * page_bytes : (int64_t)page_bytes;
    if (to_staging)
        hipLaunchKernelGGL(page_copy_kernel<true>, grid, dim3(kCopyThreads), 0, st,
                           (char*)pool.base, pool.layer_stride * 2, pool.page_stride * 2, pool.num_pages,
                           layer_begin, ids, (char*)staging, stg_layer, stg_page, page_bytes, cpp);
    else
        hipLaunchKernelGGL(page_copy_kernel<false>, grid, dim3(kCopyThreads), 0, st,
                           (char*)pool.base, pool.layer_stride * 2, pool.page_stride * 2, pool.num_pages,
                           layer_begin, ids, (char*)staging, stg_layer, stg_page, page_bytes, cpp);
    return check_launch("page_copy_kernel");
}

// ------------------------------------------------------------------------------------
// Token-granular checkpoint copies (paper Sec. 4.4: KV state is kept per token; after a
// generation step only the newly generated tokens are checkpointed).  The staging buffer
// holds plain rows, [layer][token][K|V][kv head][D].
//
// Bound by the cache lines the page format spreads a token over: per kv head 16 K units of 16
// bytes, each in a line of its own, and the 2 KiB of V units that hold its 128 features (head dim
// 128): 400 MB of lines for 50 MB of tokens, and on the way back as many partly written ones.  So
// every line is asked for once and everything is in flight together: one wavefront per (token, kv
// head or two of head dim 64, layer); a K lane moves one 16-byte unit, a V lane the 2-byte elements of features lane and
// lane + 64 (consecutive lanes, consecutive units: 8 lines an instruction, where a lane that moved
// 8 features touched 64 lines with each), and K and V are loaded before either is stored.  Only the staging
// side streams past the caches: the lines of the page hold up to 16 neighbouring tokens, which meet in
// the L2 (written past it, 2-byte elements cost a restore of neighbours 2-4 times as much; of tokens alone in
// their pages 1.5-2.3 times up to 300 MB of lines, which the last-level cache holds, and 0.8 from 500 MB on:
// streaming those alone was measured, by a look at 64 tokens of the list, and made shuffled neighbours 2.5 times
// as slow).  Eight elements a lane -> this, 1024 tokens x 48 layers x 8 kv heads, 1 / 4 / 15 neighbours a page: gather
// 344 / 219 / 209 -> 342 / 134 / 115 us, restore 797 / 327 / 271 -> 805 / 163 / 139 us.
// ------------------------------------------------------------------------------------
constexpr int kTokenCopyThreads = 64;

template <bool kToStaging, int D>
__global__ __launch_bounds__(kTokenCopyThreads) void token_copy_kernel(
    uint16_t* __restrict__ pool_base, int64_t layer_stride, int64_t page_stride,
    int32_t num_pages, int32_t layer_begin, const int32_t* __restrict__ token_slots, int32_t n, int32_t first, int32_t end,
    uint16_t* __restrict__ staging, int32_t Hkv, int32_t page_shift, int32_t streams)
{
    constexpr int kHeads = 128 / D;                              // kv heads of a wavefront: as much work at head dim 64 as at 128
    constexpr int kVPerLane = D / 64;
    // Workgroup x runs on XCD x % 8: with fewer than 8 of them a token the list is walked in `streams` parts at
    // once, so that the next token of the list, often a neighbour in the page, is on the same XCD's L2.
    const int32_t per_token = (Hkv + kHeads - 1) / kHeads, hs = per_token * streams, part = (end - first + streams - 1) / streams;
    const int32_t h0 = (int32_t)(blockIdx.x % per_token) * kHeads, l = blockIdx.y, lane = threadIdx.x;
    const int32_t i = first + (int32_t)(blockIdx.x % hs) / per_token * part + (int32_t)(blockIdx.x / hs);
    if (i >= end) return;
    const int32_t slot = token_slots[i];
    const int32_t page = slot >> page_shift, t = slot & ((1 << page_shift) - 1);
    if (slot < 0 || page >= num_pages) return;                   // never touch a bad slot
    const int32_t block_elems = D << page_shift;                 // one kv head's K (or V) block
    uint16_t* kblk = pool_base + (int64_t)(layer_begin + l) * layer_stride + (int64_t)page * page_stride + (int64_t)h0 * block_elems;
    uint16_t* vblk = kblk + (int64_t)Hkv * block_elems;
    uint16_t* krow = staging + (((int64_t)l * n + i) * 2 * Hkv + h0) * D;
    uint16_t* vrow = krow + Hkv * D;
    // feature d of token t: K unit (d/8) * page tokens + t; V element
    // (((d/16)*groups + t/8)*16 + d%16)*8 + t%8, groups = page tokens / 8: 64 features further on is
    // 4 * groups * 128 elements further on.  (The heads' rows of the staging side follow each other.)
    const int32_t unit = lane & (D / 8 - 1), kh = lane / (D / 8);
    const bool has_k = kh < kHeads && h0 + kh < Hkv;
    u32x4* kp = (u32x4*)(kblk + kh * block_elems + ((unit << page_shift) + t) * 8);
    uint16_t* vp = vblk + ((lane >> 4) << (page_shift + 4)) + ((t >> 3) << 7) + ((lane & 15) << 3) + (t & 7);
    u32x4* ks = (u32x4*)krow + lane;
    u32x4 k;
    uint16_t v[kHeads * kVPerLane];
    if (has_k) k = kToStaging ? *kp : __builtin_nontemporal_load(ks);
#pragma unroll
    for (int j = 0; j < kHeads * kVPerLane; ++j) {
        if (h0 + j / kVPerLane >= Hkv) break;
        uint16_t* p = vp + j / kVPerLane * block_elems + (j % kVPerLane << (page_shift + 6));
        v[j] = kToStaging ? *p : __builtin_nontemporal_load(vrow + lane + j * 64);
    }
    if (has_k) {
        if constexpr (kToStaging) __builtin_nontemporal_store(k, ks); else *kp = k;
    }
#pragma unroll
    for (int j = 0; j < kHeads * kVPerLane; ++j) {
        if (h0 + j / kVPerLane >= Hkv) break;
        uint16_t* p = vp + j / kVPerLane * block_elems + (j % kVPerLane << (page_shift + 6));
        if constexpr (kToStaging) __builtin_nontemporal_store(v[j], vrow + lane + j * 64); else *p = v[j];
    }
}

int launch_token_copy(const cs_kv_pool& pool, int32_t layer_begin, int32_t layer_end,
                      const int32_t* token_slots, int32_t n, void* staging, bool to_staging, hipStream_t st)
{
    const int32_t layers = layer_end - layer_begin;
    if (n == 0 || layers == 0) return CS_OK;
    const int32_t page_shift = pool.page_size == 16 ? 4 : 3;
    // (a launch holds fewer than 2^32 lanes along x: more tokens than that go in several)
    const int32_t per_token = pool.head_dim == 128 ? pool.num_kv_heads : (pool.num_kv_heads + 1) / 2;
    const int32_t streams = per_token < 8 && 8 % per_token == 0 ? 8 / per_token : 1;
    const int32_t max_tokens = 0x3ffffff / per_token / streams * streams;
#define CS_LAUNCH_TOKEN_COPY(DIR, DD)                                                                            \
    hipLaunchKernelGGL((token_copy_kernel<DIR, DD>), grid, dim3(kTokenCopyThreads), 0, st, (uint16_t*)pool.base,   \
                       pool.layer_stride, pool.page_stride, pool.num_pages, layer_begin, token_slots, n, first, first + m, \
                       (uint16_t*)staging, pool.num_kv_heads, page_shift, streams);
    for (int32_t first = 0, m; first < n; first += m) {
        m = n - first < max_tokens ? n - first : max_tokens;
        const dim3 grid((uint32_t)((m + streams - 1) / streams) * streams * per_token, (uint32_t)layers);
        if (pool.head_dim == 128) { if (to_staging) { CS_LAUNCH_TOKEN_COPY(true, 128) } else { CS_LAUNCH_TOKEN_COPY(false, 128) } }
        else                      { if (to_staging) { CS_LAUNCH_TOKEN_COPY(true, 64) } else { CS_LAUNCH_TOKEN_COPY(false, 64) } }
    }
#undef CS_LAUNCH_TOKEN_COPY
    return check_launch("token_copy_kernel");
}

// ------------------------------------------------------------------------------------
// Plain copy: the same inner loop without the page indirection.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(kCopyThreads) void plain_copy_kernel(
    char* __restrict__ dst, const char* __restrict__ src, int64_t bytes)
{
    const int64_t off0 = (int64_t)blockIdx.x * kChunkBytes + threadIdx.x * 16;
    u32x4 r[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const int64_t off = off0 + u * kCopyThreads * 16;
        if (off < bytes) r[u] = __builtin_nontemporal_load((const u32x4*)(src + off));
    }
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const int64_t off = off0 + u * kCopyThreads * 16;
        if (off < bytes) __builtin_nontemporal_store(r[u], (u32x4*)(dst + off));
    }
}

int launch_plain_copy(void* dst, const void* src, size_t bytes, hipStream_t st)
{
    if (bytes == 0) return CS_OK;
    const uint64_t blocks = (bytes + kChunkBytes - 1) / kChunkBytes;
    hipLaunchKernelGGL(plain_copy_kernel, dim3((uint32_t)blocks), dim3(kCopyThreads), 0, st,
                       (char*)dst, (const char*)src, (int64_t)bytes);
    return check_launch("plain_copy_kernel");
}

// ------------------------------------------------------------------------------------
// KV append (the cache is append-only: paper Sec. 1, 4.4).  A workgroup of 4 wavefronts
// owns one (page touched this step, kv head) and writes that page's K and V blocks in the
// order they lie in memory, so every store instruction of a wavefront covers 1 KiB of
// consecutive bytes; slots the step does not fill are simply masked out.  Sequences with a
// single new token go through append_token_kernel below instead.
// Workgroup slots are dealt to sequences as start(s) = cu_q_lens[s]/16 + 2s (a step of q
// tokens touches at most q/16 + 2 pages), found by owner_of.
// ------------------------------------------------------------------------------------
constexpr int kAppendThreads = 256;
constexpr int kAppendSlotShift = 4;

// The work of workgroup `block` of the chunk path.
template <int PS>
__device__ __forceinline__ void append_page_block(
    int32_t block,
    uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t D, int32_t S,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new)
{
    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Groups of 8 page
    // slots are numbered head-major, so the workgroups of one page -- which together read
    // whole token rows and write one whole page -- all land on the same XCD.
    const int32_t per = 8 * Hkv;
    const int32_t group = block / per, in_group = block - group * per;
    const int32_t h = in_group >> 3;
    const int32_t slot_id = group * 8 + (in_group & 7);
    // (arguments come in first: scalar loads return in any order, so a wait for one of them is a wait for the
    // page table's entry too)
    asm volatile("" :: "s"(k_new), "s"(v_new), "s"(layer_base), "s"(page_stride), "s"(num_pages), "s"(block_tables), "s"(max_blocks));
    const OwnedBy own = owner_of(cu_q_lens, ctx_lens, 0, S, slot_id, [](int32_t t, int32_t i) { return (t >> kAppendSlotShift) + 2 * i; });
    const int32_t s = own.seq, t_seq = own.token;
    const int32_t first = own.ctx;                                // the step fills positions [first, last)
    const int32_t last = first + own.q_len;
    if (last - first == 1) return;                               // single tokens: append_token_kernel
    // the workgroup's 16 positions: one page, or (pages of 8 tokens) two consecutive table entries
    const int32_t blk = (first >> 4) + (slot_id - ((t_seq >> kAppendSlotShift) + 2 * s));
    const int32_t p0 = blk << 4;                                  // first of the 16 positions
    if (p0 >= last) return;
    const int32_t block_elems = PS * D;
    const int32_t row = Hkv * D;                                  // elements between consecutive tokens
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave * 32 >= D) return;                                   // head_dim 64: two wavefronts suffice

    // Wavefront w moves features 32w .. 32w+31 of the page's 16 tokens.
    // K: lane (feature block dl = lane/16, token = lane%16) loads the 16 bytes of its token's
    //    row and stores them as unit dblk*16 + token.
    // V: a 16-byte unit is one feature of 8 consecutive tokens.  Lane (tile = lane/32, token
    //    half th = (lane/16)%2, feature f = lane%16) loads its feature from each of the half's
    //    8 token rows and stores the unit; the unit index is 64w + lane.
    // Either way consecutive lanes store consecutive units: 1 KiB per store instruction.
    const int32_t tok = lane & 15, dblk = wave * 4 + (lane >> 4);
    const int32_t th = (lane >> 4) & 1, feat = wave * 32 + (lane >> 5) * 16 + (lane & 15);
    // table entries of this lane's K token and of its V half (the same entry for pages of 16)
    const int32_t k_entry = PS == 16 ? blk : 2 * blk + (tok >> 3);
    const int32_t v_entry = PS == 16 ? blk : 2 * blk + th;
    const int32_t* table = block_tables + (int64_t)s * max_blocks;
    int32_t k_page = k_entry < max_blocks ? table[k_entry] : -1;
    int32_t v_page = v_entry < max_blocks ? table[v_entry] : -1;
    // packed token index of page position p0 (may lie before the step's first token)
    const int64_t tok_base = (int64_t)t_seq + (p0 - first);
    const int32_t pos = p0 + tok;
    const int32_t vpos = p0 + th * 8;                             // first position of the half
    const uint16_t* ksrc = k_new + (tok_base + tok) * row + (int64_t)h * D + dblk * 8;
    const uint16_t* vsrc = v_new + (tok_base + th * 8) * row + (int64_t)h * D + feat;
    // The rows come in beside the table's entries: one trip to memory less in a workgroup that is little but
    // trips (the empty asm below keeps the loads in front of the pages' checks).  Whole steps hardly show it (replayed
    // from a graph, append + attention of three chunks, 32/8 heads, 98.9 us with and without; eight decodes, by the same
    // in append_token_block, 16.4 -> 16.1).
    const bool k_row = pos >= first && pos < last, v_rows = vpos >= first && vpos + 8 <= last;
    u32x4 kv = {0u, 0u, 0u, 0u};
    uint16_t e[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (k_row) kv = __builtin_nontemporal_load((const u32x4*)ksrc);
    if (v_rows) {
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = __builtin_nontemporal_load(vsrc + j * row);
    }
    asm volatile("" : "+v"(k_page), "+v"(v_page), "+v"(kv));
    const bool k_page_ok = k_page >= 0 && k_page < num_pages, v_page_ok = v_page >= 0 && v_page < num_pages;
    const bool k_ok = k_page_ok && k_row, v_full = v_page_ok && v_rows;
    uint16_t* kblk = layer_base + (int64_t)(k_page_ok ? k_page : 0) * page_stride + (int64_t)h * block_elems;
    // V unit of this lane: 64*wave + lane in a page of 16 tokens (two halves per feature tile),
    // (2*wave + lane/32)*16 + lane%16 in the page of its half otherwise
    const int32_t v_unit = PS == 16 ? wave * 64 + lane : (wave * 2 + (lane >> 5)) * 16 + (lane & 15);
    uint16_t* dst = layer_base + (int64_t)(v_page_ok ? v_page : 0) * page_stride + (int64_t)(Hkv + h) * block_elems + v_unit * 8;
    if (k_ok) __builtin_nontemporal_store(kv, (u32x4*)(kblk + (dblk * PS + (tok & (PS - 1))) * 8));
    if (v_full) {
        const u32x4 unit = { (uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16),
                             (uint32_t)e[4] | ((uint32_t)e[5] << 16), (uint32_t)e[6] | ((uint32_t)e[7] << 16) };
        __builtin_nontemporal_store(unit, (u32x4*)dst);
    } else if (v_page_ok) {
        // a half the step fills only partly: element by element
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (vpos + j >= first && vpos + j < last) dst[j] = vsrc[j * row];
    }
}

// Single new tokens (decode): one lane per 16-byte unit (8 features) of the token's K row
// and V row.  The K unit is stored as it is; the V unit is scattered as 8 two-byte stores
// (the V block keeps 8 consecutive TOKENS of one feature together).  Sequences with more
// than one new token are left to append_page_kernel.
__device__ __forceinline__ void append_token_block(
    int32_t block,
    uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t D, int32_t S, int32_t T,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, int32_t page_size)
{
    const int32_t units_per_tok = Hkv * (D >> 3);
    const int64_t gid = (int64_t)block * kAppendThreads + threadIdx.x;
    const int32_t t = (int32_t)(gid / units_per_tok);
    if (t >= T) return;
    const int32_t u = (int32_t)(gid - (int64_t)t * units_per_tok);
    const int32_t h = u / (D >> 3);
    const int32_t dblk = u - h * (D >> 3);
    // sequence of token t.  In an online-first batch the decode sequences lead, so token t is
    // usually sequence t: try that, its length along, before bisecting the prefix sums.
    int32_t s = min(t, S - 1);
    int32_t first = cu_q_lens[s], end = cu_q_lens[s + 1], pos = ctx_lens[s];
    asm volatile("" : "+v"(first), "+v"(end), "+v"(pos));         // all three asked for here, not each where a branch needs it
    if (!(first <= t && t < end)) {
        int32_t lo = 0, hi = S;                                   // invariant: cu[lo] <= t < cu[hi]
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (cu_q_lens[mid] <= t) lo = mid; else hi = mid;
        }
        s = lo;
        first = cu_q_lens[s];
        end = cu_q_lens[s + 1];
        pos = ctx_lens[s];
    }
    if (end - first != 1) return;
    const int32_t blk = pos / page_size;
    if (pos < 0 || blk >= max_blocks) return;
    // the rows come in beside the table's entry: with the length above, two trips to memory instead of four
    const int64_t src = ((int64_t)t * Hkv + h) * D + dblk * 8;
    int32_t page = block_tables[(int64_t)s * max_blocks + blk];
    u32x4 kk = *(const u32x4*)(k_new + src);
    u32x4 vv = *(const u32x4*)(v_new + src);
    asm volatile("" : "+v"(page), "+v"(kk), "+v"(vv));
    if (page < 0 || page >= num_pages) return;
    const int32_t slot = pos - blk * page_size;
    const int32_t block_elems = page_size * D;
    uint16_t* kblk = layer_base + (int64_t)page * page_stride + (int64_t)h * block_elems;
    uint16_t* vblk = kblk + (int64_t)Hkv * block_elems;
    *(u32x4*)(kblk + (dblk * page_size + slot) * 8) = kk;
    // feature d = dblk*8 + e  ->  (((d/16)*groups + slot/8)*16 + d%16)*8 + slot%8, groups = page_size/8
    const int32_t vbase = (((dblk >> 1) * (page_size >> 3) + (slot >> 3)) * 16 + (dblk & 1) * 8) * 8 + (slot & 7);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t w = vv[e >> 1];
        vblk[vbase + e * 8] = (uint16_t)((e & 1) ? (w >> 16) : (w & 0xffffu));
    }
}

template <int PS>
__global__ __launch_bounds__(kAppendThreads) void append_page_kernel(
    uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t D, int32_t S,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, int64_t next_layer, int64_t next_kv)
{
    layer_base += blockIdx.y * next_layer; k_new += blockIdx.y * next_kv; v_new += blockIdx.y * next_kv;   // grid.y: layers
    append_page_block<PS>((int32_t)blockIdx.x, layer_base, page_stride, num_pages, Hkv, D, S, block_tables, max_blocks,
                          ctx_lens, cu_q_lens, k_new, v_new);
}

__global__ __launch_bounds__(kAppendThreads) void append_token_kernel(
    uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t D, int32_t S, int32_t T,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, int32_t page_size, int64_t next_layer, int64_t next_kv)
{
    layer_base += blockIdx.y * next_layer; k_new += blockIdx.y * next_kv; v_new += blockIdx.y * next_kv;
    append_token_block((int32_t)blockIdx.x, layer_base, page_stride, num_pages, Hkv, D, S, T, block_tables, max_blocks,
                       ctx_lens, cu_q_lens, k_new, v_new, page_size);
}

// A step with both chunks and single tokens (a mixed batch): the workgroups of the chunk path
// first, those of the single-token path behind them, in one launch (the calls are launch-bound
// at the batch sizes of a serving step, so the second launch was a third of the time).
template <int PS>
__global__ __launch_bounds__(kAppendThreads) void append_mixed_kernel(
    uint16_t* __restrict__ layer_base, int64_t page_stride, int32_t num_pages,
    int32_t Hkv, int32_t D, int32_t S, int32_t T,
    const int32_t* __restrict__ block_tables, int32_t max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ cu_q_lens,
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, uint32_t page_blocks, int64_t next_layer, int64_t next_kv)
{
    layer_base += blockIdx.y * next_layer; k_new += blockIdx.y * next_kv; v_new += blockIdx.y * next_kv;
    if (blockIdx.x < page_blocks)
        append_page_block<PS>((int32_t)blockIdx.x, layer_base, page_stride, num_pages, Hkv, D, S, block_tables, max_blocks,
                              ctx_lens, cu_q_lens, k_new, v_new);
    else
        append_token_block((int32_t)(blockIdx.x - page_blocks), layer_base, page_stride, num_pages, Hkv, D, S, T,
                           block_tables, max_blocks, ctx_lens, cu_q_lens, k_new, v_new, PS);
}

int launch_append(const cs_kv_pool& pool, int32_t layer, const cs_batch& b,
                  const void* k_new, const void* v_new, hipStream_t st)
{
    return launch_append_layers(pool, layer, LayerSpan{1, 0, 0, 0}, b, k_new, v_new, st);
}

int launch_append_layers(const cs_kv_pool& pool, int32_t layer, const LayerSpan& span, const cs_batch& b,
                         const void* k_new, const void* v_new, hipStream_t st)
{
    if (b.num_tokens == 0) return CS_OK;
    bool any_single = false, any_chunk = false;
    for (int32_t s = 0; s < b.num_seqs; ++s) {
        const int32_t ql = b.h_cu_q_lens[s + 1] - b.h_cu_q_lens[s];
        any_single |= ql == 1;
        any_chunk |= ql > 1;
    }
    uint16_t* layer_base = (uint16_t*)pool.base + (int64_t)layer * pool.layer_stride;
    const int64_t slots = (((int64_t)(b.num_tokens >> kAppendSlotShift) + 2ll * b.num_seqs) + 7) & ~7ll;   // whole groups of 8
    const int64_t page_blocks = any_chunk ? slots * pool.num_kv_heads : 0;
    const int64_t units = (int64_t)b.num_tokens * pool.num_kv_heads * (pool.head_dim / 8);
    const int64_t token_blocks = any_single ? (units + kAppendThreads - 1) / kAppendThreads : 0;
    if (page_blocks + token_blocks > 2147483647ll) return CS_ERR_UNSUPPORTED;
    const uint16_t* kn = (const uint16_t*)k_new;
    const uint16_t* vn = (const uint16_t*)v_new;
    if (any_chunk && any_single) {
        const dim3 grid((uint32_t)(page_blocks + token_blocks), (uint32_t)span.n);
        if (pool.page_size == 16)
            hipLaunchKernelGGL(append_mixed_kernel<16>, grid, dim3(kAppendThreads), 0, st,
                               layer_base, pool.page_stride, pool.num_pages, pool.num_kv_heads, pool.head_dim,
                               b.num_seqs, b.num_tokens, b.block_tables, b.max_blocks_per_seq, b.ctx_lens, b.cu_q_lens,
                               kn, vn, (uint32_t)page_blocks, span.pool, span.kv);
        else
            hipLaunchKernelGGL(append_mixed_kernel<8>, grid, dim3(kAppendThreads), 0, st,
                               layer_base, pool.page_stride, pool.num_pages, pool.num_kv_heads, pool.head_dim,
                               b.num_seqs, b.num_tokens, b.block_tables, b.max_blocks_per_seq, b.ctx_lens, b.cu_q_lens,
                               kn, vn, (uint32_t)page_blocks, span.pool, span.kv);
    } else if (any_chunk) {
        if (pool.page_size == 16)
            hipLaunchKernelGGL(append_page_kernel<16>, dim3((uint32_t)page_blocks, (uint32_t)span.n), dim3(kAppendThreads), 0, st,
                               layer_base, pool.page_stride, pool.num_pages, pool.num_kv_heads, pool.head_dim,
                               b.num_seqs, b.block_tables, b.max_blocks_per_seq, b.ctx_lens, b.cu_q_lens, kn, vn,
                               span.pool, span.kv);
        else
            hipLaunchKernelGGL(append_page_kernel<8>, dim3((uint32_t)page_blocks, (uint32_t)span.n), dim3(kAppendThreads), 0, st,
                               layer_base, pool.page_stride, pool.num_pages, pool.num_kv_heads, pool.head_dim,
                               b.num_seqs, b.block_tables, b.max_blocks_per_seq, b.ctx_lens, b.cu_q_lens, kn, vn,
                               span.pool, span.kv);
    } else if (any_single) {
        hipLaunchKernelGGL(append_token_kernel, dim3((uint32_t)token_blocks, (uint32_t)span.n), dim3(kAppendThreads), 0, st,
                           layer_base, pool.page_stride, pool.num_pages, pool.num_kv_heads, pool.head_dim,
                           b.num_seqs, b.num_tokens, b.block_tables, b.max_blocks_per_seq, b.ctx_lens,
                           b.cu_q_lens, kn, vn, pool.page_size, span.pool, span.kv);
    }
    return check_launch("append kernels");
}

}  // namespace cs
