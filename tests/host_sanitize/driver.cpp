// Host-side exercise of libconserve_kv under AddressSanitizer / UndefinedBehaviorSanitizer.
// The page map, the launch-plan queries and the argument checks return before a kernel launch; the
// iterations over layers go through to stand-ins of the launchers, which hold what each launch
// would use against the workspace of the call.  Device pointers are fakes that are never
// dereferenced on the host.
// Prints "ok <count>" and exits 0; any sanitizer report makes the process exit non-zero.
#include <cstdint>
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <random>
#include <stdexcept>
#include <string>
#include <vector>
#include "conserve_kv.h"
#include "cs_plan.h"
#include "launch_window.h"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); std::exit(3); } } while (0)

static cs_batch make_batch(const std::vector<int32_t>& ctx, const std::vector<int32_t>& cu, int32_t max_blocks) {
    cs_batch b = {};
    b.num_seqs = (int32_t)ctx.size();
    b.num_tokens = cu.back();
    b.block_tables = (const int32_t*)0x20000;      // device pointers: fakes
    b.max_blocks_per_seq = max_blocks;
    b.ctx_lens = (const int32_t*)0x30000;
    b.cu_q_lens = (const int32_t*)0x40000;
    b.h_ctx_lens = ctx.data();
    b.h_cu_q_lens = cu.data();
    return b;
}

// A machine without a source of randomness: nothing behind the C interface may throw for it.
void std::random_device::_M_init(const std::string&) { throw std::runtime_error("no random device"); }

// One iteration over `layers` layers, not preempted, through the stand-ins.
static int iterate(const cs_batch& b, const int* sh, int32_t layers, const void* workspace, size_t bytes, int32_t check_every) {
    cs_kv_pool pool = {(void*)0x100000, layers, 1 << 22, 16, sh[1], sh[2], 0, 0};
    pool.page_stride = 2ll * sh[1] * pool.page_size * sh[2];
    pool.layer_stride = pool.page_stride * pool.num_pages;
    const int32_t flag = 0;
    const cs_safepoint sp = {&flag, nullptr, nullptr, check_every, b.num_seqs / 2, 0};
    const int64_t q_elems = (int64_t)b.num_tokens * sh[0] * sh[2], kv_elems = (int64_t)b.num_tokens * sh[1] * sh[2];
    g_window = LaunchWindow{true, workspace, bytes, 0, 0, 0};
    int32_t first = 7;
    const int rc = cs_run_layers(&pool, 0, layers, &b, (void*)(1ll << 44), (void*)(2ll << 44), (void*)(3ll << 44), (void*)(4ll << 44),
                                 q_elems, kv_elems, sh[0], 0.1f, (void*)workspace, bytes, check_every > 0 ? &sp : nullptr, &first, nullptr);
    g_window.open = false;
    CHECK(rc != CS_OK || first == -1);
    return rc;
}

int main() {
    std::mt19937 rng(12345);
    long checks = 0;
    for (int i = 0; i < 100; ++i) CHECK(cs::next_launch_number() != cs::next_launch_number());
    // ---- launch plans over random batches, three chip sizes, all shapes ----
    const int shapes[][3] = {{32, 8, 128}, {28, 4, 128}, {64, 8, 128}, {40, 8, 128}, {4, 2, 64}, {16, 1, 64}};
    std::vector<uint32_t> items(1024);
    std::vector<int32_t> order(512);
    for (int round = 0; round < 300; ++round) {
        const int* sh = shapes[rng() % 6];
        const int S = round == 0 ? 65535 : round == 1 ? 881 : round == 2 ? 880 : 1 + (int)(rng() % 300);
        std::vector<int32_t> ctx(S), cu(S + 1, 0);
        int32_t max_need = 1;
        for (int s = 0; s < S; ++s) {
            const int kind = rng() % 10;
            const int32_t q = S > 1000 ? 1 : kind < 6 ? 1 : kind < 7 ? 0 : 2 + (int32_t)(rng() % 3000);
            ctx[s] = S > 1000 ? (int32_t)(rng() % 64) : (int32_t)(rng() % (kind == 9 ? 200000 : 9000));
            cu[s + 1] = cu[s] + q;
            max_need = std::max(max_need, (ctx[s] + q + 7) / 8);
        }
        cs_batch b = make_batch(ctx, cu, max_need);
        cs_debug_set_cu_count(round % 3 == 0 ? 0 : round % 3 == 1 ? 128 : 512);
        // where a mixed batch's decode work runs, and forced cuts of the last tiles, change the plan
        cs_set_mixed_fusion((int32_t)(rng() % 4));
        if (round % 4 == 1) cs_debug_set_tail_cut((int32_t)(rng() % 50), 2 + (int32_t)(rng() % 2));
        else cs_debug_set_tail_cut(-1, 0);
        const size_t need = cs_paged_attention_workspace_bytes(&b, sh[0], sh[1], sh[2]);
        CHECK(cs_paged_attention_workspace_bytes(&b, sh[0], sh[1], sh[2]) == need);      // remembered, same answer
        int32_t split = 0;
        const int32_t n = cs_debug_decode_items(&b, sh[1], sh[2], items.data(), (int32_t)items.size(), &split);
        CHECK(n >= 0 || n <= -1000000);
        CHECK(split >= 256 && split % 16 == 0);
        const int32_t ahead = cs_debug_decode_pages_ahead(&b, sh[1], sh[2]);
        CHECK(ahead == 1 || ahead == 2);
        int32_t counted = -1;
        CHECK(cs_debug_decode_loads(&b, sh[1], sh[2], 1, &counted) == ahead && (counted == 0 || counted == 1));
        const int32_t n_ord = cs_debug_prefill_order(&b, sh[0], sh[1], sh[2], order.data(), (int32_t)order.size());
        CHECK(n_ord >= 0 && n_ord <= 512);
        int32_t first_cut = -1, ranges = -1;
        const int32_t n_slots = cs_debug_mixed_tail_cut(&b, sh[0], sh[1], sh[2], &first_cut, &ranges);
        CHECK(n_slots == CS_ERR_INVALID_ARG || (n_slots >= 0 && first_cut >= 0 && first_cut <= n_slots && ranges >= 1));
        if (n_slots > 0 && ranges > 1)
            CHECK(need >= (size_t)(n_slots - first_cut) * sh[1] * ranges * (8 * 16 * (sh[2] + 4) * sizeof(float)));
        const int32_t arrangement = cs_debug_mixed_arrangement(&b, sh[0], sh[1], sh[2]);
        CHECK(arrangement == CS_ERR_INVALID_ARG || (arrangement >= 0 && arrangement <= 2));
        const int32_t n_on = (int32_t)(rng() % (S + 1));
        CHECK(cs_run_layers_workspace_bytes(&b, n_on, sh[0], sh[1], sh[2]) >= need);
        // the attention call itself with a workspace one byte short: refused on the host
        cs_kv_pool pool = {(void*)0x100000, 2, 1 << 22, (int32_t)(rng() % 2 ? 16 : 8), sh[1], sh[2], 0, 0};
        pool.page_stride = 2ll * sh[1] * pool.page_size * sh[2];
        pool.layer_stride = pool.page_stride * pool.num_pages;
        if (need > 0 && b.num_tokens > 0 && (int64_t)max_need * 8 >= 0) {
            const int rc = cs_paged_attention_mixed(&pool, 0, &b, (void*)0x50000, (void*)0x60000, sh[0], 0.1f, (void*)0x70000,
                                                    need - 1, nullptr);
            CHECK(rc == CS_ERR_WORKSPACE_TOO_SMALL || rc == CS_ERR_INVALID_ARG);
        }
        // an iteration of several layers, with the least workspace the call accepts and with more
        if (S <= 300 && b.num_tokens > 0) {
            const int32_t layers = 1 + (int32_t)(rng() % 9), every = (int32_t)(rng() % 5);
            const size_t least = std::max(need, cs_run_layers_workspace_bytes(&b, S / 2, sh[0], sh[1], sh[2]));
            bool decodes = false, chunks = false;
            for (int s = 0; s < S; ++s) { decodes |= cu[s + 1] - cu[s] == 1; chunks |= cu[s + 1] - cu[s] > 1; }
            for (const size_t bytes : {least, 2 * least, 4 * least + 64}) {
                CHECK(iterate(b, sh, layers, (void*)0x70000, bytes, every) == CS_OK);
                CHECK(g_window.layers_appended == layers && g_window.layers_decoded == (decodes ? layers : 0) &&
                      g_window.layers_prefilled == (chunks ? layers : 0));
            }
            // layers that share a launch are cut as each would be alone
            const cs::Plans one = cs::plans_for(&b, sh[0], sh[1], sh[2]);
            for (int32_t n = 2; n <= 4; ++n) {
                const cs::Plans& many = cs::plans_for(&b, sh[0], sh[1], sh[2], n);
                CHECK(many.need <= cs::workspace_for_layers(&b, sh[0], sh[1], sh[2], n));
                CHECK((cs::workspace_for_layers(&b, sh[0], sh[1], sh[2], n) == 0) == (one.need == 0));
                // (what the header advises to bring)
                CHECK(cs::workspace_for_layers(&b, sh[0], sh[1], sh[2], n) <= n * one.need + one.need / 8 + 256);
                CHECK(many.d.split_tokens == one.d.split_tokens && many.d.total_items == one.d.total_items && many.d.num_multi == one.d.num_multi);
                CHECK(std::equal(one.d.arg_items.e, one.d.arg_items.e + (one.d.in_args ? one.d.total_items : 0), many.d.arg_items.e));
                CHECK(many.p.range_steps == one.p.range_steps && many.p.max_ranges == one.p.max_ranges);
                CHECK(many.p.cut_first_pos == one.p.cut_first_pos && (one.p.cut_first_pos == 0 || many.p.backwards == one.p.backwards));
            }
            // a pointer that the call has no reason to look at must not be used, whatever size comes with it
            if (least == 0) {
                CHECK(iterate(b, sh, layers, nullptr, (size_t)1 << 30, every) == CS_OK);
                CHECK(iterate(b, sh, layers, (void*)0x70001, (size_t)1 << 30, every) == CS_OK);
            }
        }
        checks += 8;
    }
    // cut tiles: a kernel merges them where one workgroup's work on them would show, the grid where two
    // ranges make it short or decode work still runs
    {
        struct Case { int32_t decodes, keys, chunk, prefix; bool in_place; };
        const Case cases[] = {{1, 40, 3, 26000, false}, {4, 500, 8, 17000, false}, {8, 900, 5, 3000, false},
                              {24, 1600, 200, 1000, true}, {64, 4000, 24, 17000, true}, {128, 8000, 3, 26000, true}};
        const int sh[3] = {32, 8, 128};
        cs_debug_set_cu_count(256);
        cs_set_mixed_fusion(1);
        cs_debug_set_tail_cut(-1, 0);
        for (const Case& c : cases) {
            std::vector<int32_t> ctx(c.decodes, c.keys), cu(1, 0);
            for (int32_t s = 0; s < c.decodes; ++s) cu.push_back(s + 1);
            ctx.push_back(c.prefix);
            cu.push_back(c.decodes + c.chunk);
            cs_batch b = make_batch(ctx, cu, 1 << 14);
            const cs::Plans& p = cs::plans_for(&b, sh[0], sh[1], sh[2]);
            CHECK(p.p.max_ranges > 1 && p.f.arrangement != 0 && p.p.merges_in_place == c.in_place);
            // cut decode sequences: never where decode workgroups walk several pairs beside the tiles
            for (int32_t mode = 2; mode <= 3; ++mode) {
                cs_set_mixed_fusion(mode);
                cs_set_decode_split_tokens(256);
                const cs::Plans& forced = cs::plans_for(&b, sh[0], sh[1], sh[2]);
                CHECK(forced.f.arrangement == (forced.d.in_args ? mode - 1 : 0) && (mode == 2 || !forced.d.merges_in_place));
                cs_set_mixed_fusion(1);
                cs_set_decode_split_tokens(0);
            }
            ++checks;
        }
        cs_debug_set_cu_count(0);
    }
    // batches that need no workspace layer by layer, but whose larger grids would gain from cuts
    {
        struct Case { int sh[3]; std::vector<int32_t> ctx, q; };
        const Case cases[] = {{{16, 4, 128}, {2500, 0, 0, 0}, {512, 512, 512, 512}},
                              {{64, 8, 128}, {41, 2395}, {392, 5}},
                              {{40, 8, 128}, {2603, 5, 190}, {5, 107, 637}}};
        cs_debug_set_cu_count(0);
        cs_set_mixed_fusion(1);
        cs_debug_set_tail_cut(-1, 0);
        for (const Case& c : cases) {
            std::vector<int32_t> cu(1, 0);
            for (int32_t q : c.q) cu.push_back(cu.back() + q);
            cs_batch b = make_batch(c.ctx, cu, 1000);
            CHECK(cs_run_layers_workspace_bytes(&b, 0, c.sh[0], c.sh[1], c.sh[2]) == 0);
            for (int32_t layers = 1; layers <= 8; ++layers) {
                CHECK(iterate(b, c.sh, layers, nullptr, (size_t)1 << 30, 0) == CS_OK);
                CHECK(iterate(b, c.sh, layers, (void*)0x70008, (size_t)1 << 30, 0) == CS_OK);
                checks += 2;
            }
        }
    }
    cs_debug_set_cu_count(0);
    cs_set_mixed_fusion(1);
    cs_debug_set_tail_cut(-1, 0);
    // ---- the slot model of the fused grid: any work list ends, no earlier than its longest piece alone ----
    for (int round = 0; round < 200; ++round) {
        const int32_t n = 1 + (int32_t)(rng() % 700), cus = 1 + (int32_t)(rng() % 300);
        std::vector<float> work(n);
        float longest = 0.f;
        for (auto& w : work) { w = (float)(rng() % 100000) * 0.01f; longest = std::max(longest, w); }
        const double until = rng() % 2 ? 0.0 : (double)(rng() % 2000);
        const double end = cs_debug_play_tiles(work.data(), n, cus, until);
        CHECK(end >= 0.78 * longest - 1e-3);
        CHECK(cs_debug_play_tiles(work.data(), n, 0, until) == -1.0);
        ++checks;
    }
    // ---- the page map against a plain model ----
    const int32_t G = 500, H = 300;
    cs_page_map* m = cs_page_map_create(G, H);
    CHECK(m != nullptr);
    std::vector<int32_t> host_of(G, -1), gpu_of(H, -2);
    for (int round = 0; round < 4000; ++round) {
        const int op = rng() % 4;
        const int32_t n = 1 + (int32_t)(rng() % 12);
        std::vector<int32_t> a(n), out(n);
        if (op == 0) {                                   // checkpoint
            for (auto& x : a) x = (int32_t)(rng() % G);
            int32_t first = -7;
            const int32_t k = cs_page_map_checkpoint(m, a.data(), n, out.data(), &first);
            if (k > 0) {
                for (int32_t i = 0; i < k; ++i) {
                    CHECK(host_of[out[i]] == -1 && gpu_of[first + i] == -2);
                    host_of[out[i]] = first + i;
                    gpu_of[first + i] = out[i];
                }
            } else {
                CHECK(k == 0 || k == CS_ERR_NO_HOST_PAGES);
            }
        } else if (op == 1) {                            // evict
            for (auto& x : a) x = (int32_t)(rng() % G);
            CHECK(cs_page_map_evict(m, a.data(), n, out.data()) == CS_OK);
            for (int32_t i = 0; i < n; ++i) {
                if (host_of[a[i]] >= 0) { CHECK(out[i] == host_of[a[i]]); gpu_of[host_of[a[i]]] = -1; host_of[a[i]] = -1; }
            }
        } else if (op == 2) {                            // drop whatever is allocated among n random host pages
            std::vector<int32_t> d;
            for (int32_t i = 0; i < n; ++i) { const int32_t h = (int32_t)(rng() % H); bool dup = false; for (int32_t y : d) dup |= y == h; if (gpu_of[h] != -2 && !dup) d.push_back(h); }
            if (!d.empty()) {
                CHECK(cs_page_map_drop(m, d.data(), (int32_t)d.size()) == CS_OK);
                for (int32_t h : d) { if (gpu_of[h] >= 0) host_of[gpu_of[h]] = -1; gpu_of[h] = -2; }
            }
        } else {                                         // bad arguments leave the map alone
            a[0] = G + 5;
            int32_t first = 0;
            CHECK(cs_page_map_checkpoint(m, a.data(), n, out.data(), &first) == CS_ERR_INVALID_ARG);
            CHECK(cs_page_map_host_of(m, -1) == -1 && cs_page_map_gpu_of(m, H) == -2);
        }
        if (round % 97 == 0) {
            int32_t free_model = 0;
            for (int32_t h = 0; h < H; ++h) { CHECK(cs_page_map_gpu_of(m, h) == gpu_of[h]); free_model += gpu_of[h] == -2; }
            for (int32_t g = 0; g < G; ++g) CHECK(cs_page_map_host_of(m, g) == host_of[g]);
            CHECK(cs_page_map_free_host_pages(m) == free_model);
        }
        ++checks;
    }
    cs_page_map_destroy(m);
    cs_page_map_destroy(nullptr);
    std::printf("ok %ld\n", checks);
    return 0;
}
