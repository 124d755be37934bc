"""The calls neither synchronise nor allocate, so a caller may record them into a HIP graph
(the per-layer loop of a small batch is launch-bound; the paper's engine launches its model
as graphs, Sec. 5).  A captured multi-layer step is replayed several times, with eager work
and synchronisations between the replays, and every replay must reproduce the eager result
bit for bit."""
import numpy as np
import pytest
import torch

from paper_2410_01228_amd import binding as cs
from paper_2410_01228_amd import synth
from helpers import Step, bits, from_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("maker,shrink", [(synth.config_tiny, None), (synth.config_qwen7b_mixed, 16),
                                          (synth.config_llama70b_long, 32)])
def test_captured_layers_replay_bit_identical(maker, shrink):
    b = maker() if shrink is None else maker(shrink=shrink)
    sh = b.shape
    L = 3
    steps = [Step(b, 70 + l, layer=l) for l in range(L)]
    cpu_pool = steps[0].prior_pool(L=L)
    for l in range(1, L):
        steps[l].layer = l
        cpu_pool[l] = steps[l].prior_pool(L=L)[l]
    bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
    ws = cs.workspace_for(bb, sh.Hq, sh.Hkv, sh.D)
    q = [st.q.cuda() for st in steps]
    kn = [st.k_new.cuda() for st in steps]
    vn = [st.v_new.cuda() for st in steps]

    def fresh_pool():
        return cs.Pool(from_bits(cpu_pool, "cuda"), L, cpu_pool.shape[1], sh.Hkv, sh.D)

    def run(pool, outs):
        for l in range(L):
            cs.cs_kv_append(pool, l, bb, kn[l], vn[l])
            cs.cs_paged_attention_mixed(pool, l, bb, q[l], outs[l], sh.Hq, sh.scale, ws)

    # eager reference
    pool_e = fresh_pool()
    outs_e = [torch.zeros((b.T, sh.Hq, sh.D), dtype=torch.bfloat16, device="cuda") for _ in range(L)]
    run(pool_e, outs_e)
    torch.cuda.synchronize()
    want = [bits(o) for o in outs_e]
    want_pool = bits(pool_e.tensor)

    # captured
    pool_g = fresh_pool()
    outs_g = [torch.zeros_like(o) for o in outs_e]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(pool_g, outs_g)                                   # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(pool_g, outs_g)
    for replay in range(3):
        for o in outs_g:
            o.fill_(float("nan"))                             # eager work between replays
        junk = torch.randn(1 << 16, device="cuda").sum().item()   # and a synchronisation
        assert np.isfinite(junk)
        graph.replay()
        torch.cuda.synchronize()
        for l in range(L):
            np.testing.assert_array_equal(bits(outs_g[l]), want[l], err_msg="replay %d layer %d" % (replay, l))
        np.testing.assert_array_equal(bits(pool_g.tensor), want_pool)


# cut sequences alone, by a kernel (ten pieces of one) and in the grid (eight); cut sequences and tiles of two ranges in one grid, all workgroups resident; tiles that a
# decode stream outlasts.  (What merges in the grid announces partials by words that the next replay must
# find cleared: a replay launches with the same number.)
@pytest.mark.parametrize("ctx,ql,ranges", [([900, 2500, 1700, 40], [1] * 4, 1), ([900, 2000, 1700, 40], [1] * 4, 1),
                                           ([900, 2500, 1700, 40, 2000], [1] * 4 + [40], 2),
                                           ([3000] * 48 + [3000], [1] * 48 + [100], 4)])
@pytest.mark.parametrize("one_call", [False, True])
def test_merges_in_the_grid_replay_bit_identical(ctx, ql, ranges, one_call):
    sh, L = synth.Shape(32, 8, 128), 3
    b = synth.make_batch(sh, ctx, ql, synth.generator(71))
    bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
    _, first, planned = cs.cs_debug_mixed_tail_cut(bb, sh.Hq, sh.Hkv, sh.D)
    assert (first, planned) == (0, ranges)
    if len(ctx) < 10:
        items, n, _ = cs.cs_debug_decode_items(bb, sh.Hkv, sh.D)
        assert any(k > 1 for _, _, k in items) and n * sh.Hkv <= 256
    g = torch.Generator(device="cuda").manual_seed(72)
    pool = cs.Pool.empty(L, b.num_pages, sh.Hkv, sh.D)
    pool.tensor.normal_(generator=g)
    q, k, v = (synth.randn_bf16((L, b.T, h, sh.D), g, "cuda") for h in (sh.Hq, sh.Hkv, sh.Hkv))
    out = torch.empty_like(q)
    ws = torch.empty(max(16, 3 * cs.cs_run_layers_workspace_bytes(bb, 0, sh.Hq, sh.Hkv, sh.D)), dtype=torch.uint8, device="cuda")

    def run():
        if one_call:
            cs.cs_run_layers(pool, 0, L, bb, q, k, v, out, sh.Hq, sh.scale, ws)
            return
        for l in range(L):
            cs.cs_kv_append(pool, l, bb, k[l], v[l])
            cs.cs_paged_attention_mixed(pool, l, bb, q[l], out[l], sh.Hq, sh.scale, ws)

    run()
    torch.cuda.synchronize()
    want = out.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for replay in range(4):
        out.fill_(float("nan"))
        if replay == 2:
            ws.random_(0, 256, generator=g)                       # somebody else used the workspace
        assert np.isfinite(torch.randn(1 << 16, device="cuda").sum().item())
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), replay
