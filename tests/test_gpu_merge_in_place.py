"""Cut decode sequences are merged either by whichever of their workgroups finishes last or, where the
workgroups run in rounds, by a kernel of its own; both run the same merge over the same partials, so
they agree bit for bit.  What the workspace held before (here: garbage, and an earlier call's
leavings) must not matter."""
import pytest
import torch

from paper_2410_01228_amd import binding as cs
from paper_2410_01228_amd import synth
from helpers import Step, assert_attention_close, from_bits

pytestmark = pytest.mark.gpu


# pieces per sequence: 1 and 2, one batch of announcements (64) and one more, more kv heads than words in a line
@pytest.mark.parametrize("Hq,Hkv,D,ctx,split", [(4, 2, 64, [15, 31, 1100], 16), (8, 2, 128, [1023, 16, 1040], 16),
                                                (24, 12, 128, [300, 700], 64), (32, 8, 128, [2000, 900, 5], 256)])
@pytest.mark.parametrize("chunk", [0, 40])
def test_merge_in_place_and_by_kernel_agree(Hq, Hkv, D, ctx, split, chunk):
    sh = synth.Shape(Hq, Hkv, D)
    q_lens = [1] * len(ctx) + ([chunk] if chunk else [])
    b = synth.make_batch(sh, ctx + ([50] if chunk else []), q_lens, synth.generator(97))
    st = Step(b, 97)
    pool = cs.Pool(from_bits(st.prior_pool(), "cuda"), 1, b.num_pages, Hkv, D)
    bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
    cs.cs_kv_append(pool, 0, bb, st.k_new.cuda(), st.v_new.cuda())
    q = st.q.cuda()
    outs = []
    cs.cs_set_decode_split_tokens(split)
    try:
        # plenty of CUs: everything resident at once; two: rounds; a decode workgroup per CU beside the tiles
        for cus, mode in ((256, 2), (2, 2), (64, 3)):
            cs.cs_debug_set_cu_count(cus)
            cs.cs_set_mixed_fusion(mode)
            ws = cs.workspace_for(bb, Hq, Hkv, D)
            ws.random_(0, 256, generator=torch.Generator(device="cuda").manual_seed(cus))
            for _ in range(2):
                out = torch.full((b.T, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
                cs.cs_paged_attention_mixed(pool, 0, bb, q, out, Hq, sh.scale, ws)
                outs.append(out)
            torch.cuda.synchronize()
    finally:
        cs.cs_set_decode_split_tokens(0)
        cs.cs_set_mixed_fusion(1)
        cs.cs_debug_set_cu_count(0)
    assert_attention_close(outs[0], st.oracle_attention(), "merged in place")
    n = len(ctx)
    for out in outs[1:]:
        assert torch.equal(out[:n].view(torch.int16), outs[0][:n].view(torch.int16))
    assert_attention_close(outs[-1], st.oracle_attention(), "merged in place beside tiles")


# pieces: fewer than, exactly and more than the eight that a merge holds in flight
# (head dim 64: in the grid also beyond eight)
@pytest.mark.parametrize("ctx,D", [(47, 128), (127, 128), (160, 128), (160, 64)])
@pytest.mark.parametrize("cus", [256, 2])
def test_an_infinity_in_v_stays_one_through_the_merge(ctx, D, cus):
    """The last piece's weight is not zero anywhere, so its infinite feature is infinite in the output and
    the other features are what they are without it."""
    sh = synth.Shape(8, 2, D)
    b = synth.make_batch(sh, [ctx], [1], synth.generator(98))
    st = Step(b, 98)
    want = st.oracle_attention()
    st.v_new[0, 1, 47] = float("inf")
    pool = cs.Pool(from_bits(st.prior_pool(), "cuda"), 1, b.num_pages, sh.Hkv, sh.D)
    bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
    cs.cs_kv_append(pool, 0, bb, st.k_new.cuda(), st.v_new.cuda())
    out = torch.full((1, sh.Hq, sh.D), float("nan"), dtype=torch.bfloat16, device="cuda")
    cs.cs_set_decode_split_tokens(16)
    try:
        cs.cs_debug_set_cu_count(cus)                   # merged in place, and by a kernel
        cs.cs_paged_attention_mixed(pool, 0, bb, st.q.cuda(), out, sh.Hq, sh.scale, cs.workspace_for(bb, sh.Hq, sh.Hkv, sh.D))
        torch.cuda.synchronize()
    finally:
        cs.cs_set_decode_split_tokens(0)
        cs.cs_debug_set_cu_count(0)
    assert (out[0, 4:, 47] == float("inf")).all()
    out[0, 4:, 47] = torch.from_numpy(want[0, 4:, 47]).to(out)
    assert_attention_close(out, want, "finite features")


@pytest.mark.parametrize("cus", [256, 2])               # merged in place, and by a kernel
def test_every_piece_is_weighted_against_the_maximum_of_all(cus):
    """The merge's own arithmetic, redone in torch from the partials that the call leaves in its
    workspace: weights 2^(m - M) with the maximum M of ALL pieces, the sums as fused multiply-adds in
    the order of the pieces (also beyond the eight that are loaded together), one division.  The
    fused multiply-add is taken in 64 bits and rounded to 32, which the rounding to fp16 (the finer of the two types) does not see."""
    sh, split = synth.Shape(32, 8, 128), 16
    ctx = [16 * 9 - 1 + 5 * s for s in range(40)]       # 9 to 21 pieces
    b = synth.make_batch(sh, ctx, [1] * len(ctx), synth.generator(99))
    st = Step(b, 99, q_gain=3.0, dtype=torch.float16)
    pool = cs.Pool(from_bits(st.prior_pool(), "cuda", torch.float16), 1, b.num_pages, sh.Hkv, sh.D)
    bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
    cs.cs_kv_append(pool, 0, bb, st.k_new.cuda(), st.v_new.cuda())
    out = torch.full((b.T, sh.Hq, sh.D), float("nan"), dtype=torch.float16, device="cuda")
    cs.cs_set_decode_split_tokens(split)
    try:
        cs.cs_debug_set_cu_count(cus)
        items, n, _ = cs.cs_debug_decode_items(bb, sh.Hkv, sh.D)
        ws = torch.empty(cs.cs_paged_attention_workspace_bytes(bb, sh.Hq, sh.Hkv, sh.D), dtype=torch.uint8, device="cuda")
        cs.cs_paged_attention_mixed_f16(pool, 0, bb, st.q.cuda(), out, sh.Hq, sh.scale, ws)
        torch.cuda.synchronize()
    finally:
        cs.cs_set_decode_split_tokens(0)
        cs.cs_debug_set_cu_count(0)
    f = ws.view(torch.float32)                          # ... | (max, sum) of every item | outputs of every item
    o = f[-n * sh.Hq * sh.D:].view(n, sh.Hq, sh.D)
    ml = f[-n * sh.Hq * (sh.D + 2):-n * sh.Hq * sh.D].view(n, sh.Hq, 2)
    at = 0
    while at < n:
        s, _, k = items[at]
        assert k > 8
        M = ml[at:at + k, :, 0].amax(0)
        L, O = torch.zeros_like(M), torch.zeros_like(o[0])
        for i in range(at, at + k):
            w = torch.exp2(ml[i, :, 0] - M)
            L = (ml[i, :, 1].double() * w.double() + L.double()).float()
            O = (o[i].double() * w.double()[:, None] + O.double()).float()
        assert torch.equal(out[s].view(torch.int16), (O / L[:, None]).half().view(torch.int16))
        at += k


# ranges: 2, 4, 16; a chunk that leaves most rows of its tiles without a token
@pytest.mark.parametrize("chunk,prefix,ranges", [(40, 2000, 2), (200, 3000, 4), (5, 30000, 16)])
def test_tiles_merged_in_the_grid_and_by_kernel_agree(chunk, prefix, ranges):
    """The same chunk alone (a kernel merges its tiles), beside one short decode (a kernel too, from three
    ranges on) and beside a decode stream that outlasts it (the grid does): the same bits."""
    sh, outs = synth.Shape(32, 8, 128), []
    g = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (synth.randn_bf16((chunk, h, sh.D), g, "cuda") for h in (sh.Hq, sh.Hkv, sh.Hkv))
    prior = [synth.randn_bf16((prefix, sh.Hkv, sh.D), g, "cuda") for _ in range(2)]
    for decodes, keys in ((0, 0), (1, 50), (64, 3000)):
        ctx = [prefix] + [keys] * decodes
        b = synth.make_batch(sh, ctx, [chunk] + [1] * decodes, synth.generator(8 + decodes))
        pool = cs.Pool.empty(1, b.num_pages, sh.Hkv, sh.D)
        pool.tensor.normal_(generator=g)
        bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
        assert cs.cs_debug_mixed_tail_cut(bb, sh.Hq, sh.Hkv, sh.D)[1:] == (0, ranges)
        first = cs.Batch(b.block_tables[:1], torch.zeros(1, dtype=torch.int32), torch.tensor([0, prefix], dtype=torch.int32))
        cs.cs_kv_append(pool, 0, first, *prior)
        pad = [torch.cat([x, torch.zeros((decodes, *x.shape[1:]), dtype=x.dtype, device="cuda")]) for x in (q, k, v)]
        cs.cs_kv_append(pool, 0, bb, pad[1], pad[2])
        ws = cs.workspace_for(bb, sh.Hq, sh.Hkv, sh.D)
        ws.random_(0, 256, generator=g)
        for _ in range(2):
            out = torch.full_like(pad[0], float("nan"))
            cs.cs_paged_attention_mixed(pool, 0, bb, pad[0], out, sh.Hq, sh.scale, ws)
            torch.cuda.synchronize()
            outs.append(out[:chunk])
    assert torch.isfinite(outs[0].float()).all()
    for out in outs[1:]:
        assert torch.equal(out.view(torch.int16), outs[0].view(torch.int16))


def test_a_tile_range_far_below_the_others_still_counts():
    """A chunk whose tiles are cut in two ranges: the keys of the first score about 130 octaves below those
    of the second, and only the first range's first key has a value, 2^127, in one feature.  What is
    left of it after the softmax, 2^127 * 2^-130.6 / (keys of the second range), is an ordinary number."""
    sh, C, P, low = synth.Shape(32, 8, 128), 2000, 40, 1024
    b = synth.make_batch(sh, [C], [P], synth.generator(5))
    st = Step(b, 5)
    bb = cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens)
    _, first, ranges = cs.cs_debug_mixed_tail_cut(bb, sh.Hq, sh.Hkv, sh.D)
    assert first == 0 and ranges == 2 and (C + P + 63) // 64 * 32 == low   # (so the first range ends at key 1024)
    pool = cs.Pool(torch.zeros_like(from_bits(st.prior_pool(), "cuda")), 1, b.num_pages, sh.Hkv, sh.D)
    prior = cs.Batch(b.block_tables, torch.zeros(1, dtype=torch.int32), torch.tensor([0, C], dtype=torch.int32))
    k = torch.zeros((C + P, sh.Hkv, sh.D), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros_like(k)
    k[low:, :, 0] = 32.0
    v[0, :, 5] = 2.0 ** 127
    cs.cs_kv_append(pool, 0, prior, k[:C].contiguous(), v[:C].contiguous())
    cs.cs_kv_append(pool, 0, bb, k[C:].contiguous(), v[C:].contiguous())
    q = torch.zeros((P, sh.Hq, sh.D), dtype=torch.bfloat16, device="cuda")
    q[:, :, 0] = 32.0
    out = torch.full_like(q, float("nan"))
    cs.cs_paged_attention_mixed(pool, 0, bb, q, out, sh.Hq, sh.scale, cs.workspace_for(bb, sh.Hq, sh.Hkv, sh.D))
    torch.cuda.synchronize()
    high = torch.arange(C + 1 - low, C + P + 1 - low, dtype=torch.float64)            # keys of the second range that row t sees
    want = 2.0 ** 127 * torch.exp(torch.tensor(-32.0 * 32.0 * sh.scale, dtype=torch.float64)) / high
    got = out[:, :, 5].double().cpu()
    # the weight is a denormal of 19 bits, the exponent -130.6 has 2^-17 of an octave; the output is bf16
    assert (got / want[:, None] - 1).abs().max() <= 2.0 ** -8
    assert (out[:, :, :5] == 0).all() and (out[:, :, 6:] == 0).all()
