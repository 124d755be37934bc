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
@pytest.mark.parametrize("ctx", [47, 127, 160])
@pytest.mark.parametrize("cus", [256, 2])
def test_an_infinity_in_v_stays_one_through_the_merge(ctx, cus):
    """The last piece's weight is not zero anywhere, so its infinite feature is infinite in the output and
    the other features are what they are without it."""
    sh = synth.Shape(8, 2, 128)
    b = synth.make_batch(sh, [ctx], [1], synth.generator(98))
    st = Step(b, 98)
    want = st.oracle_attention()
    st.v_new[0, 1, 77] = float("inf")
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
    assert (out[0, 4:, 77] == float("inf")).all()
    out[0, 4:, 77] = torch.from_numpy(want[0, 4:, 77]).to(out)
    assert_attention_close(out, want, "finite features")
