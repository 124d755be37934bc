"""cs_run_layers puts several layers into one launch where their tensors allow it; whatever it does, each
layer's pool and output must be what the single calls give."""
import ctypes

import pytest
import torch

from paper_2410_01228_amd import binding as cs
from paper_2410_01228_amd import synth

pytestmark = pytest.mark.gpu


def setup(sh, ctx, ql, L, seed):
    b = synth.make_batch(sh, ctx, ql, synth.generator(seed))
    g = torch.Generator(device="cuda").manual_seed(seed)
    pool = cs.Pool.empty(L, b.num_pages, sh.Hkv, sh.D)
    pool.tensor.normal_(generator=g)
    q, k, v = (synth.randn_bf16((L, b.T, h, sh.D), g, "cuda") for h in (sh.Hq, sh.Hkv, sh.Hkv))
    return b, cs.Batch(b.block_tables, b.ctx_lens, b.cu_q_lens), pool, q, k, v


def layer_by_layer(sh, bb, pool, q, k, v):
    out = torch.full_like(q, float("nan"))
    ws = cs.workspace_for(bb, sh.Hq, sh.Hkv, sh.D)
    for l in range(q.shape[0]):
        cs.cs_kv_append(pool, l, bb, k[l], v[l])
        cs.cs_paged_attention_mixed(pool, l, bb, q[l], out[l], sh.Hq, sh.scale, ws)
    torch.cuda.synchronize()
    return out


def close(got, want):
    """Both are within half the path's bar (2e-2 absolute, 1e-2 relative in the Frobenius norm) of the exact
    result, so they are within all of it of each other: another cut of a sequence rounds its
    weights to 16 bits against another running maximum."""
    got, want = got.float(), want.float()
    assert torch.isfinite(got).all()
    assert (got - want).abs().max() <= 2e-2 and (got - want).norm() <= 1e-2 * want.norm()


# decode only (cut and whole), chunks only (cut; more tiles than a round), both kinds; layers that
# leave a remainder of 1, 2, 3; safepoints at other distances than the launches'
@pytest.mark.parametrize("sh,ctx,ql", [
    (synth.Shape(8, 2, 128), [5000, 17, 300], [1, 1, 1]),
    (synth.Shape(4, 2, 64), [40] * 70, [1] * 70),
    (synth.Shape(28, 4, 128), [6000, 100], [40, 33]),
    (synth.Shape(32, 8, 128), [700, 0], [300, 900]),
    (synth.Shape(32, 8, 128), [900, 2500, 31, 400], [1, 1, 1, 200]),
    (synth.Shape(8, 2, 64), [90, 0, 1200], [1, 50, 1])])
@pytest.mark.parametrize("L,every", [(4, 4), (7, 3), (2, None)])
def test_layers_in_one_launch_match_single_calls(sh, ctx, ql, L, every):
    b, bb, pool, q, k, v = setup(sh, ctx, ql, L, 300 + L)
    twin = cs.Pool(pool.tensor.clone(), L, b.num_pages, sh.Hkv, sh.D)
    want = layer_by_layer(sh, bb, twin, q, k, v)
    flag = ctypes.c_int32(0)
    sp = cs.cs_safepoint(ctypes.addressof(flag), cs.POLL_FN(0), None, every, 1, 0) if every else None
    need = cs.cs_run_layers_workspace_bytes(bb, 1, sh.Hq, sh.Hkv, sh.D)
    for extra in (0, 4 * need):                        # the least workspace a caller may bring, and plenty
        ws = torch.empty(max(16, need + extra), dtype=torch.uint8, device="cuda")
        out = torch.full_like(q, float("nan"))
        assert cs.cs_run_layers(pool, 0, L, bb, q, k, v, out, sh.Hq, sh.scale, ws, sp) == -1
        torch.cuda.synchronize()
        close(out, want)
        assert torch.equal(pool.tensor.view(torch.int16), twin.tensor.view(torch.int16))


# the same shapes and a many-piece batch: every grouping that safepoints, a remainder and the workspace lead
# to, against the single calls, bit for bit
@pytest.mark.parametrize("sh,ctx,ql", [
    (synth.Shape(8, 2, 128), [5000, 17, 300], [1, 1, 1]),
    (synth.Shape(28, 4, 128), [6000, 100], [40, 33]),
    (synth.Shape(32, 8, 128), [700, 0], [300, 900]),
    (synth.Shape(32, 8, 128), [900, 2500, 31, 400], [1, 1, 1, 200]),
    (synth.Shape(16, 4, 128), [2500, 0, 0, 0], [512, 512, 512, 512]),      # whole alone, but several layers' grid would like cuts
    (synth.Shape(64, 8, 128), [8651, 3000, 12160], [1, 1, 22]),
    (synth.Shape(8, 2, 64), [90, 0, 1200], [1, 50, 1])])
def test_how_layers_are_grouped_changes_no_bit(sh, ctx, ql):
    L = 7
    b, bb, pool, q, k, v = setup(sh, ctx, ql, L, 320)
    want = layer_by_layer(sh, bb, cs.Pool(pool.tensor.clone(), L, b.num_pages, sh.Hkv, sh.D), q, k, v)
    need = cs.cs_run_layers_workspace_bytes(bb, 1, sh.Hq, sh.Hkv, sh.D)
    flag = ctypes.c_int32(0)
    for size in (need, 2 * need, 3 * need, 4 * need):
        ws = torch.empty(max(16, size), dtype=torch.uint8, device="cuda")
        for every in (None, 1, 3, 4):
            sp = cs.cs_safepoint(ctypes.addressof(flag), cs.POLL_FN(0), None, every, 1, 0) if every else None
            out = torch.full_like(q, float("nan"))
            cs.cs_run_layers(pool, 0, L, bb, q, k, v, out, sh.Hq, sh.scale, ws, sp)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16)), (size, every)


def test_layers_that_share_or_chain_their_tensors_run_one_after_the_other():
    sh, L = synth.Shape(8, 2, 128), 4
    b, bb, pool, q, k, v = setup(sh, [500, 60, 33], [1, 20, 1], L, 311)
    ws = cs.run_layers_workspace_for(bb, 0, sh.Hq, sh.Hkv, sh.D)
    want = layer_by_layer(sh, bb, pool, q, k, v)
    # one output buffer for all layers: the last layer's result stays
    shared = q[:1].expand(L, *q.shape[1:])
    out = torch.full_like(q[:1], float("nan"))
    cs.cs_run_layers(pool, 0, L, bb, shared, k, v, out, sh.Hq, sh.scale, ws)
    # layer l + 1's queries are layer l's output
    chain = torch.empty((L + 1, *q.shape[1:]), dtype=torch.bfloat16, device="cuda")
    chain[0] = q[0]
    cs.cs_run_layers(pool, 0, L, bb, chain[:L], k, v, chain[1:], sh.Hq, sh.scale, ws)
    torch.cuda.synchronize()
    assert torch.equal(chain[1].view(torch.int16), want[0].view(torch.int16))
    ref = layer_by_layer(sh, bb, pool, shared.contiguous(), k, v)
    assert torch.equal(out[0].view(torch.int16), ref[L - 1].view(torch.int16))
    x = q[0]
    for l in range(L):
        y = torch.empty_like(x)
        cs.cs_paged_attention_mixed(pool, l, bb, x, y, sh.Hq, sh.scale, cs.workspace_for(bb, sh.Hq, sh.Hkv, sh.D))
        x = y
    torch.cuda.synchronize()
    assert torch.equal(chain[L].view(torch.int16), x.view(torch.int16))
