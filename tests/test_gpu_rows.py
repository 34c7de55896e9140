"""A row's result does not depend on which other rows share the call: a
sequence is bit for bit the same alone, in a batch, and at the head of a longer
causal call, whatever the tokens after it hold; in a prefix, in the encoder and
in a decode step."""
import numpy as np
import pytest

import synth
from paper_2608_14586_amd import binding as vb
from prefix_cases import EncCase, LlmCase
from synth.configs import llama_like

pytestmark = pytest.mark.gpu


def _bits(t):
    import torch
    return t.contiguous().view(torch.int16 if t.element_size() == 2 else torch.int32).numpy().copy()


def _prefix(ctx, s, dt, tok, k, frame):
    """(boundary as fp32, KV as bit patterns) of one call over tok[B][L][d]."""
    B, L = tok.shape[:2]
    bnd = vb.Boundary(B, L, s.d_model, k, s.n_kv_heads, s.head_dim, stack_dtype=dt, out_dtype="f32")
    ctx.vla_run_prefix(frame, np.ascontiguousarray(tok), B, L, k, bnd)
    ctx.vla_wait_boundary(frame, 60000)
    return bnd.hidden.numpy().copy(), _bits(bnd.kv)


# long K with few rows and with many: 7B down (K = 11008), 0.5B down (K =
# 4864); gate/up in two launches at 1000 rows, QKV (rotary embedding, K, V and
# V^T behind columns that another launch wrote) at 1601 split and at 2113
@pytest.mark.parametrize("name,L,B,longer", [("llm7b", 16, 3, 203), ("llm7b", 203, 2, 1000), ("llm7b", 512, 1, 1601),
                                             ("llm7b", 1000, 1, 2113), ("small_llm", 65, 4, 700),
                                             ("small_llm", 333, 2, 2000)])
@pytest.mark.parametrize("split", [False, True])
def test_prefix_rows_alone_and_together(name, L, B, longer, split):
    c = LlmCase(name, longer, 1, B=B, perturbed=True)
    if split:
        c.ctx.vla_set_precision(vb.VLA_STACK_LLM, vb.VLA_PREC_SPLIT)
    tok = c.tokens(frame=3)
    hid, kv = _prefix(c.ctx, c.s, "bf16", tok[:, :L], 1, 1)
    assert np.isfinite(hid).all()
    for b in range(B):
        h1, kv1 = _prefix(c.ctx, c.s, "bf16", tok[b:b + 1, :L], 1, 2 + b)
        assert np.array_equal(h1[0], hid[b]) and np.array_equal(kv1[:, :, 0], kv[:, :, b]), b
    # whole blocks of 32 queries: the attention rescales by the block's rows
    n = L // 32 * 32
    h1, kv1 = _prefix(c.ctx, c.s, "bf16", tok[:1], 1, 9)
    assert np.array_equal(kv1[:, :, 0, :, :L], kv[:, :, 0])
    assert np.array_equal(h1[0, :n], hid[0, :n])
    c.close()


@pytest.mark.parametrize("L,n_img", [(100, 3), (257, 6)])
def test_encoder_images_alone_and_together(L, n_img):
    c = EncCase("vit_l", n_img, L, n_blocks=2, perturbed=True)
    p = c.patches(frame=2)
    whole = c.run(p)
    c.n_img = 1
    for i in range(n_img):
        assert np.array_equal(_bits(c.run(np.ascontiguousarray(p[i:i + 1]))[0]), _bits(whole[i])), i
    c.close()


def _stack(s, dt, L, B, name):
    wl = synth.Workload(name, dt, s, None, batch=B, seq=L)
    ctx = vb.Context(llm=vb.stack_cfg(s, dt, max_tokens=L, max_batch=B))
    for l in range(s.n_blocks):
        ctx.vla_load_block_weights(vb.VLA_STACK_LLM, l, synth.llm_block_weights(wl, l, perturbed=True))
    return ctx, synth.tokens(wl, frame=1)


# gate/up of 8200 columns: under and over 256 tiles of 64x64
def test_fp32_rows_alone_and_together():
    s = llama_like(1, 512, 8, 2, 64, 4100)
    ctx, tok = _stack(s, "f32", 64, 4, "rows_f32")
    hid, kv = _prefix(ctx, s, "f32", tok, 1, 1)
    assert np.isfinite(hid).all()
    for b in range(4):
        h1, kv1 = _prefix(ctx, s, "f32", tok[b:b + 1], 1, 2 + b)
        assert np.array_equal(h1[0], hid[b]) and np.array_equal(kv1[:, :, 0], kv[:, :, b]), b
    ctx.vla_destroy()


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("j", [1, 16, 63, 64, 100, 129])
def test_fp32_tokens_before_one_that_is_not_finite(j, bad):
    """Causality also for what a later token poisons: the rows before it keep
    their bits, whatever key tile and query block they share with it."""
    s = llama_like(2, 256, 4, 2, 64, 688)
    ctx, tok = _stack(s, "f32", 130, 1, "rows_nan")
    hid, kv = _prefix(ctx, s, "f32", tok, 2, 1)
    tok[0, j, 5] = bad
    h1, kv1 = _prefix(ctx, s, "f32", tok, 2, 2)
    assert np.array_equal(h1[0, :j], hid[0, :j]) and np.array_equal(kv1[:, :, 0, :, :j], kv[:, :, 0, :, :j])
    assert not np.isfinite(h1[0, j:]).any()
    ctx.vla_destroy()


# the O-projection combines the split-key partials for one sequence and a
# launch of its own does for four: one split, a few, past 16; many tokens, as
# a last bit of the combined value shows only where its bf16 rounds the other way
TOKENS = 24
@pytest.mark.parametrize("pos", [100, 1500, 2048, 2600, 4100])
def test_decode_rows_alone_and_together(pos):
    import torch
    s = llama_like(1, 896, 14, 2, 64, 512)
    B, L_cap = 4, pos + 5
    ctx, _ = _stack(s, "bf16", L_cap, B, "rows_decode")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(pos)
    cache = torch.empty((1, 2, B, 2, L_cap, 64), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=gen)
    x = synth.normal_bf16(synth.seed_of("rows_decode_x", pos), (TOKENS, B, 896))

    def step(t, frame, rows):
        n = len(rows)
        c = cache[:, :, rows].contiguous()
        torch.cuda.synchronize()  # written on torch's stream, read on the context's
        ob = vb.Boundary(n, 1, 896, 0, 2, 64, out_dtype="f32", with_kv=False)
        ctx.vla_decode_step(frame, np.ascontiguousarray(x[t, rows]), n, pos, 1, c, L_cap, ob)
        ctx.vla_wait_boundary(frame, 60000)
        return ob.hidden.numpy().reshape(n, -1).copy()

    for t in range(TOKENS):
        whole = step(t, 8 * t, list(range(B)))
        assert np.isfinite(whole).all()
        for b in range(B):
            assert np.array_equal(step(t, 8 * t + 1 + b, [b])[0], whole[b]), (t, b)
    ctx.vla_destroy()
