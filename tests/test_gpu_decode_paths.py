"""The decode step's routes by size: streaming and chunked products, preloaded
input rows, one and several sequences, the split-key partials combined in a
launch of their own or in the O-projection, and the boundary stored by a
kernel or copied, on the copy stream."""
import numpy as np
import pytest

import synth
from paper_2608_14586_amd import binding as vb
from prefix_cases import rel_l2
from synth.configs import llama_like
from test_gpu_decode import _oracle_rows, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,B,L,prec", [
    # K below, at and above half a chunk, one chunk, one slab past it
    (llama_like(1, 448, 7, 1, 64, 448), 1, 5, 0), (llama_like(1, 512, 4, 4, 128, 512), 1, 5, 0),
    (llama_like(1, 896, 14, 2, 64, 4864), 1, 700, 0), (llama_like(1, 1024, 8, 8, 128, 1088), 1, 63, 1),
    # one row past the preloaded widths: d = 4160, d_ff = 12352
    (llama_like(1, 4160, 2, 1, 64, 12352), 1, 40, 0), (llama_like(1, 4160, 2, 1, 64, 256), 2, 3, 1),
    # partials combined in the O-projection: one split, the split's edges, one
    # split past a batch of eight, several sequences
    (llama_like(1, 256, 4, 2, 64, 256), 1, 126, 0), (llama_like(1, 256, 4, 2, 64, 256), 1, 127, 0),
    (llama_like(1, 256, 2, 1, 128, 256), 1, 1030, 0), (llama_like(1, 896, 14, 2, 64, 512), 4, 520, 1),
    # and in a launch of their own: 32 heads over several splits
    (llama_like(1, 512, 32, 4, 128, 256), 2, 600, 0),
])
def test_decode_routes_match_oracle(shape, B, L, prec):
    name = "route_%d_%d_%d_%d" % (shape.d_model, shape.d_ff, B, L)
    wl, W, toks, outs, _, ctx = _run(shape, B, L, 1, 2, name, prec=prec)
    x, ref = _oracle_rows(wl, W, toks, L, 2, 1)
    for t in range(2):
        for b in range(B):
            # the blocks' update of the residual, at the prefix's 1e-2 bar
            assert rel_l2(outs[t][b] - x[b, t], ref[b, t] - x[b, t]) < 1e-2, (t, b)
    ctx.vla_destroy()


def test_decode_boundary_at_any_alignment():
    """A boundary buffer off 16 bytes takes the copy instead of the kernel's
    store; both hold the same bytes, bf16 and fp32, and finish their frame."""
    import torch
    shape = llama_like(1, 512, 4, 2, 128, 512)
    B, L = 3, 20
    _, _, toks, _, cache, ctx = _run(shape, B, L, 1, 1, "route_align")
    x = np.ascontiguousarray(toks[:, L])
    frame = 50
    for dt, tdt in (("bf16", torch.bfloat16), ("f32", torch.float32)):
        got = []
        for off in (0, 4):
            ob = vb.Boundary(B, 1, 512, 0, 2, 128, out_dtype=dt, with_kv=False)
            buf = torch.zeros(B * 512 + 16, dtype=tdt, pin_memory=True)
            at = off // buf.element_size()
            ob.c.hidden = buf.data_ptr() + off
            frame += 1
            ctx.vla_decode_step(frame, x, B, L, 1, cache, cache.shape[4], ob)
            ctx.vla_wait_boundary(frame, 60000)
            g, t, total = ctx.vla_frame_times(frame)
            assert g > 0 and t >= 0 and total >= g
            got.append(buf[at:at + B * 512].clone())
            assert not buf[at + B * 512:].any()
        assert got[0].any() and torch.equal(got[0], got[1])
    ctx.vla_destroy()


# widths the chunked products took before the streaming ones staged their rows
# early, and widths above one chunk: each has its own form of the remainder
@pytest.mark.parametrize("d,B", [(512, 1), (896, 3), (1024, 1), (4096, 1), (4096, 3)])
def test_split_operands_to_the_last_bit(d, B):
    """hi = bf16(v), lo = bf16(v - hi) of the normalised row, bit for bit.  With
    w_o = 0, one gate feature for all and unit up and down rows the boundary is
    x + G (hi + lo), every step of it exact or one fp32 rounding."""
    import torch
    F = d
    s = llama_like(1, d, 1, 1, 64, F)
    wl = synth.Workload("split_bits_%d" % d, "bf16", s, None)
    W = synth.llm_block_weights(wl, 0, perturbed=True)
    one, gate = np.uint16(0x3F80), np.uint16(0x4280)  # 1, 64
    W["w_o"] = np.zeros_like(W["w_o"])
    W["w_gate"], W["w_up"], W["w_down"] = (np.zeros_like(W[n]) for n in ("w_gate", "w_up", "w_down"))
    W["w_gate"][:, 0] = gate
    W["w_up"][np.arange(F), np.arange(F)] = one
    W["w_down"][np.arange(d), np.arange(F)] = one
    ctx = vb.Context(llm=vb.stack_cfg(s, "bf16", max_tokens=64, max_batch=B))
    ctx.vla_load_block_weights(vb.VLA_STACK_LLM, 0, W)
    ctx.vla_set_precision(vb.VLA_STACK_LLM, vb.VLA_PREC_SPLIT)
    rng = np.random.default_rng(d + B)
    x = rng.integers(1, 16, (B, d)) * rng.choice([-1, 1], (B, d))  # sums of their squares are exact
    x[:, 0] = 15
    cache = torch.zeros((1, 2, B, 1, 8, 64), dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    ob = vb.Boundary(B, 1, d, 0, 1, 64, out_dtype="f32", with_kv=False)
    x16 = torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16)
    ctx.vla_decode_step(1, x16.view(torch.int16).numpy().view(np.uint16), B, 0, 1, cache, 8, ob)
    ctx.vla_wait_boundary(1, 60000)

    def bf(a):
        return torch.from_numpy(np.asarray(a, np.float32)).to(torch.bfloat16).to(torch.float32).numpy()

    f = np.float32
    ms = (x * x).sum(1).astype(f) / f(d) + f(s.norm_eps)
    hs = x.astype(f) * (f(1) / np.sqrt(ms))[:, None]
    g = synth.as_f32(W["norm2_g"])
    y = hs * g
    hi = bf(y)
    exact = (hs.astype(np.float64) * g - hi).astype(f)
    u = hi + bf(exact if d < 1024 else y - hi)
    a = (u[:, :1] * f(64)) * u
    ahi = bf(a)
    want = x.astype(f) + (ahi + bf(a - ahi))
    got = ob.hidden.numpy().reshape(B, d)
    assert np.array_equal(got, want), (np.argwhere(got != want)[:5], (got != want).sum())
    ctx.vla_destroy()


def test_waiting_for_a_prefix_leaves_the_core():
    """The wait for a prefix frame sleeps; only a decode step's is polled."""
    import time

    import torch
    from prefix_cases import LlmCase
    c = LlmCase("llm7b", 2048, 1, perturbed=True)
    tok = c.tokens()
    dev = torch.from_numpy(tok.view(np.int16)).cuda()
    bnd = c.boundary()
    cpu = wall = 0.0
    for f in range(24):
        c.ctx.vla_run_prefix(f, dev, 1, 2048, 1, bnd)
        t, w = time.thread_time(), time.perf_counter()
        c.ctx.vla_wait_boundary(f, 60000)
        if f >= 4:
            cpu, wall = cpu + time.thread_time() - t, wall + time.perf_counter() - w
    # about 0.9 ms a frame in sleeps of 70-80 us, each followed by one query
    assert cpu < 0.5 * wall, (cpu, wall)
    c.close()


def _step(ctx, frame, x, B, pos, cache, hidden, dt="f32"):
    """One decode step whose boundary goes to the pinned address `hidden`."""
    ob = vb.Boundary(B, 1, x.shape[-1], 0, 2, 128, out_dtype=dt, with_kv=False)
    ob.c.hidden = hidden
    ctx.vla_decode_step(frame, np.ascontiguousarray(x), B, pos, 1, cache, cache.shape[4], ob)


def test_decode_boundary_follows_the_copy_stream():
    """A read of the boundary buffer that the caller has queued on the copy
    stream comes before the next step's handoff into that buffer."""
    import torch
    shape = llama_like(1, 512, 4, 2, 128, 512)
    B, L = 2, 20
    _, _, toks, _, cache, ctx = _run(shape, B, L, 1, 2, "route_order")
    copy = ctx.copy_stream
    hidden = torch.zeros(B * 512, dtype=torch.float32, pin_memory=True)
    big = torch.zeros(1 << 28, dtype=torch.int32, device="cuda")
    got = torch.empty(B * 512, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    _step(ctx, 60, toks[:, L], B, L, cache, hidden.data_ptr())
    ctx.vla_wait_boundary(60, 60000)
    first = hidden.clone()
    with torch.cuda.stream(copy):
        for _ in range(20):  # milliseconds of earlier work on the copy stream
            big.add_(1)
        got.copy_(hidden, non_blocking=True)
    _step(ctx, 61, toks[:, L + 1], B, L + 1, cache, hidden.data_ptr())
    ctx.vla_wait_boundary(61, 60000)
    torch.cuda.synchronize()
    assert not torch.equal(hidden, first)
    assert torch.equal(got.cpu(), first)
    ctx.vla_destroy()


def test_decode_boundary_into_any_pinned_memory():
    """Into the middle of an allocation and into non-coherent host memory: the
    same bytes, and none around them."""
    import ctypes

    import torch
    shape = llama_like(1, 512, 4, 2, 128, 512)
    B, L, nb = 1, 20, 512 * 4
    _, _, toks, _, cache, ctx = _run(shape, B, L, 1, 1, "route_pinned")
    hip = ctypes.CDLL("libamdhip64.so")
    got = []
    for i, flags in enumerate((0x0, 0x40000000, 0x80000000)):  # default, coherent, non-coherent
        p = ctypes.c_void_p()
        assert hip.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(3 * nb), ctypes.c_uint(flags)) == 0
        ctypes.memset(p, 0, 3 * nb)
        _step(ctx, 70 + i, toks[:, L], B, L, cache, p.value + nb)
        ctx.vla_wait_boundary(70 + i, 60000)
        whole = np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_float)), (3 * 512,)).copy()
        assert not whole[:512].any() and not whole[1024:].any()
        got.append(whole[512:1024])
        assert hip.hipHostFree(p) == 0
    assert got[0].any() and all(np.array_equal(g, got[0]) for g in got)
    ctx.vla_destroy()
