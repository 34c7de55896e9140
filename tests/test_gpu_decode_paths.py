"""The decode step's routes by size: streaming and chunked products, preloaded
input rows, one and several sequences, the split-key partials combined in a
launch of their own or in the O-projection, and the boundary stored by a
kernel or copied."""
import numpy as np
import pytest

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
