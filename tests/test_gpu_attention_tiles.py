"""The attention's key-tile pipeline: scores formed one tile ahead, two stages
of K and V^T, the running maximum raised in later tiles."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


# one to four key tiles of 64 and their edges (an odd and an even number of
# tiles, one key in the last), a second and a third query block
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("L", [1, 63, 64, 65, 128, 129, 191, 193, 257, 320])
def test_attention_tiles(L, dh, causal):
    import torch
    from paper_2608_14586_amd import binding as vb
    B, H, Hkv = 2, 4, 2
    tag = ("pipe", L, dh, causal)
    q = synth.normal_bf16(synth.seed_of("q", *tag), (B, H, L, dh))
    k = synth.normal_bf16(synth.seed_of("k", *tag), (B, Hkv, L, dh))
    v = synth.normal_bf16(synth.seed_of("v", *tag), (B, Hkv, L, dh))
    # keys grow along the sequence, so the maximum rises by more than the lazy
    # rescale's margin in many tiles
    k = torch.from_numpy(synth.as_f32(k) * (1.0 + np.arange(L) / 48.0)[:, None].astype(np.float32)).to(torch.bfloat16)
    ldvt = (L + 15) // 16 * 16 if L % 2 else (L + 63) // 64 * 64
    cols = np.arange(L)
    cols = (cols & ~12) | ((cols & 4) << 1) | ((cols & 8) >> 1)
    vt = np.full((B, Hkv, dh, ldvt), 0x7FC0, np.uint16)  # NaN past the keys: never used
    vt[..., cols] = v.transpose(0, 1, 3, 2)
    o = torch.empty((B, L, H * dh), dtype=torch.bfloat16, device="cuda")
    dq, dvt = (torch.from_numpy(a.view(np.int16)).cuda() for a in (q, vt))
    vb.vla_op_attention_bf16(dq, k.cuda(), dvt, ldvt, o, B, H, Hkv, L, dh, causal)
    torch.cuda.synchronize()
    got, k = o.float().cpu().numpy(), k.float().numpy()
    for b in range(B):
        q64, k64, v64 = (t.transpose(1, 0, 2).astype(np.float64) for t in (synth.as_f32(q[b]), k[b], synth.as_f32(v[b])))
        ref = oracle.attention(q64, k64, v64, causal).reshape(L, H * dh)
        # each probability and each output rounded to bf16 once (2^-8 each):
        # |o - ref| <= 2^-8 |ref| + 2^-8 sum_j p_j |v_j|, with a factor 2
        mag = oracle.attention(q64, k64, np.abs(v64), causal).reshape(L, H * dh)
        err, bound = np.abs(got[b] - ref), 2.0 ** -7 * (np.abs(ref) + mag) + 1e-6
        worst = np.unravel_index(np.argmax(err / bound), err.shape)
        assert (err <= bound).all(), (b, worst, err[worst], bound[worst])
