"""The GEMM's tiles over the sizes where the choice changes, whole blocks of few
rows, and several sequences in one call."""
import numpy as np
import pytest

import oracle
import synth
from paper_2608_14586_amd import binding as vb
from prefix_cases import EncCase, LlmCase, rel_l2, to_f32
from test_gemm_routes import T192x256, TILES

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16) if a.dtype == np.uint16 else a.copy()).cuda()


# the tiles the estimate takes at short K (64x64, 64x128 and 128x128, 256x256
# for the two widest GELU grids): rows and columns on and off the tile edges,
# grids of a few workgroups, about one per CU, about two, and several rounds
@pytest.mark.parametrize("M,N,K", [(1, 96, 64), (19, 4096, 128), (64, 896, 192), (65, 1152, 256), (130, 4096, 320),
                                   (203, 1000, 384), (257, 3072, 448), (513, 4096, 512), (1001, 4096, 192),
                                   (1154, 1024, 1024), (1300, 9728, 128), (2050, 4096, 256)])
def test_products_over_tiles(M, N, K):
    import torch
    A = synth.normal_bf16(synth.seed_of("tileA", M, N, K), (M, K))
    W = synth.normal_bf16(synth.seed_of("tileW", M, N, K), (N, K))
    b = synth.normal_f32(synth.seed_of("tileb", M, N, K), (N,))
    H0 = synth.normal_f32(synth.seed_of("tileH", M, N, K), (M, N))
    H, out = _dev(H0), torch.empty((M, N), dtype=torch.int16, device="cuda")
    dA, dW, db = _dev(A), _dev(vb.vla_op_pack_weight_bf16(W, N, K)), _dev(b)
    vb.vla_op_gemm_residual_bf16(dA, dW, H, db, M, N, K)
    vb.vla_op_gemm_bias_bf16(dA, dW, out, db, M, N, K, True)
    torch.cuda.synchronize()
    a64, w64 = synth.as_f32(A).astype(np.float64), synth.as_f32(W).astype(np.float64)
    z, mag = a64 @ w64.T + b, np.abs(a64) @ np.abs(w64).T
    # fp32 accumulation: K / 16 MFMA steps, each one rounding of the running
    # sum (<= 2^-18 of the sum of |products| for K <= 1024), with a factor 4
    acc = 2.0 ** -16 * mag + 2.0 ** -22 * (np.abs(z) + np.abs(H0))
    err = np.abs(H.cpu().numpy() - (H0 + z))
    assert (err <= acc).all(), np.unravel_index(np.argmax(err - acc), err.shape)
    ref = oracle.gelu_erf(z)
    # and one bf16 rounding (2^-9, with a factor 2), GELU's slope (<= 1.13),
    # and the erfc approximation (1.5e-7 on Phi)
    err = np.abs(synth.as_f32(out.cpu().numpy().view(np.uint16)) - ref)
    bound = 2.0 ** -8 * np.abs(ref) + 1.2 * acc + 2e-7 * np.abs(z)
    assert (err <= bound).all(), np.unravel_index(np.argmax(err - bound), err.shape)


# Every tile of every epilogue, whatever the estimate takes it for: one row, one
# off and two past a tile's edge in rows, columns cut inside the tile (whole
# tiles where it is only for those), K of one slab to one past the deepest ring
# (four slabs).  Element by element; nothing beside the output is written.
@pytest.mark.parametrize("op,tile", [(op, t) for op in (vb.VLA_GEMM_RESIDUAL, vb.VLA_GEMM_BIAS, vb.VLA_GEMM_GELU)
                                     for t in TILES[op]])
def test_each_tile(op, tile):
    import torch
    bm, bn, _ = tile
    whole = tile == T192x256
    tag = ("each", op) + tile
    Ns = [2 * bn] if whole else [8, bn - 8, bn + 8, 2 * bn]
    A = synth.normal_bf16(synth.seed_of("A", *tag), (2 * bm + 2, 320))
    W = synth.normal_bf16(synth.seed_of("W", *tag), (2 * bn, 320), std=0.3)
    b = synth.normal_f32(synth.seed_of("b", *tag), (2 * bn,))
    H0 = synth.normal_f32(synth.seed_of("H", *tag), (2 * bm + 2, 2 * bn))
    a64, w64 = synth.as_f32(A).astype(np.float64), synth.as_f32(W).astype(np.float64)
    for i, (M, K) in enumerate([(1, 128), (bm - 1, 320), (bm, 64), (bm + 1, 192), (2 * bm + 2, 256)]):
        N = Ns[i % len(Ns)]
        dA = _dev(np.ascontiguousarray(A[:M, :K]))
        dW = _dev(vb.vla_op_pack_weight_bf16(np.ascontiguousarray(W[:N, :K]), N, K))
        bias = _dev(b[:N]) if i % 2 == 0 else None
        z = a64[:M, :K] @ w64[:N, :K].T + (b[:N] if i % 2 == 0 else 0.0)
        mag = np.abs(a64[:M, :K]) @ np.abs(w64[:N, :K]).T
        if op == vb.VLA_GEMM_RESIDUAL:
            out = torch.full((M * N + 4096,), 7.0, device="cuda")
            out[:M * N] = _dev(H0[:M, :N]).reshape(-1)
            guard, ref = 7.0, H0[:M, :N] + z
        else:
            out = torch.full((M * N + 4096,), 7.0, dtype=torch.bfloat16, device="cuda")
            guard, ref = 7.0, oracle.gelu_erf(z) if op == vb.VLA_GEMM_GELU else z
        vb.vla_op_gemm_tile_bf16(op, tile, dA, dW, out, bias, M, N, K)
        torch.cuda.synchronize()
        got = out.float().cpu().numpy()
        assert (got[M * N:] == guard).all(), (M, N, K)
        err = np.abs(got[:M * N].reshape(M, N) - ref)
        # fp32 accumulation (K / 16 <= 20 roundings of the running sum, 2^-24
        # each, with a factor 4) and the sums after it; for bf16 outputs one
        # rounding (2^-9, with a factor 2) behind GELU's slope (<= 1.13) and
        # the erfc approximation (1.5e-7 on Phi)
        acc = 80 * 2.0 ** -24 * mag + 2.0 ** -22 * (np.abs(z) + np.abs(ref))
        bound = acc if op == vb.VLA_GEMM_RESIDUAL else 2.0 ** -8 * np.abs(ref) + 1.2 * acc + 2e-7 * np.abs(z)
        worst = np.unravel_index(np.argmax(err - bound), err.shape)
        assert (err <= bound).all(), ((M, N, K), worst, err[worst], bound[worst])
    # a tile that is not this product's, or not for these columns, is refused
    for t in [(256, 192, 8), (128, 64, 4)] + ([tile] if whole else []):
        with pytest.raises(vb.VlaError) as e:
            vb.vla_op_gemm_tile_bf16(op, t, dA, dW, out, bias, M, 24, K)
        assert e.value.name == "VLA_ERR_UNSUPPORTED"


@pytest.mark.parametrize("name,L,B", [("small_llm", 1, 1), ("small_llm", 19, 1), ("small_llm", 65, 2),
                                      ("small_llm", 333, 1), ("llm7b", 33, 1), ("llm7b", 203, 1)])
def test_blocks_of_few_rows(name, L, B):
    """Few rows, where the residual products leave most of the chip idle.  The
    boundary (bf16, fp32), the next block's norm and the KV match the oracle, a
    run in two ranges is bit for bit one run, and a context with room for more
    rows gives the same bits."""
    k = 2 if name == "small_llm" else 1
    c = LlmCase(name, L, k, B=B, perturbed=True)
    tok = c.tokens(frame=4)
    ref, kv = c.oracle(tok)
    whole = c.run(tok, frame=1, out_dtype="f32")
    assert rel_l2(whole.hidden.numpy(), ref) <= 1e-2
    assert max(rel_l2(to_f32(whole.kv[l]), kv[l]) for l in range(k)) <= 1e-2
    assert rel_l2(to_f32(c.run(tok, frame=2).hidden), ref) <= 1e-2
    first = c.run(tok, frame=3, k1=k - 1, out_dtype="f32")
    second = c.run(first.hidden.numpy().copy(), frame=4, k0=k - 1, out_dtype="f32")
    assert np.array_equal(second.hidden.numpy(), whole.hidden.numpy())
    c.close()
    big = LlmCase(name, L, k, B=B, perturbed=True, max_tokens=1024)
    assert np.array_equal(big.run(tok, frame=1, out_dtype="f32").hidden.numpy(), whole.hidden.numpy())
    big.close()


@pytest.mark.parametrize("n_img,L", [(1, 50), (2, 131), (1, 257)])
def test_encoder_blocks_of_few_rows(n_img, L):
    c = EncCase("vit_l", n_img, L, n_blocks=2, perturbed=True)
    p = c.patches(frame=2)
    assert rel_l2(to_f32(c.run(p)), c.oracle(p)) <= 1e-2
    c.close()


# fp32 path: head dims that are not multiples of 4 or 16, rows that are not
# 16-byte aligned (odd widths), K and L off the step of 8, the query tile of
# 16 and the key tile of 64, grouped heads; a grid of 64x64 tiles (the last)
@pytest.mark.parametrize("d,H,Hkv,dh,F,L,B", [(36, 3, 1, 10, 50, 17, 1), (64, 2, 2, 128, 129, 65, 2),
                                              (100, 4, 2, 6, 77, 1, 1), (256, 4, 4, 64, 688, 130, 1),
                                              (132, 2, 1, 66, 31, 16, 3), (512, 8, 2, 64, 8200, 200, 1)])
def test_fp32_path_odd_shapes(d, H, Hkv, dh, F, L, B):
    s = synth.configs.llama_like(2, d, H, Hkv, dh, F)
    wl = synth.Workload("tile_f32_%d_%d" % (d, F), "f32", s, None, batch=B, seq=L)
    W = [synth.llm_block_weights(wl, l, perturbed=True) for l in range(2)]
    ctx = vb.Context(llm=vb.stack_cfg(s, "f32", max_tokens=L, max_batch=B))
    for l in range(2):
        ctx.vla_load_block_weights(vb.VLA_STACK_LLM, l, W[l])
    tok = synth.tokens(wl, frame=1)
    bnd = vb.Boundary(B, L, d, 2, Hkv, dh, stack_dtype="f32", out_dtype="f32")
    ctx.vla_run_prefix(1, tok, B, L, 2, bnd)
    ctx.vla_wait_boundary(1, 60000)
    W64 = [{n: a.astype(np.float64) for n, a in w.items()} for w in W]
    ref, kv = oracle.run_prefix(tok.astype(np.float64), lambda l: W64[l], s, 2, dtype=np.float64)
    # fp32 sums of up to 8200 products in chains of a quarter of them: well
    # under 1e-5; a dropped or doubled element is off by more than 1e-3
    assert rel_l2(bnd.hidden.numpy(), ref) <= 1e-5
    assert rel_l2(bnd.kv.numpy(), kv) <= 1e-5
    ctx.vla_destroy()


# Several sequences in one call, of lengths that are not multiples of 16 (or of
# the quad, or shorter than a group): the V^T groups of a sequence are cut by
# tiles and by its neighbours.  Every row's sums run in one order in every tile,
# so each sequence is bit for bit its own call.
@pytest.mark.parametrize("L,B", [(1, 4), (3, 4), (15, 3), (16, 4), (17, 4), (31, 3), (50, 4), (66, 4), (77, 3),
                                 (130, 4), (333, 2)])
def test_sequences_side_by_side(L, B):
    import torch
    s = synth.configs.llama_like(2, 256, 4, 2, 64, 384)
    wl = synth.Workload("tile_seqs", "bf16", s, None, batch=B, seq=L)
    ctx = vb.Context(llm=vb.stack_cfg(s, "bf16", max_tokens=L, max_batch=B))
    for l in range(2):
        ctx.vla_load_block_weights(vb.VLA_STACK_LLM, l, synth.llm_block_weights(wl, l, perturbed=True))
    tok = synth.tokens(wl, frame=1)

    def run(frame, t, n):
        bnd = vb.Boundary(n, L, 256, 2, 2, 64, stack_dtype="bf16", out_dtype="f32")
        ctx.vla_run_prefix(frame, t, n, L, 2, bnd)
        ctx.vla_wait_boundary(frame, 60000)
        return bnd.hidden.numpy().copy(), bnd.kv.view(torch.int16).numpy().copy()

    hid, kv = run(1, tok, B)
    assert np.isfinite(hid).all()
    for b in range(B):
        h1, kv1 = run(2 + b, np.ascontiguousarray(tok[b:b + 1]), 1)
        assert np.array_equal(h1[0], hid[b]), (b, np.argwhere(h1[0] != hid[b])[:3])
        assert np.array_equal(kv1[:, :, 0], kv[:, :, b]), b
    ctx.vla_destroy()


# 192x128 tiles: long K where they leave one tile per CU, ragged rows, the last
# tile of columns cut, one row past a tile
@pytest.mark.parametrize("M,N,K", [(1345, 4000, 4096), (1153, 4096, 4096), (4801, 1024, 4096)])
def test_residual_192_row_tiles(M, N, K):
    import torch
    A = synth.normal_bf16(synth.seed_of("t192A", M, N, K), (M, K))
    W = synth.normal_bf16(synth.seed_of("t192W", M, N, K), (N, K))
    H0 = synth.normal_f32(synth.seed_of("t192H", M, N, K), (M, N))
    H, b = _dev(H0), synth.normal_f32(synth.seed_of("t192b", M, N, K), (N,))
    vb.vla_op_gemm_residual_bf16(_dev(A), _dev(vb.vla_op_pack_weight_bf16(W, N, K)), H, _dev(b), M, N, K)
    torch.cuda.synchronize()
    rows = np.unique(np.r_[0:M:37, 190:194, M - 3:M])
    a64, w64 = synth.as_f32(A)[rows].astype(np.float64), synth.as_f32(W).astype(np.float64)
    z, mag = a64 @ w64.T + b, np.abs(a64) @ np.abs(w64).T
    # K / 16 MFMA steps of one fp32 rounding each (2^-24), with a factor 4
    acc = K / 16 * 2.0 ** -22 * mag + 2.0 ** -22 * (np.abs(z) + np.abs(H0[rows]))
    err = np.abs(H.cpu().numpy()[rows] - (H0[rows] + z))
    assert (err <= acc).all(), np.unravel_index(np.argmax(err - acc), err.shape)


# Products in two launches, whole rounds of 256-column tiles and the rest in
# smaller ones: every column of both, with rows off the tiles.  A column's sums
# run over K in one order in every tile, so the columns equal, bit for bit,
# those of a product of the first columns alone (one launch).
@pytest.mark.parametrize("M,N,K,cut", [(1001, 22016, 4096, 4096), (700, 22016, 4096, 8192), (4206, 4096, 1024, 512)])
def test_products_in_two_launches(M, N, K, cut):
    import torch
    A = synth.normal_bf16(synth.seed_of("twoA", M, N, K), (M, K))
    W = synth.normal_bf16(synth.seed_of("twoW", M, N, K), (N, K))
    b = synth.normal_f32(synth.seed_of("twob", M, N, K), (N,))
    dA = _dev(A)

    def product(n0, n1):
        out = torch.full((M, n1 - n0), 0x7FC0, dtype=torch.int16, device="cuda")
        vb.vla_op_gemm_bias_bf16(dA, _dev(vb.vla_op_pack_weight_bf16(np.ascontiguousarray(W[n0:n1]), n1 - n0, K)), out,
                                 _dev(b[n0:n1]), M, n1 - n0, K, True)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    whole = product(0, N)
    for n0 in list(range(0, N - cut, cut)) + [N - cut]:
        assert np.array_equal(product(n0, n0 + cut), whole[:, n0:n0 + cut]), n0
