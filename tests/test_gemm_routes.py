"""How the products of the blocks run, by size: the tile or the two launches
that the cost estimate chooses.  The GPU tests that are written for one tile
name its shapes here too, so that a change of the estimate cannot move them
onto another kernel unseen.  Host only."""
import pytest

from paper_2608_14586_amd import binding as vb

T64, T64x128, T128, T128x4 = (64, 64, 4), (64, 128, 4), (128, 128, 8), (128, 128, 4)
T256x128, T256, T256x192 = (256, 128, 8), (256, 256, 8), (256, 192, 8)
T192x384, T192x256, T192x128 = (192, 384, 8), (192, 256, 8), (192, 128, 8)
F32, RES, BIAS = vb.VLA_GEMM_F32, vb.VLA_GEMM_RESIDUAL, vb.VLA_GEMM_BIAS
GELU, SWIGLU, QKV = vb.VLA_GEMM_GELU, vb.VLA_GEMM_SWIGLU, vb.VLA_GEMM_QKV
TILES = {RES: [T64, T64x128, T128, T128x4, T256x128, T192x128],
         BIAS: [T64, T64x128, T128, T128x4, T256x128, T256, T192x128],
         GELU: [T64, T64x128, T128, T128x4, T256x128, T256, T192x256, T192x128],
         SWIGLU: [T64x128, T128, T128x4, T256x128, T256],
         QKV: [T64, T64x128, T128, T128x4, T256x128, T256x192, T192x384, T192x128],
         F32: [T64, T64x128, T128, T128x4, T256x128, T256]}


@pytest.mark.parametrize("op,M,N,K,parts,want", [
    # the blocks: 7B prefixes of 203, 1001 and 2048 tokens, ViT-L over six
    # cameras of 1024 patches, the 0.5B decoder over 4096
    (QKV, 203, 12288, 4096, 1, [T128]), (QKV, 2048, 12288, 4096, 1, [T256x192]),
    (SWIGLU, 203, 22016, 4096, 1, [T256x128]), (SWIGLU, 2048, 22016, 4096, 1, [T256]),
    (SWIGLU, 1001, 22016, 4096, 1, [(16384, T256), (5632, T256x128)]),
    (RES, 203, 4096, 4096, 1, [T64]), (RES, 203, 4096, 11008, 1, [T64]),
    (RES, 1001, 4096, 4096, 1, [T128]), (RES, 1001, 4096, 11008, 2, [T128]),
    (RES, 2048, 4096, 4096, 1, [T256x128]), (RES, 2048, 4096, 11008, 1, [T256x128]),
    (QKV, 6144, 3072, 1024, 1, [T192x384]), (RES, 6144, 1024, 1024, 1, [T128x4]),
    (GELU, 6144, 4096, 1024, 1, [T192x256]), (RES, 6144, 1024, 4096, 1, [T192x128]),
    (QKV, 4096, 1280, 896, 1, [T128x4]), (SWIGLU, 4096, 9728, 896, 1, [T256]),
    # residual products of several rounds at short K: not the tile whose
    # epilogue the next round waits for
    (RES, 16384, 8192, 1024, 1, [T128x4]), (RES, 24576, 1024, 1024, 1, [T128x4]), (RES, 4096, 8192, 1024, 1, [T128x4]),
    (RES, 1600, 4096, 4096, 1, [T256x128]),
    # test_gpu_ops, test_gpu_tiles, test_gpu_rows
    (GELU, 6144, 4096, 128, 1, [T128x4]), (GELU, 6000, 4096, 64, 1, [T128x4]), (BIAS, 2048, 16384, 64, 1, [T256]),
    (GELU, 300, 1000, 128, 1, [T64]), (BIAS, 2048, 16384, 4096, 1, [T256]), (RES, 6104, 1000, 192, 1, [T128x4]),
    (RES, 1024, 4096, 128, 1, [T64x128]), (RES, 1345, 4000, 4096, 1, [T192x128]),
    (RES, 1153, 4096, 4096, 1, [T192x128]), (RES, 4801, 1024, 4096, 1, [T192x128]),
    (GELU, 700, 22016, 4096, 1, [(21760, T256), (256, T64)]), (GELU, 4206, 4096, 1024, 1, [(3840, T256), (256, T64)]),
    (QKV, 2113, 12288, 4096, 1, [(10752, T256x192), (1536, T128)]),
    (QKV, 1601, 12288, 4096, 2, [(10752, T192x384), (1536, T128)]),
    (QKV, 1000, 12288, 4096, 1, [T256x192]), (QKV, 1000, 12288, 4096, 2, [T256x192]),
    (SWIGLU, 2113, 22016, 4096, 1, [(21760, T256), (256, T64x128)]),
    (SWIGLU, 1000, 22016, 4096, 1, [(16384, T256), (5632, T256x128)]),
])
def test_route(op, M, N, K, parts, want):
    want = [w if isinstance(w[1], tuple) else (N, w) for w in want]
    assert vb.vla_op_gemm_route(op, M, N, K, parts) == want


@pytest.mark.parametrize("op,shapes", [
    (RES, [(4096, 4096), (4096, 11008), (896, 4864), (1024, 1024), (1024, 4096)]), (BIAS, [(4096, 4096), (896, 896)]),
    (GELU, [(4096, 1024), (4096, 4096)]), (SWIGLU, [(22016, 4096), (9728, 896)]),
    (QKV, [(12288, 4096), (1280, 896), (3072, 1024)]), (F32, [(4096, 4096), (1000, 512), (16384, 1024)])])
def test_every_tile_is_chosen_somewhere(op, shapes):
    """Over 1 to 6144 rows of the blocks' products: no other tile than the ones
    the forced-tile test runs, and none of them for nothing.  A split covers
    all columns."""
    seen = set()
    for M in sorted({int(1.05 ** i) for i in range(180)}):
        for N, K in shapes:
            for parts in (1, 2):
                route = vb.vla_op_gemm_route(op, M, N, K, parts)
                assert sum(n for n, _ in route) == N
                assert len(route) == 1 or (op != RES and route[0][0] % route[0][1][1] == 0)
                seen |= {t for _, t in route}
    assert seen == set(TILES[op])


def test_route_refuses():
    for args in ((RES, 0, 64, 64, 1), (RES, 1, 0, 64, 1), (RES, 1, 64, 100, 1), (RES, 1, 64, 64, 3)):
        with pytest.raises(vb.VlaError):
            vb.vla_op_gemm_route(*args)
    with pytest.raises(vb.VlaError) as e:
        vb.vla_op_gemm_route(6, 1, 64, 64, 1)
    assert e.value.name == "VLA_ERR_INVALID_ARG"
