"""GPU parity of the small-batch regime (17 tokens up to the prefill GEMM's range) for I2_S and TL1 weights, against the
oracle, through bitnet_mpgemm and bitnet_mpgemm_fused: the tile kernels, the decode GEMV in token slices of up to 16 (12, 8
or 4 where a slice's codes must fit in LDS, one launch for all slices), and the boundaries of the regime (113 tokens, no
token sums)."""
import numpy as np
import pytest
import torch

import paper_2502_11880_amd as B
from oracle import bitnet_oracle as O
from paper_2502_11880_amd import inputs
from tests import hip_runner as H
from tests.test_routes_cpu import SLICES, _route

pytestmark = pytest.mark.gpu


def _announce(*what):
    print("case:", *what, flush=True)


def _vs_oracle(layout, M, N, K, seed, rowsum=True):
    W = inputs.weight_f32(N, K, seed=seed)
    x = inputs.activation_f32(M, K, seed=seed + 1)
    packed, w_scale = H.pack(W, layout)
    xq, s, rs = H.quantize(x, with_rowsum=True)
    y, acc = H.mpgemm(layout, packed, w_scale, N, K, xq, s, x_rowsum=rs if rowsum else None)
    y_ref, acc_ref, *_ = O.mpgemm_reference(x.numpy(), W.numpy())
    assert np.array_equal(H.to_np(acc), acc_ref)
    H.check_y(H.to_np(y), y_ref, acc_ref)


# One shape of every size class.  The slices of the GEMV: (32, 4096, 4096), (64, 1024, 8640) and (100, 512, 14336); tiles of
# 32 rows: 320 and 64 of K (4 waves), (48, 208, 3200) (8); of 64 rows: (112, 4096, 4096) and (24, 9600, 4096) (8).
@pytest.mark.parametrize("layout", ["i2s", "tl1"])
@pytest.mark.parametrize("M,N,K", [(17, 64, 320), (24, 9600, 4096), (32, 4096, 4096), (48, 208, 3200),
                                   (64, 1024, 8640), (100, 512, 14336), (112, 4096, 4096), (33, 16, 64)])
def test_small_batch_parity(layout, M, N, K):
    _announce("small batch", layout, M, N, K)
    _vs_oracle(layout, M, N, K, seed=inputs.seed_for(14, M * 7 + N + K))


@pytest.mark.parametrize("layout", ["i2s", "tl1"])
@pytest.mark.parametrize("M,rowsum", [(113, True), (40, False)])
def test_small_batch_boundaries(layout, M, rowsum):
    _announce("small batch boundary", layout, M, rowsum)
    _vs_oracle(layout, M, 256, 1536, seed=inputs.seed_for(14, 900 + M), rowsum=rowsum)


# Every shape of the GEMV's token slices: 4-wave groups (more than 128 row groups, K <= 4096) with 2, 3 and 4 blocks a wave,
# 16-wave groups with 1, 2, 3 and 4; slices of 16, 12 (K = 10112), 8 (12672 and 16128) and 4 (16384) tokens, the last one
# full or of 1 to 15; short last blocks.
@pytest.mark.parametrize("layout", ["i2s", "tl1"])
@pytest.mark.parametrize("M,N,K", [(112, 4608, 1536), (17, 3072, 1536), (33, 2560, 2560), (17, 3456, 3456), (41, 1152, 3392),
                                   (46, 1136, 7808), (31, 512, 10112), (26, 304, 12672), (65, 48, 16128), (109, 16, 16384)])
def test_small_batch_token_slices(layout, M, N, K):
    _announce("small batch token slices", layout, M, N, K)
    assert _route(M, K, [N]) == SLICES
    _vs_oracle(layout, M, N, K, seed=inputs.seed_for(14, 6000 + M + N + K))


# Rows longer than the decode GEMV takes in slices (K > 16384), past 16 tokens: tiles of 32 and 64 rows, and TL1 with more
# than 112 tokens.
@pytest.mark.parametrize("layout", ["i2s", "tl1"])
@pytest.mark.parametrize("M,N,K", [(40, 48, 16448), (129, 32, 33024), (70, 4240, 17088)])
def test_small_batch_long_rows(layout, M, N, K):
    _announce("small batch long rows", layout, M, N, K)
    _vs_oracle(layout, M, N, K, seed=inputs.seed_for(14, 7000 + M + N + K))


# Long rows where the split GEMM is the faster one, unless the workspace is that of one weight.
@pytest.mark.parametrize("split_ws", [False, True], ids=["one weight's workspace", "the group's workspace"])
def test_long_rows_fused(split_ws):
    _announce("long rows fused", split_ws)
    from tests.test_gpu_fused import _fused_case
    _fused_case("i2s", 65, 44096, [256, 256], seed=inputs.seed_for(14, 7500), split_ws=split_ws)


# The 8B-class groups at 32, 64 and 112 tokens through the fused call (the quantiser, then one launch per group).
@pytest.mark.parametrize("layout", ["i2s", "tl1"])
@pytest.mark.parametrize("M,K,Ns", [(32, 4096, [4096, 1024, 1024]), (112, 4096, [14336, 14336]),
                                    (64, 14336, [4096])])
def test_small_batch_fused(layout, M, K, Ns):
    _announce("small batch fused", layout, M, K, Ns)
    from tests.test_gpu_fused import _fused_case
    _fused_case(layout, M, K, Ns, seed=inputs.seed_for(14, 2000 + M + K + len(Ns)))


# Every tile shape of the small-batch kernels at its edges (32-row x 32-token tiles t against 256 CUs): 32 rows with 4 and
# 8 waves, 64 rows with 8 waves (256 < t <= 512) and 4 (to 1024), the wide kernel (past 1024; odd and even numbers of
# 512-k stages); short last blocks of 1, 2 and 3 sub-tiles; row counts that end inside a tile; one token past a tile;
# past 112 tokens the launches that leave the prefill GEMM, and TL1 at its last 256 tokens and one past (TL2 through its
# rewritten words).  Sums are exact integers.
@pytest.mark.parametrize("layout", ["i2s", "tl1"])
@pytest.mark.parametrize("M,N,K", [(65, 304, 704), (97, 48, 1088), (49, 4176, 2112), (112, 5136, 1152),
                                   (112, 8304, 1216), (65, 11024, 1088), (112, 10256, 192), (129, 208, 1344),
                                   (300, 528, 832), (256, 9216, 576), (257, 4128, 320)])
def test_small_batch_shapes(layout, M, N, K):
    _announce("small batch shape", layout, M, N, K)
    _vs_oracle(layout, M, N, K, seed=inputs.seed_for(14, 3000 + M + N + K))


# With the workspace of the largest weight (less than TL1's rewritten words of all of them) and with the whole one.
@pytest.mark.parametrize("split_ws", [False, True], ids=["one weight's workspace", "the group's workspace"])
@pytest.mark.parametrize("layout", ["i2s", "tl1", "tl2"])
@pytest.mark.parametrize("M,K,Ns", [(40, 1536, [1040, 272, 16]), (113, 4096, [4096, 1024, 1024]),
                                    (200, 1152, [3472, 3456])])
def test_small_batch_fused_shapes(layout, M, K, Ns, split_ws):
    _announce("small batch fused shape", layout, M, K, Ns, split_ws)
    from tests.test_gpu_fused import _fused_case
    _fused_case(layout, M, K, Ns, seed=inputs.seed_for(14, 4000 + M + K + len(Ns)), split_ws=split_ws)


# 2^28 rows at 112 tokens: 2^32 threads of the wide kernel in one launch would be one too many, so the tokens go in two.
# Every weight is the same 16 rows over and over, so one small product is the whole oracle.
@pytest.mark.parametrize("layout", ["i2s", "tl1"])
def test_small_batch_more_rows_than_one_launch_holds(layout):
    _announce("small batch, 2^28 rows", layout)
    M, N, K, count = 112, 1 << 25, 64, 8
    W = inputs.weight_f32(16, K, seed=inputs.seed_for(14, 5000))
    x = inputs.activation_f32(M, K, seed=inputs.seed_for(14, 5001))
    tile, scale = H.pack(W, layout)
    packed = tile.repeat(N // 16)
    xq, s, rs = H.quantize(x, with_rowsum=True)
    y = torch.full((M, N), float("nan"), device=H.DEV)           # every weight of the call writes the same values here
    ws = torch.empty(max(16, B.bitnet_mpgemm_fused_workspace_bytes(layout, [N] * count, K, M)), dtype=torch.uint8,
                     device=H.DEV)
    B.bitnet_mpgemm_fused(layout, [packed] * count, [scale] * count, None, xq, s, rs, [y] * count, ws=ws)
    y_ref, acc_ref, *_ = O.mpgemm_reference(x.numpy(), W.numpy())
    first = y[:, :16].clone()
    H.check_y(H.to_np(first), y_ref, acc_ref)
    for m in range(M):
        assert bool((y[m].view(-1, 16) == first[m]).all()), m
