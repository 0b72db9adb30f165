"""The host rules that choose a kernel, on the CPU (256 CUs are assumed where there is no device): launches whose routes
were measured against each other go where they were faster."""
import ctypes

import pytest

import paper_2502_11880_amd as B

MAX_FUSED = 8
SLICES, T32X4, T32X8, T64X8, T64X4, WIDE = range(6)


class FusedLinears(ctypes.Structure):
    """bitnet::FusedLinears (csrc/bitnet_internal.hpp)."""
    _fields_ = [("packed", ctypes.c_void_p * MAX_FUSED), ("w_scale", ctypes.c_void_p * MAX_FUSED),
                ("y", ctypes.c_void_p * MAX_FUSED), ("acc", ctypes.c_void_p * MAX_FUSED), ("N", ctypes.c_int * MAX_FUSED),
                ("rg_start", ctypes.c_int * (MAX_FUSED + 1)), ("count", ctypes.c_int), ("total", ctypes.c_int)]


def _linears(Ns):
    L = FusedLinears()
    for i, N in enumerate(Ns):
        L.N[i] = N
        L.rg_start[i] = L.total
        L.total += N // 16
    L.count = len(Ns)
    return L


def _call(name, res, *args):
    fn = getattr(B.lib(), name)
    fn.restype = res
    return fn(*args)


def _route(M, K, Ns):
    return _call("_ZN6bitnet16smallbatch_routeERKNS_12FusedLinearsEll", ctypes.c_int, ctypes.byref(_linears(Ns)),
                 ctypes.c_int64(M), ctypes.c_int64(K))


def _beats(M, K, Ns, rewrite, split_fits=True):
    return _call("_ZN6bitnet24smallbatch_beats_prefillERKNS_12FusedLinearsEllbb", ctypes.c_bool, ctypes.byref(_linears(Ns)),
                 ctypes.c_int64(M), ctypes.c_int64(K), ctypes.c_bool(rewrite), ctypes.c_bool(split_fits))


# Slices of the GEMV against the tiles: the difference was 7% or more of the time.
@pytest.mark.parametrize("M,K,Ns,route", [
    (31, 10112, [512], SLICES), (84, 11648, [64], SLICES), (96, 12608, [32], SLICES), (32, 9280, [800], SLICES),
    (24, 10688, [3072], SLICES), (112, 1536, [1536] * 3, SLICES), (41, 3392, [1152], SLICES), (46, 7808, [1136], SLICES),
    (33, 3520, [1280], SLICES), (26, 12672, [304], SLICES), (17, 3456, [3456], SLICES),
    (45, 4096, [4096, 1024, 1024], T64X8), (45, 14336, [4096], T32X8), (45, 4096, [14336] * 2, WIDE),
    (32, 4096, [14336] * 2, T64X4), (92, 1088, [1088], T32X8), (112, 4096, [4096] * 3, WIDE), (64, 1024, [3072] * 2, T32X4),
    (98, 2048, [6144] * 2, WIDE), (106, 2880, [4176], T64X4)])
def test_small_batch_routes(M, K, Ns, route):
    assert _route(M, K, Ns) == route


# The prefill GEMM against the small-batch kernels, past 112 tokens or K = 16384; with TL1's rewrite in the last column.
@pytest.mark.parametrize("M,K,Ns,rewrite,small", [
    (67, 22720, [7488], False, False), (34, 26752, [9024], False, False), (87, 22720, [6848], False, False),
    (120, 4096, [4096, 1024, 1024], False, True), (512, 4096, [4096], False, True), (256, 14336, [4096], False, True),
    (2048, 4096, [4096, 1024, 1024], False, False), (512, 4096, [14336] * 2, False, False),
    (192, 4096, [14336] * 2, True, True), (256, 4096, [4096], True, True), (256, 3200, [8640] * 2, True, True),
    (253, 1472, [32224] * 2, True, False), (248, 1664, [23792] * 2, True, False), (240, 3712, [29472] * 2, True, False)])
def test_prefill_or_small_batch(M, K, Ns, rewrite, small):
    assert _beats(M, K, Ns, rewrite) is small


# A fused call may bring the workspace of its largest weight alone, which does not hold the slices of all of them.
@pytest.mark.parametrize("M,K,Ns", [(65, 44096, [256, 256]), (400, 17472, [640, 640])])
def test_a_split_without_its_workspace_is_not_waited_for(M, K, Ns):
    assert not _beats(M, K, Ns, False) and _beats(M, K, Ns, False, split_fits=False)
