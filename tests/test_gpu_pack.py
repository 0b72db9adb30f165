"""Weight packing where the exact mean and the ternary threshold can go wrong: beta bits and packed bytes of every
ternary layout against the oracle, for weights over many exponents (values outside a wave's window of 32 exponents take
another path), subnormals, zeros, weights of exactly beta / 2 and its neighbours, and ragged tile sizes."""
import numpy as np
import pytest
import torch

from oracle import bitnet_oracle as O
from paper_2502_11880_amd import inputs
from tests import hip_runner as H

PACK = {"i2s": O.pack_i2s, "tl2": O.pack_tl2, "tl1": O.pack_tl1}


def _gauss(N, K):
    return inputs.weight_f32(N, K, seed=inputs.seed_for(21, N + K)).numpy()


def _wide(N, K):
    g = np.random.default_rng(N + K)
    return (g.standard_normal((N, K)) * np.exp2(g.integers(-60, 20, (N, K)))).astype(np.float32)


def _huge(N, K):
    w = _wide(N, K)
    w[0, :8] = [3.0e38, -3.0e38, 1.0e38, 2.0e-38, 1e-45, -1e-45, 0.0, -0.0]
    return w


def _subnormal(N, K):
    g = np.random.default_rng(7)
    return (g.integers(-9, 10, (N, K)).astype(np.int32) * np.float32(1e-45)).astype(np.float32)


def _vanishing(N, K):
    w = np.zeros((N, K), dtype=np.float32)
    w[3, 5] = 1e-45                                          # the mean rounds to 0: every code is 0
    return w


def _half(N, K):
    """One third of the entries +-1, the rest +-1/4: beta = 1/2 and the rest are exactly beta / 2 (t = 0); three of
    them are the neighbours of it (beta still rounds to 1/2)."""
    w = np.full(N * K, 0.25, dtype=np.float32)
    w[::3] = 1.0
    w[1] = np.nextafter(np.float32(0.25), np.float32(1))
    w[2] = -w[1]
    w[4] = np.nextafter(np.float32(0.25), np.float32(0))
    w[5::4] *= -1
    return w.reshape(N, K)


KINDS = {f.__name__[1:]: f for f in (_gauss, _wide, _huge, _subnormal, _vanishing, _half)}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("layout", list(PACK))
@pytest.mark.parametrize("N,K", [(48, 64), (48, 448), (16, 384), (96, 1152), (528, 3200)])
def test_pack_beta_and_bytes(layout, kind, N, K):
    print("case: pack", layout, kind, N, K, flush=True)
    W = KINDS[kind](N, K)
    packed, beta = H.pack(torch.from_numpy(W), layout)
    t_ref, beta_ref = O.ternarize(W)
    assert H.to_np(beta).view(np.uint32)[0] == np.float32(beta_ref).view(np.uint32)
    assert np.array_equal(H.to_np(packed), PACK[layout](t_ref))


def test_threshold_equals_the_rounded_division():
    """clamp(rint(fp32(w / beta)), -1, 1) == 0 exactly where 2 |w| <= beta, for normal and subnormal beta, with w at and
    around beta / 2."""
    g = np.random.default_rng(11)
    bits = np.concatenate([g.integers(1, 0x7F800000, 20000), np.arange(1, 4000), 0x00800000 + np.arange(-2000, 2000),
                           0x7F800000 - np.arange(1, 2000)]).astype(np.uint32)
    beta = bits.view(np.float32)
    half = (beta * np.float32(0.5)).view(np.uint32).astype(np.int64)
    with np.errstate(over="ignore"):
        for d in range(-4, 5):
            w = np.clip(half + d, 0, 0x7F7FFFFF).astype(np.uint32).view(np.float32)
            assert np.array_equal(np.rint(w / beta) == 0, w + w <= beta), d
