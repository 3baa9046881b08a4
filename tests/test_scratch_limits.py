"""Scratch that calls may ask for (host code): a limit that callers who keep a workspace, or pass none, rely on."""
import math
import random

import pytest

from paper_2308_09723_amd import fq


def _integer_path_slabs(M, N, K):
    """Slabs of int32 partial sums that filling 256 compute units alone asks for."""
    KB, tiles16 = K // 128, N // 16
    if M <= 16:
        groups, best, slabs = -(-tiles16 // 3), -1.0, 1
        for gp in range(1, 13):
            kw = min(12 // gp, KB)
            if M * 8 > 128 * gp:                      # more than two activation units per lane
                continue
            blocks, turns = -(-groups // gp), -(-KB // kw)
            gs = min(256 // blocks if blocks <= 128 else 1, 8, turns)
            rounds = -(-blocks * gs // 256)
            score = (groups * gs / (rounds * 256 * gp)) ** 2 * min(1.0, math.sqrt(gp * kw * 6 / 64)) / (1 + 0.1 * (rounds - 1))
            score *= (0.8 if M * 8 > 64 * gp else 1.0) * (0.8 if gs > 1 else 1.0)
            score *= (0.85 if gp * kw < 6 else 1.0) * (0.95 if kw == 1 else 1.0)
            if score > best + 1e-9:
                best, slabs = score, gs
        return slabs
    rows = 32 if M <= 32 else 64 if M <= 64 else 128
    tiles = -(-M // rows) * -(-N // 384)
    slabs = min(256 // tiles if tiles < 192 else 1, 8, KB)
    return -(-KB // -(-KB // slabs))


def _most_bytes(M, N, K):
    slabs = _integer_path_slabs(M, N, K)
    return slabs * M * N * 4 if slabs > 1 else 0


@pytest.mark.parametrize("M,K,N,g", [(470, 14848, 15296, 64), (697, 15104, 10240, 128), (1313, 15616, 5360, 128), (376, 15616, 21136, 128),
                                     (1229, 15360, 6176, 96), (253, 16256, 29088, 128), (2, 8192, 2928, 128), (13, 15744, 11040, 96),
                                     (10, 5376, 1392, 96)])
def test_integer_path_asks_for_no_more_than_filling_the_chip_takes(M, K, N, g):
    assert fq.gemm_w4a8_workspace_bytes(M, N, K, g) <= _most_bytes(M, N, K)


def test_integer_path_scratch_over_many_shapes():
    r = random.Random(6)
    split = 0
    for _ in range(6000):
        M, K, N = (int(math.exp(r.uniform(0.0, math.log(m)))) for m in (4096, 128, 2600))
        K, N = 128 * K, 16 * N
        g = r.choice([g for g in (32, 64, 96, 128, 0) if g == 0 or K % g == 0])
        need = fq.gemm_w4a8_workspace_bytes(M, N, K, g)
        assert need <= _most_bytes(M, N, K), (M, K, N, g)
        split += need > 0
    assert split > 300


def test_one_workspace_size_serves_every_type():
    """fq_gemm_workspace_bytes is the largest need over activation types and scale formats, on narrow matrices too, where binary16
    products alone take some block shapes."""
    r = random.Random(7)
    for _ in range(20000):
        M, K, N = (int(math.exp(r.uniform(math.log(a), math.log(b)))) for a, b in ((49, 2400), (1, 64), (1, 511)))
        K, N = 128 * K, 16 * N
        bits, g = r.choice([3, 4, 8]), r.choice([32, 64, 128])
        most = fq.gemm_workspace_bytes(M, N, K, bits, g)
        assert all(fq.gemm_workspace_bytes_for(M, N, K, bits, g, a, s) <= most for a, s in ((0, 0), (1, 0), (1, 1))), (M, K, N, bits, g)
