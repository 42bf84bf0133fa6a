"""Which GEMM kernel a product takes, by rows and sizes (host only)."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_17299_amd", "libwar.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libwar.so not built")
PARTIAL, ARGMAX, SWIGLU = 0, 1, 2


def _plan(*a, **k):
    from paper_2607_17299_amd import war
    return war.debug_gemm_plan(*a, **k)


@pytest.mark.parametrize("M,ids,tiled", [
    (80, 151936, False), (81, 151936, False), (96, 151936, False), (97, 151936, True), (96, 257 * 128, False),
    (80, 32768, False), (81, 32768, True), (96, 1024, True)])
def test_large_lm_heads_stream_up_to_96_rows(M, ids, tiled):
    for K in (1024, 4096, 5120):
        shape, splits, kper = _plan(M, ids, K, ARGMAX)
        assert (shape >= 0) == tiled and (splits, kper) == (1, K)


# (N, K, rows, splits): counts of an unrolled kernel, or the runtime loop where that
# is still the faster (11008, 28672, 15360: the other count has far more workgroups
# than CUs, or fewer and a longer loop)
@pytest.mark.parametrize("N,K,rows,splits", [
    (4096, 12288, (1, 32, 64, 80), 8), (6144, 4096, (1, 48, 80), 4), (4096, 4096, (1, 48, 80), 8),
    (1024, 1024, (1, 48, 80), 16), (1024, 4096, (1, 48, 80), 32), (1536, 1024, (1, 80), 16),
    (4096, 14336, (1, 16, 48, 72), 7), (3584, 3584, (1, 16, 48, 72), 7), (2048, 6144, (1, 48, 80), 12),
    (2560, 9728, (1, 48, 80), 19), (5120, 17408, (1, 16, 48, 72), 8), (6144, 16384, (16, 72), 8),
    (6144, 16384, (48,), 4), (10240, 8192, (16, 72), 4), (10240, 8192, (48,), 2), (20480, 4096, (16, 72), 2),
    (4096, 11008, (16, 48, 72), 4), (8192, 28672, (1, 16, 48, 72), 4), (4096, 15360, (1, 48, 72), 8),
    (7168, 18432, (1, 48, 72), 4)])
def test_split_counts(N, K, rows, splits):
    for M in rows:
        shape, s, kper = _plan(M, N, K, PARTIAL)
        assert (shape, s, kper) == (-1, splits, K // splits), M


@pytest.mark.parametrize("d", [896, 1024, 2048, 2560, 3072, 3584, 4096, 5120, 6144, 8192])
def test_splits_cover_k_within_the_cap(d):
    for N, K in [(d, d), (d, 3 * d), (d, 128 * 37), (3 * d // 128 * 128, d)]:
        for M in (1, 17, 33, 64, 65, 80, 81, 200, 2048):
            for cap in (64 << 20, 64 * M * N, M * N):
                shape, s, kper = _plan(M, N, K, PARTIAL, cap)
                if s == 0:
                    continue
                assert kper % 64 == 0 and (s - 1) * kper < K <= s * kper and s * M * N <= cap


@pytest.mark.parametrize("M,N,K,epi,shape", [
    (193, 12288, 4096, PARTIAL, 0), (512, 24576, 4096, ARGMAX, 0), (512, 24576, 4096, SWIGLU, 0),
    (129, 12288, 4096, PARTIAL, 1), (257, 24576, 4096, ARGMAX, 1), (257, 24576, 4096, SWIGLU, 1),
    (81, 12288, 4096, PARTIAL, 2), (193, 24576, 4096, ARGMAX, 2), (193, 24576, 4096, SWIGLU, 2),
    (193, 6528, 4096, PARTIAL, 3), (1280, 6528, 4096, ARGMAX, 3),
    (129, 6144, 4096, PARTIAL, 4), (129, 24576, 4096, ARGMAX, 4), (129, 24576, 4096, SWIGLU, 4),
    (81, 4096, 4096, PARTIAL, 5), (81, 4096, 4096, ARGMAX, 5), (81, 1024, 4096, SWIGLU, 5)])
def test_tile_shapes(M, N, K, epi, shape):
    """Every kernel there is has sizes that take it."""
    assert _plan(M, N, K, epi)[0] == shape


def test_gate_up_never_takes_the_256_by_128_tile():
    """(It has no such kernel.)"""
    for N in range(256, 65537, 256):
        for M in (81, 128, 129, 192, 256, 257, 300, 384, 512, 600, 768, 1000, 1152, 1280, 1536, 2048, 4096, 65536):
            assert _plan(M, N, 64, SWIGLU)[0] not in (-1, 3)
