"""The GEMM kernels one by one (war_debug_gemm) against float64 products of the
same bf16 operands: every tile shape and every few-row kernel with each of their
epilogues, at the edges of the row tiles, over 1, 2 and 3 k-steps (fewer than the
pipelines have stages), with uneven last splits, and with widths that leave the
last 256-column tile half empty and the last group of n-blocks short.

Bound: an fp32 sum of n products in any order is off by at most n 2^-24 sum |a w|
(each step rounds once; the products are exact).  SwiGLU adds its bf16 result's
half unit (8 significant bits: at most 2^-8 of the value) and a few fp32 roundings."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
PARTIAL, ARGMAX, SWIGLU = 0, 1, 2
TILES = [(256, 256), (192, 256), (128, 256), (256, 128), (192, 128), (128, 128)]


def _operands(M, N, K, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    new = lambda *s: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g)
    return new(M, K), new(N, K)


def _check_partial(war, A, W, shape, splits, kper):
    got = war.debug_gemm(A, W, PARTIAL, shape, splits, kper)
    K = A.shape[1]
    for s in range(splits):
        a, w = A[:, s * kper:min(K, (s + 1) * kper)].double(), W[:, s * kper:min(K, (s + 1) * kper)].double()
        err = (got[s].double() - a @ w.t()).abs()
        assert (err <= a.shape[1] * 2.0 ** -24 * (a.abs() @ w.abs().t())).all(), (tuple(A.shape), tuple(W.shape), shape, s)


def _check_argmax(war, A, W, shape, a_rows=None):
    got, best, col = war.debug_gemm(A, W, ARGMAX, shape, a_rows=a_rows)
    a, w = (A if a_rows is None else A[a_rows.long()]).double(), W.double()
    err = (got.double() - a @ w.t()).abs()
    assert (err <= A.shape[1] * 2.0 ** -24 * (a.abs() @ w.abs().t())).all(), (tuple(A.shape), tuple(W.shape), shape)
    blocks = got.cpu().numpy().reshape(got.shape[0], -1, 128)
    np.testing.assert_array_equal(best.cpu().numpy(), blocks.max(-1))
    np.testing.assert_array_equal(col.cpu().numpy(), blocks.argmax(-1) + 128 * np.arange(blocks.shape[1]))


def _check_swiglu(war, A, W, shape):
    F, K = W.shape[0] // 2, A.shape[1]
    got = war.debug_gemm(A, W[:F], SWIGLU, shape, W2=W[F:]).double()
    a, wg, wu = A.double(), W[:F].double(), W[F:].double()
    g, u, gam = a @ wg.t(), a @ wu.t(), K * 2.0 ** -24
    dg, du = gam * (a.abs() @ wg.abs().t()), gam * (a.abs() @ wu.abs().t())
    silu = g * torch.sigmoid(g)
    ref = silu * u
    bound = ref.abs() * (2.0 ** -8 + 2.0 ** -20) + 1.1 * dg * u.abs() + silu.abs() * du + 1.1 * dg * du + 2.0 ** -126
    assert ((got - ref).abs() <= bound).all(), (tuple(A.shape), tuple(W.shape), shape)


@pytest.mark.parametrize("shape", range(6))
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 7])
def test_tiled_kernels(shape, steps):
    from paper_2607_17299_amd import war
    bm, bn = TILES[shape]
    K = 64 * steps
    # (17 groups of 128: eight n-blocks share their XCDs and one is left; 3: none do)
    for M, N in [(1, 128), (81, 384), (bm - 1, 384), (bm, 256), (bm + 1, 640), (2 * bm + 5, 17 * 128)]:
        A, W = _operands(M, N, K, shape * 100 + steps)
        for splits in {1, 2, min(3, steps)}:
            kper = -(-steps // splits) * 64
            if (splits - 1) * kper < K:
                _check_partial(war, A, W, shape, splits, kper)
        _check_argmax(war, A, W, shape)
        if shape != 3 and N % 256 == 0:
            _check_swiglu(war, A, W, shape)
    if shape != 3:
        A, W = _operands(bm + 3, 768, K, 7)
        _check_swiglu(war, A, W, shape)
    rows = torch.arange(bm + 9, 0, -2, dtype=torch.int32, device=DEV)      # gathered rows, fewer than A has
    A, W = _operands(bm + 10, 384, K, 8)
    _check_argmax(war, A, W, shape, rows)


def test_long_tiled_sums():
    """All of a large K in one split: the longest chains of fp32 sums."""
    from paper_2607_17299_amd import war
    for shape in range(6):
        A, W = _operands(TILES[shape][0], 256, 12288, shape)
        _check_partial(war, A, W, shape, 1, 12288)


@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 48, 49, 64, 65, 80, 96])
def test_few_row_kernels(M):
    """Each unrolled count of k-steps and the runtime loop (3, 7, uneven splits)."""
    from paper_2607_17299_amd import war
    for steps in (1, 2, 3, 4, 7, 8, 12, 16, 24, 32, 48, 64):
        A, W = _operands(M, 256, 128 * steps, M + steps)
        if M <= 80:
            _check_partial(war, A, W, -1, 2, 64 * steps)
            if steps > 1:
                _check_partial(war, A, W, -1, 2, 64 * (steps + 1))
        A, W = A[:, :64 * steps].contiguous(), W[:, :64 * steps].contiguous()
        _check_argmax(war, A, W, -1)
        if M <= 80:
            _check_swiglu(war, A, W, -1)


def test_debug_gemm_refuses_what_does_not_fit():
    from paper_2607_17299_amd import war
    A, W = _operands(81, 256, 128, 1)
    for kw in [dict(epi=PARTIAL, shape=-1), dict(epi=PARTIAL, shape=6), dict(epi=PARTIAL, shape=0, splits=3, kper=64),
               dict(epi=PARTIAL, shape=0, splits=1, kper=64), dict(epi=ARGMAX, shape=0, splits=2, kper=64)]:
        with pytest.raises(war.WarError):
            war.debug_gemm(A, W, **kw)
    with pytest.raises(war.WarError):
        war.debug_gemm(A, W, SWIGLU, 3, W2=W)
