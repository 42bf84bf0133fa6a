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
