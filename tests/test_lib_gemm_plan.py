"""Host-side rules of the bf16 GEMM's plan (no GPU needed)."""
import itertools

import pytest

from paper_2605_30859_amd import binding as B


@pytest.fixture(scope="module", autouse=True)
def _lib():
    B.load_library()


def test_large_tiles_stay_within_32_bit_offsets():
    """The persistent large-tile kernel addresses 256 rows of A, W and C by 32-bit
    byte offsets: no plan may give it rows that reach 2 GiB, whether they are
    the operands' (K), the result's or a split's fp32 partial sums."""
    edges = [2 ** p + d for p in (20, 21, 22) for d in (-768, -256, 0, 256)]
    ns = [1024, 4096, 24576] + edges + [2 ** 22 + 2 ** 19, 2 ** 23, 2 ** 24]
    ks = [256, 2048, 4096] + edges + [2 ** 22 + 2048, 2 ** 23, 2 ** 24]
    taken = 0
    for m, n, k, epi in itertools.product((129, 256, 257, 512, 4096, 16384), ns, ks, range(4)):
        kind, _, _, split, alt, _ = B.darts_debug_gemm_plan(m, n, k, epi)
        if not alt:
            continue
        taken += 1
        ldc, size = (n, 4) if split > 1 or epi in (0, 2) else (n // 2, 2) if epi == 3 else (n, 2)
        assert 256 * max(2 * k, size * ldc) < 2 ** 31, (m, n, k, epi, kind, split)
    assert taken > 200


@pytest.mark.parametrize("m,n,k,epi", [(389, 24576, 4096, 3), (16384, 24576, 4096, 3), (4096, 6144, 4096, 0),
                                       (2048, 4096, 12288, 2), (512, 151936, 4096, 0), (4096, 2 ** 21 - 256, 1024, 0)])
def test_large_tiles_run_ordinary_shapes(m, n, k, epi):
    """The projections of the supported decoders, and the widest rows in reach."""
    assert B.darts_debug_gemm_plan(m, n, k, epi)[4] == 1


@pytest.mark.parametrize("m,n,k,nt", [(45, 24576, 4096, 0), (45, 4096, 12288, 0), (9, 32768, 4096, 0), (9, 36864, 4096, 1),
                                      (16, 151936, 4096, 1), (48, 151936, 2048, 1), (49, 151936, 2048, 0),
                                      (128, 24576, 8192, 1), (129, 24576, 8192, 0)])
def test_weights_that_a_cache_may_hold_are_loaded_normally(m, n, k, nt):
    """A stateless call may be repeated with the same weights: only those that the
    256 MiB Infinity Cache cannot keep are loaded non-temporal, and only for
    batches where that was measured to gain."""
    assert B.darts_debug_gemm_plan(m, n, k, 0)[5] == nt


@pytest.mark.parametrize("m,n,k,epi,alt", [(160, 12288, 5120, 0, 0), (280, 6144, 4096, 0, 0), (160, 5120, 12288, 2, 0),
                                           (140, 24576, 4096, 3, 0), (160, 18432, 4096, 0, 1), (300, 4096, 12288, 2, 1),
                                           (400, 4096, 12288, 2, 1), (640, 8192, 8192, 0, 1)])
def test_splits_that_stream_weights_keep_the_ring(m, n, k, epi, alt):
    """Split plans alternate only where that was measured to be no slower."""
    kind, _, _, split, got, _ = B.darts_debug_gemm_plan(m, n, k, epi)
    assert 3 <= kind <= 5 and split > 1 and got == alt


@pytest.mark.parametrize("m,n,k,epi,alt", [(256, 151936, 1024, 0, 0), (2048, 20480, 512, 0, 0), (3000, 16384, 256, 0, 0), (3000, 1536, 1024, 0, 1),
                                           (256, 151936, 2048, 0, 0), (400, 151936, 2048, 0, 1), (256, 151936, 4096, 0, 1),
                                           (2048, 32768, 256, 1, 1), (1024, 8192, 512, 2, 1)])
def test_short_k_with_fp32_results_keeps_the_ring(m, n, k, epi, alt):
    """Plain fp32 results of a short K are bound by their stores."""
    kind, _, _, split, got, _ = B.darts_debug_gemm_plan(m, n, k, epi)
    assert 3 <= kind <= 5 and split == 1 and got == alt
