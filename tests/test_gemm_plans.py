"""Which kernel a projection takes, on the CPU.  The lists hold shapes on which both kernels were
timed; the times are us."""
import random

import pytest

from tests.plans import (EPI_QKV, EPI_RESID, EPI_STORE_F32, EPI_SWIGLU, f32_small, padk, stream_plan, tile_plan)


@pytest.mark.parametrize("epi,M,N,K", [
    (EPI_STORE_F32, 161, 32000, 4096),   # tiles 65.4, streamed 85.1: two passes for one
    (EPI_STORE_F32, 192, 32000, 4096),   # 71.6, 89.4
    (EPI_STORE_F32, 192, 128256, 2048),  # tiles four passes, streamed six
    (EPI_STORE_F32, 64, 32000, 512),     # 13.3, 13.9
    (EPI_STORE_F32, 96, 32000, 1024),    # 18.9, 21.5
    (EPI_STORE_F32, 160, 32000, 2048),   # 31.9, 34.6
    (EPI_STORE_F32, 128, 32000, 4096),   # weights displaced from the caches: 92.5, 95.0
    (EPI_STORE_F32, 16, 24576, 1024),    # 12.6, 13.4
    (EPI_STORE_F32, 128, 8192, 4096),    # 35.7, 39.5
    (EPI_SWIGLU, 161, 27648, 5120),      # 84.1, 103.3
    (EPI_SWIGLU, 192, 57344, 8192),      # 253.9, 288.3
    (EPI_RESID, 192, 8192, 28672),       # 126.9, 145.0
    (EPI_RESID, 192, 3072, 3072),        # 21.6, 23.0
    (EPI_RESID, 96, 8192, 8192),         # 42.0, 46.9
    (EPI_RESID, 160, 5120, 13824),       # 51.0, 53.6
    (EPI_SWIGLU, 160, 27648, 512),       # 16.6, 20.3
    (EPI_SWIGLU, 160, 22016, 512),       # 15.4, 17.5
    (EPI_QKV, 1, 768, 256),              # 6.3, 6.9
    (EPI_RESID, 16, 1024, 1024),         # a layer 37.9, 38.6
    (EPI_RESID, 192, 5120, 13824),       # 53.7, 56.5
])
def test_tiles_where_streaming_is_slower(epi, M, N, K):
    assert stream_plan(epi, M, N, K) is None


@pytest.mark.parametrize("epi,M,N,K,plan", [
    (EPI_SWIGLU, 16, 22016, 4096, (1, 3, 1)),    # tiles 36.0, streamed 34.0
    (EPI_SWIGLU, 64, 22016, 4096, (2, 3, 1)),    # 48.0, 38.1
    (EPI_SWIGLU, 135, 22016, 4096, (5, 3, 1)),   # 60.3, 55.2
    (EPI_QKV, 160, 12288, 4096, (5, 3, 2)),      # 43.8, 41.8
    (EPI_RESID, 160, 4096, 4096, (5, 2, 4)),     # 26.8, 25.1
    (EPI_RESID, 96, 8192, 28672, (3, 4, 4)),     # 97.8, 91.7
    (EPI_SWIGLU, 192, 5632, 1024, (6, 1, 1)),    # 24.9, 11.8
    (EPI_SWIGLU, 192, 11008, 2048, (6, 2, 1)),   # 30.4, 26.2
    (EPI_QKV, 192, 6144, 2048, (6, 3, 4)),       # 29.3, 26.6
    (EPI_QKV, 192, 24576, 8192, (6, 3, 1)),      # 123.5, 117.4
    (EPI_SWIGLU, 192, 22016, 4096, (6, 3, 1)),   # a layer 179.5, 177.5
    (EPI_RESID, 192, 6144, 16384, (6, 3, 4)),    # 70.1, 66.8
    (EPI_STORE_F32, 33, 4096, 1024, (2, 1, 1)),  # 11.2, 7.5
    (EPI_STORE_F32, 96, 22016, 5120, (3, 3, 1)),  # 83.2, 80.1
    (EPI_STORE_F32, 64, 22016, 1024, (2, 3, 1)),  # with norm and argmax 28.2, 26.2
    (EPI_STORE_F32, 64, 32000, 4096, (2, 4, 1)),  # with norm and argmax 61.7, 60.8
])
def test_streamed_where_it_is_faster(epi, M, N, K, plan):
    assert stream_plan(epi, M, N, K) == plan


def test_streamed_sums_fit_where_the_tiles_sums_fit():
    """A plan splits K no further than the tiles would, and every split has the k steps that the
    kernel asks for."""
    rng = random.Random(7)
    for _ in range(4000):
        epi, M = rng.choice([EPI_STORE_F32, EPI_RESID, EPI_SWIGLU, EPI_QKV]), rng.randint(1, 192)
        N, K = 16 * rng.randint(1, 3000), 32 * rng.randint(1, 400)
        p = stream_plan(epi, M, N, K)
        if p is None:
            continue
        fm, cb, S = p
        assert fm == (M + 31) // 32 and 1 <= cb <= (4 if fm < 6 else 3)
        assert S <= tile_plan(M, N, K).splits
        assert padk(K) // 64 // S >= (40 // (fm + cb) if fm > 5 else 1)
    assert stream_plan(EPI_RESID, 193, 4096, 4096) is None


@pytest.mark.parametrize("M,N,K,small", [
    (34, 768, 256, True),       # tiles of 96 x 128 27.8, of 16 x 32 6.6
    (34, 256, 688, True),       # 23.7, 7.6
    (200, 1376, 256, True),     # 26.0, 7.8
    (3, 512, 256, True),        # 11.2, 7.0
    (16, 12288, 4096, True),    # 56.9, 51.5
    (32, 4096, 4096, True),     # 43.4, 28.2
    (128, 4096, 1024, True),    # 33.8, 28.3
    (512, 1024, 2048, True),    # 49.2, 40.0
    (512, 1024, 2816, True),    # 65.9, 51.9
    (17, 12288, 4096, False),   # 49.0, 64.9
    (32, 16384, 4096, False),   # 54.3, 82.0
    (32, 16384, 512, False),    # 16.2, 19.3
    (24, 6144, 1024, False),    # 15.0, 18.5
    (16, 9984, 4096, False),    # 37.3, 42.8
    (80, 6144, 4096, False),    # 66.0, 84.5
    (144, 3072, 8192, False),   # 121.6, 160.6
    (400, 1024, 8192, False),   # 120.8, 146.9
    (64, 8192, 8192, False),    # 118.2, 149.9
])
def test_small_fp32_tiles_where_they_are_faster(M, N, K, small):
    assert f32_small(M, N, K) is small
