"""Dispatch rules on the CPU: which kernel and tile a layer's sizes pick."""
import pytest

import rules

WIDE = (65536, 65568, 98304, 128256, 131072, 151936, 262144)


@pytest.mark.parametrize("n", (256, 4096, 11008) + WIDE)
def test_weight_only_decode_streams_its_weights_at_every_width(n):
    """Up to 32 tokens the weight-only layer is its weight stream, a vocabulary head of any width included."""
    for k in (128, 2048, 4096, 11008, 32768):
        for m in range(1, 33):
            assert rules.w4_tile(m, n, k) >= 0, (m, n, k)


def test_weight_only_prefill_takes_the_tiled_kernel():
    for m, n, k in ((33, 131072, 4096), (2048, 4096, 4096), (2048, 12288, 4096), (8192, 4096, 11008), (512, 12288, 4096)):
        assert rules.w4_tile(m, n, k) == -1, (m, n, k)


# microseconds measured with cold weights: the tiled kernel's 128-token tiles, the streaming kernel with its tile
MEASURED = [(384, 12288, 128, 7.0, 16.3), (200, 24576, 128, 7.3, 16.8), (100, 49152, 128, 7.4, 16.2), (64, 65536, 128, 7.3, 14.5),
            (384, 12288, 384, 10.8, 20.3), (256, 24576, 256, 10.2, 18.3), (33, 65536, 384, 11.3, 16.8), (512, 8192, 512, 12.3, 15.4),
            (128, 32768, 768, 16.4, 19.5), (128, 4096, 4096, 55.0, 10.0), (400, 4096, 4096, 55.5, 24.1),
            (256, 4096, 11008, 119.0, 34.1), (200, 12288, 4096, 56.7, 41.3)]


@pytest.mark.parametrize("m,n,k,tiled,streaming", MEASURED)
def test_weight_only_mid_batch_takes_the_kernel_that_measured_faster(m, n, k, tiled, streaming):
    """A wide layer with a short K is one round of the tiled kernel and several of the streaming one's."""
    assert (rules.w4_tile(m, n, k) >= 0) == (streaming < tiled)
