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
