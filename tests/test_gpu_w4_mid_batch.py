"""GPU parity of the weight-only INT4 kernels: each tile of the streaming one (channels x tokens) at its ragged edges - a last token
block of one row, an odd number of 32-channel blocks, fewer K units than wavefronts - and with K of several rounds of
its ring - and the tiled one's cut last round, on operands whose every partial sum is exactly representable, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_w4a16 import _exact_case, _forward, _pack, w4  # noqa: F401

pytestmark = pytest.mark.gpu


# short K: the tiles' edges
SHORT = [(9, 288, 128), (17, 4096, 384), (33, 4096, 256), (45, 4128, 128), (64, 4096, 128),
         (65, 4096, 640), (100, 4096, 128), (32, 12288, 128), (31, 11040, 256), (45, 11040, 128),
         (64, 11008, 256), (100, 11040, 128), (128, 11008, 384), (257, 4096, 256)]
# per tile: a wavefront's share of K is more units of 64 channels than its ring has slots, by at least one round of the ring
# (two where the tile is for a K of up to 1024), with shares of unequal length
MAIN_LOOP = [(5, 288, 4224), (13, 288, 4224), (16, 4096, 3200), (33, 4096, 2176), (31, 11040, 2176), (65, 4096, 2176),
             (45, 11040, 1152), (64, 11008, 1408), (128, 11008, 1152), (257, 4096, 1408), (5, 8224, 896), (8, 8224, 1024),
             (13, 8224, 896), (16, 8256, 1024)]


# tiles of 16 channels (up to 16 tokens): one and both row counts' edges, fewer groups than wavefronts, shares of unequal
# length over several rounds of the ring, the last 16 channels of a 32-channel block
TILES16 = [(1, 256, 128), (8, 288, 896), (9, 288, 1152), (16, 320, 3200), (3, 4096, 2176), (16, 4096, 1408), (7, 8224, 256),
           (1, 12288, 384), (8, 4128, 4096)]
# the 32-channel tiles of those token counts where the 16-channel ones do not take the layer
WIDE_MAIN_LOOP = [(5, 12320, 4224), (13, 4128, 4224), (8, 12320, 1024)]


# the tiled kernel's last round in quarters and in halves of a tile: a last tile of 20, 85 and 120 rows, whose later pieces are
# empty or partial, and one of 10 rows; a last tile of channels that overlaps its neighbour; 8, 64, 85 and 96 tiles in the round
QUARTERS = [(1300, 11808, 128), (1365, 11808, 256), (2500, 8192, 256)]
HALVES = [(1290, 15392, 128), (2040, 11008, 256)]


@pytest.mark.parametrize("m,n,k", SHORT + MAIN_LOOP + TILES16 + WIDE_MAIN_LOOP + QUARTERS + HALVES)
def test_mid_batch_exact_operands(w4, m, n, k):  # noqa: F811
    print(f"w4a16 mid batch {m} x {n} x {k}", flush=True)
    x16, codes, scales, zeros = _exact_case(700 + m + n + k, m, n, k)
    if k > 2048:
        scales[:] = np.float16(0.5)
    acc, _ = w4.product(x16, w4.dequant(codes, scales, zeros))
    acc32 = acc.astype(np.float32)
    assert np.array_equal(acc32.astype(np.float64), acc)
    pw, psz = _pack(codes, scales, zeros)
    rng = np.random.default_rng(8)
    mult = (1 + 0.25 * rng.standard_normal(n)).astype(np.float32)
    fbias = rng.standard_normal(n).astype(np.float32)
    o32, o16 = w4.epilogue_f32(acc32, mult, fbias)
    np.testing.assert_array_equal(_forward(x16, pw, psz, n, None, None, torch.float32).cpu().numpy(), acc32)
    np.testing.assert_array_equal(_forward(x16, pw, psz, n, mult, fbias, torch.float32, ldo=n + 12).cpu().numpy(), o32)
    outh = _forward(x16, pw, psz, n, mult, fbias, torch.float16, ldo=n + 24)
    np.testing.assert_array_equal(outh.cpu().numpy().view(np.uint16), o16.view(np.uint16))
