"""GPU parity of the weight-only INT4 layer on few tokens of layers wider than 65536 channels (a vocabulary head): the
weight-streaming kernel by the library's choice and with its wavefronts and ring depth forced, on operands whose every
partial sum is exactly representable, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_w4a16 import _exact_case, _forward, _pack, w4  # noqa: F401

pytestmark = pytest.mark.gpu


# every token count of the streaming tiles at its edge; 65568 and 131104 channels are an odd number of 32-channel blocks
@pytest.mark.parametrize("m,n,k", [(1, 65568, 128), (8, 131104, 256), (9, 65568, 384), (16, 65792, 128), (17, 65568, 256),
                                   (32, 131072, 128)])
def test_wide_layer_exact_operands(w4, m, n, k):  # noqa: F811
    print(f"w4a16 wide layer {m} x {n} x {k}", flush=True)
    x16, codes, scales, zeros = _exact_case(400 + m + n + k, m, n, k)
    acc, _ = w4.product(x16, w4.dequant(codes, scales, zeros))
    acc32 = acc.astype(np.float32)
    assert np.array_equal(acc32.astype(np.float64), acc)
    pw, psz = _pack(codes, scales, zeros)
    rng = np.random.default_rng(9)
    mult = (1 + 0.25 * rng.standard_normal(n)).astype(np.float32)
    fbias = rng.standard_normal(n).astype(np.float32)
    _, o16 = w4.epilogue_f32(acc32, mult, fbias)
    for waves, depth in ((0, 0), (4, 0), (8, 3)):
        np.testing.assert_array_equal(_forward(x16, pw, psz, n, None, None, torch.float32, waves=waves, depth=depth).cpu().numpy(),
                                      acc32)
        outh = _forward(x16, pw, psz, n, mult, fbias, torch.float16, ldo=n + 24, waves=waves, depth=depth)
        np.testing.assert_array_equal(outh.cpu().numpy().view(np.uint16), o16.view(np.uint16))
