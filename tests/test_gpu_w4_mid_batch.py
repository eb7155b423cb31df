"""GPU parity of the weight-streaming INT4 kernel on batches of more than eight tokens: each of its tiles (channels x
tokens) at its ragged edges - a last token block of one row, an odd number of 32-channel blocks, fewer K units than
wavefronts - on operands whose every partial sum is exactly representable, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_w4a16 import _exact_case, _forward, _pack, w4  # noqa: F401

pytestmark = pytest.mark.gpu


# the sizes reach, in this order, the tiles 32 channels x 16, 32 and 64 tokens, 64 channels x 32, 64 and 128 tokens
@pytest.mark.parametrize("m,n,k", [(9, 288, 128), (17, 4096, 384), (33, 4096, 256), (45, 4128, 128), (64, 4096, 128),
                                   (65, 4096, 640), (100, 4096, 128), (32, 12288, 128), (31, 11040, 256), (45, 11040, 128),
                                   (64, 11008, 256), (100, 11040, 128), (128, 11008, 384), (257, 4096, 256)])
def test_mid_batch_exact_operands(w4, m, n, k):  # noqa: F811
    print(f"w4a16 mid batch {m} x {n} x {k}", flush=True)
    x16, codes, scales, zeros = _exact_case(700 + m + n + k, m, n, k)
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
