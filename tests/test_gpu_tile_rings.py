"""GPU parity of the direct-to-LDS kernel's 128-token tiles with 128-byte K steps (two and three stages, one and several
rounds of the ring, ragged edges), of their code-table epilogue and of their implicit-GEMM form, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2505_20932_amd as P
from tuning import tuning_of

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# 128 x 128: K < 1536 two stages, else three; 128 x 256: K >= 3072 three stages of 128 bytes; K % 128 == 64: 64-byte steps
@pytest.mark.parametrize("m,n,k,pipe", [(256, 256, 128, "q"), (300, 272, 256, "q"), (257, 400, 1408, "q"), (256, 256, 1536, "q"),
                                        (385, 272, 1664, "q"), (300, 304, 1792, "q"), (300, 272, 192, "q"), (300, 272, 3072, "duo"),
                                        (257, 528, 3200, "duo"), (384, 256, 3328, "duo"), (300, 272, 2944, "duo")])
def test_ring_bit_exact(orc, m, n, k, pipe):
    print(f"ring {m} x {n} x {k} {pipe}", flush=True)
    rng = np.random.default_rng(m + 7 * n + 13 * k)
    xq = rng.integers(-128, 128, (m, k), dtype=np.int8)
    wq = rng.integers(-127, 128, (n, k), dtype=np.int8)
    acc = orc.gemm_i8(xq, wq)
    mult = (np.abs(rng.standard_normal(n)) * 3e-4 + 1e-5).astype(np.float32)
    off = rng.integers(-5000, 5000, n).astype(np.int32)
    fb = rng.standard_normal(n).astype(np.float32)
    sxr = (np.abs(rng.standard_normal(m)) * 0.5 + 0.5).astype(np.float32)
    table = rng.permutation(np.arange(-128, 128)).astype(np.int8)
    tun = tuning_of("fast", pipe=pipe)
    for zr in (4, -7):
        code = orc.folded_forward(acc, off, mult, zr)
        qp, qpt = P.make_qparams(z_r=zr), P.make_qparams(P.CWAC_EPI_FP_BIAS, True, 1.0, 0, 1.0, zr)
        o8 = torch.empty(m, n, dtype=torch.int8, device=DEV)
        P.qlinear_cwac_forward(dev(xq), dev(wq), qp, dev(mult), dev(off), None, None, P.CWAC_OUT_INT8, o8, tuning=tun)
        np.testing.assert_array_equal(o8.cpu().numpy(), code)
        P.qlinear_cwac_forward(dev(xq), dev(wq), qpt, dev(mult), dev(off), dev(fb), dev(sxr), P.CWAC_OUT_INT8, o8, tuning=tun)
        np.testing.assert_array_equal(o8.cpu().numpy(), orc.folded_forward(acc, off, mult, zr, fb, sxr))
        P.qlinear_cwac_forward_table(dev(xq), dev(wq), qp, dev(mult), dev(off), dev(table), o8, tuning=tun)
        np.testing.assert_array_equal(o8.cpu().numpy(), table[code.astype(np.int32) + 128])
    o32 = torch.empty(m, n, dtype=torch.float32, device=DEV)
    P.qlinear_cwac_forward(dev(xq), dev(wq), None, dev(mult), dev(off), dev(fb), dev(sxr), P.CWAC_OUT_FP32, o32, tuning=tun)
    np.testing.assert_array_equal(o32.cpu().numpy(), orc.folded_forward(acc, off, mult, 0, fb, sxr, want_f32=True)[1])


# convolutions of few 128 x 128 tiles and a long K by the library's own choice, and beside its bounds (K, c_in % 128, rows)
@pytest.mark.parametrize("shape", [(2, 14, 13, 256, 256, 3, 3, 1, 1), (7, 7, 7, 512, 272, 3, 3, 1, 1), (2, 12, 11, 128, 256, 3, 4, 1, 1),
                                   (3, 10, 10, 192, 256, 3, 3, 1, 1), (1, 14, 14, 256, 256, 3, 3, 1, 1), (2, 14, 13, 128, 256, 3, 3, 1, 1)])
@pytest.mark.parametrize("kind", ["int8", "fp32", "int32"])
def test_conv_of_few_tiles_bit_exact(orc, shape, kind):
    b, h, w, c, n, kh, kw, stride, pad = shape
    print(f"conv of few tiles {shape} {kind}", flush=True)
    rng = np.random.default_rng(sum(shape))
    xq = rng.integers(-128, 128, (b, h, w, c), dtype=np.int8)
    wq = rng.integers(-127, 128, (n, kh, kw, c), dtype=np.int8)
    acc = orc.conv2d_i8(xq, wq, stride, pad, -3)
    mult = (np.abs(rng.standard_normal(n)) * 3e-4 + 1e-5).astype(np.float32)
    off = rng.integers(-5000, 5000, n).astype(np.int32)
    fb = rng.standard_normal(n).astype(np.float32)
    qp = P.make_qparams(z_x=-3, z_r=5)
    if kind == "int8":
        out = torch.empty(acc.shape[0], n, dtype=torch.int8, device=DEV)
        P.qconv2d_cwac_forward(dev(xq), dev(wq), stride, pad, qp, dev(mult), dev(off), None, P.CWAC_OUT_INT8, out)
        np.testing.assert_array_equal(out.cpu().numpy(), orc.folded_forward(acc, off, mult, 5))
    elif kind == "fp32":
        out = torch.empty(acc.shape[0], n, dtype=torch.float32, device=DEV)
        P.qconv2d_cwac_forward(dev(xq), dev(wq), stride, pad, qp, dev(mult), dev(off), dev(fb), P.CWAC_OUT_FP32, out)
        np.testing.assert_array_equal(out.cpu().numpy(), orc.folded_forward(acc, off, mult, 0, fb, None, want_f32=True)[1])
    else:
        out = torch.empty(acc.shape[0], n, dtype=torch.int32, device=DEV)
        P.qconv2d_cwac_forward(dev(xq), dev(wq), stride, pad, qp, None, dev(off), None, P.CWAC_OUT_INT32, out)
        np.testing.assert_array_equal(out.cpu().numpy(), acc + off)


@pytest.mark.parametrize("shape", [(2, 14, 13, 128, 256, 3, 3, 1, 1), (5, 8, 9, 256, 272, 3, 3, 1, 1), (3, 17, 17, 128, 256, 2, 2, 2, 0)])
def test_conv_ring_bit_exact(orc, shape):
    b, h, w, c, n, kh, kw, stride, pad = shape
    print(f"conv ring {shape}", flush=True)
    rng = np.random.default_rng(sum(shape))
    xq = rng.integers(-128, 128, (b, h, w, c), dtype=np.int8)
    wq = rng.integers(-127, 128, (n, kh, kw, c), dtype=np.int8)
    acc = orc.conv2d_i8(xq, wq, stride, pad, 9)
    mult = (np.abs(rng.standard_normal(n)) * 3e-4 + 1e-5).astype(np.float32)
    off = rng.integers(-5000, 5000, n).astype(np.int32)
    out = torch.empty(acc.shape[0], n, dtype=torch.int8, device=DEV)
    P.qconv2d_cwac_forward(dev(xq), dev(wq), stride, pad, P.make_qparams(z_x=9, z_r=3), dev(mult), dev(off), None,
                           P.CWAC_OUT_INT8, out, tuning=tuning_of("fast", pipe="q"))
    np.testing.assert_array_equal(out.cpu().numpy(), orc.folded_forward(acc, off, mult, 3))


# layers whose plain forward takes a register-staged tile: the code table in the split-K kernel (four rounds of 32 x 32 tiles, for
# some K up to six, or fewer than 128 tokens), in 128 x 128 tiles (beyond; one row of tiles, two that overlap in all rows but one, ragged
# channels, both K steps and ring depths), and as a pass of its own (K no multiple of 64)
@pytest.mark.parametrize("m,n,k", [(394, 1536, 384), (591, 1536, 384), (700, 1520, 384), (592, 2048, 512), (100, 11008, 48), (700, 1520, 400),
                                   (128, 8208, 128), (129, 6672, 192), (255, 4144, 384), (128, 12288, 1536), (129, 6672, 3072),
                                   (197, 5120, 1280), (131, 5120, 704), (250, 6144, 1280), (224, 6656, 1024)])
def test_code_table_of_layers_between_the_kernels(orc, m, n, k):
    print(f"code table {m} x {n} x {k}", flush=True)
    rng = np.random.default_rng(m + n + k)
    xq = rng.integers(-128, 128, (m, k), dtype=np.int8)
    wq = rng.integers(-127, 128, (n, k), dtype=np.int8)
    mult = (np.abs(rng.standard_normal(n)) * 3e-4 + 1e-5).astype(np.float32)
    off = rng.integers(-5000, 5000, n).astype(np.int32)
    table = rng.permutation(np.arange(-128, 128)).astype(np.int8)
    full = torch.full((m, n + 16), 55, dtype=torch.int8, device=DEV)
    P.qlinear_cwac_forward_table(dev(xq), dev(wq), P.make_qparams(z_r=5), dev(mult), dev(off), dev(table), full[:, :n])
    code = orc.folded_forward(orc.gemm_i8(xq, wq), off, mult, 5)
    np.testing.assert_array_equal(full[:, :n].cpu().numpy(), table[code.astype(np.int32) + 128])
    assert (full[:, n:] == 55).all()
