"""GPU parity of the kernel that splits K over a workgroup's wavefronts (few tokens or few tiles), against the oracle,
bit for bit: every tile it has at its edges (rows, channels, K remainders of 128 and of 64 bytes, fewer K units
than wavefronts, K of several rounds of the ring), every epilogue, padded pitches and an output that does not admit
vector stores."""
import numpy as np
import pytest
import torch

import paper_2505_20932_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# tile 1: m <= 16; tile 2: m <= 32 with few tiles; tile 4: 64 x 64 tiles (long K, one round of them); else 32 x 32
SHAPES = [(1, 1, 16), (1, 17, 48), (16, 33, 64), (15, 50, 112), (7, 16, 144), (16, 100, 640), (3, 31, 1008), (16, 64, 4096),
          (17, 31, 16), (32, 33, 128), (31, 100, 784), (20, 4096, 256), (33, 32, 96), (50, 65, 192), (65, 130, 656),
          (197, 96, 384), (197, 161, 768), (129, 4090, 1040), (255, 2049, 1024)]
# per tile: a wavefront's share of K is several rounds of its ring (4, 3, 2 and 2 units of 128 bytes), with nothing, one or two
# 64-byte steps behind the last whole unit; 80 and 2064 channels run the code-table epilogue
MAIN_LOOP = [(16, 80, 4096), (9, 50, 4240), (13, 33, 4208), (20, 65, 4240), (31, 80, 4096), (17, 33, 3184), (65, 66, 3152),
             (197, 96, 3136), (197, 80, 3072), (129, 4090, 2064), (255, 2064, 3184), (200, 4096, 2048)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def padded(a, pad):
    """The matrix with `pad` extra columns of garbage behind every row."""
    full = np.full((a.shape[0], a.shape[1] + pad), 77, dtype=a.dtype)
    full[:, :a.shape[1]] = a
    return dev(full)[:, :a.shape[1]]


@pytest.mark.parametrize("m,n,k", SHAPES + MAIN_LOOP)
def test_small_problem_bit_exact(orc, m, n, k):
    print(f"small problem {m} x {n} x {k}", flush=True)
    rng = np.random.default_rng(m * 7919 + n * 31 + k)
    xq = rng.integers(-128, 128, (m, k), dtype=np.int8)
    wq = rng.integers(-127, 128, (n, k), dtype=np.int8)
    acc = orc.gemm_i8(xq, wq)
    mult = (np.abs(rng.standard_normal(n)) * 3e-4 + 1e-5).astype(np.float32)
    off = rng.integers(-5000, 5000, n).astype(np.int32)
    fb = rng.standard_normal(n).astype(np.float32)
    sxr = (np.abs(rng.standard_normal(m)) * 0.5 + 0.5).astype(np.float32)
    zr = int(rng.integers(-20, 20))
    qp, qpt = P.make_qparams(z_r=zr), P.make_qparams(P.CWAC_EPI_FP_BIAS, True, 1.0, 0, 1.0, zr)
    m0 = rng.integers(1 << 30, (1 << 31) - 1, n).astype(np.int32)
    shift = rng.integers(38, 46, n).astype(np.int32)
    table = rng.permutation(np.arange(-128, 128)).astype(np.int8)
    code = orc.folded_forward(acc, off, mult, zr)
    for pad, ldo in ((0, n), (48, n + 8), (16, n + 3)):
        x, w = padded(xq, pad), padded(wq, pad)

        def run(dt, call):
            full = torch.full((m, ldo), 55, dtype=dt, device=DEV)
            call(full[:, :n])
            torch.cuda.synchronize()
            got = full.cpu().numpy()
            assert np.all(got[:, n:] == 55), "wrote outside the output columns"
            return got[:, :n]

        def fwd(kind, dt, q, *vec):
            v = [None if a is None else dev(a) for a in vec]
            return run(dt, lambda o: P.qlinear_cwac_forward(x, w, q, *v, kind, o))

        eq = np.testing.assert_array_equal
        eq(fwd(P.CWAC_OUT_INT32, torch.int32, None, None, off, None, None), acc + off[None, :])
        eq(fwd(P.CWAC_OUT_INT8, torch.int8, qp, mult, off, None, None), code)
        eq(fwd(P.CWAC_OUT_INT8, torch.int8, qpt, mult, off, fb, sxr), orc.folded_forward(acc, off, mult, zr, fb, sxr))
        _, want = orc.folded_forward(acc, off, mult, 0, fb, sxr, want_f32=True)
        eq(fwd(P.CWAC_OUT_FP32, torch.float32, None, mult, off, fb, sxr), want)
        eq(run(torch.int8, lambda o: P.qlinear_cwac_forward_fixed_point(x, w, qp, dev(m0), dev(shift), dev(off), o)),
           orc.fixed_point_forward(acc, off, m0, shift, zr))
        if n % 16 == 0 and ldo % 16 == 0:
            eq(run(torch.int8, lambda o: P.qlinear_cwac_forward_table(x, w, qp, dev(mult), dev(off), dev(table), o)),
               table[code.astype(np.int32) + 128])


@pytest.mark.parametrize("m,n,k", [(300, 272, 192), (257, 3000, 144), (1000, 65, 640)])
def test_forced_on_larger_layers_and_pointwise_convolutions(orc, m, n, k):
    """cwac_tuning.kernel = CWAC_KERNEL_SPLIT_K beyond the kernel's own rule: 32 x 32 tiles, the same codes."""
    print(f"forced split-K {m} x {n} x {k}", flush=True)
    rng = np.random.default_rng(m + n + k)
    xq = rng.integers(-128, 128, (m, k), dtype=np.int8)
    wq = rng.integers(-127, 128, (n, k), dtype=np.int8)
    mult = (np.abs(rng.standard_normal(n)) * 3e-4 + 1e-5).astype(np.float32)
    off = rng.integers(-5000, 5000, n).astype(np.int32)
    want = orc.folded_forward(orc.gemm_i8(xq, wq), off, mult, 5)
    tun, out = P.make_tuning(kernel=P.binding.CWAC_KERNEL_SPLIT_K), torch.zeros(m, n, dtype=torch.int8, device=DEV)
    P.qlinear_cwac_forward(dev(xq), dev(wq), P.make_qparams(z_r=5), dev(mult), dev(off), None, None, P.CWAC_OUT_INT8, out, tuning=tun)
    np.testing.assert_array_equal(out.cpu().numpy(), want)
    out.zero_()
    P.qconv2d_cwac_forward(dev(xq).view(1, 1, m, k), dev(wq).view(n, 1, 1, k), 1, 0, P.make_qparams(z_r=5), dev(mult), dev(off),
                           None, P.CWAC_OUT_INT8, out, tuning=tun)
    np.testing.assert_array_equal(out.cpu().numpy(), want)
    # a filter with taps has no split-K form: the automatic choice runs
    w4 = rng.integers(-127, 128, (n, 1, 3, 16), dtype=np.int8)
    x4 = rng.integers(-128, 128, (1, 5, 40, 16), dtype=np.int8)
    acc = orc.conv2d_i8(x4, w4, 1, 0, 0)
    o4 = torch.zeros(acc.shape[0], n, dtype=torch.int8, device=DEV)
    P.qconv2d_cwac_forward(dev(x4), dev(w4), 1, 0, P.make_qparams(z_r=5), dev(mult), dev(off), None, P.CWAC_OUT_INT8, o4, tuning=tun)
    np.testing.assert_array_equal(o4.cpu().numpy(), orc.folded_forward(acc, off, mult, 5))
