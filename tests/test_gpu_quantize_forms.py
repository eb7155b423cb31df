"""The quantizers' register-resident and flat forms: every number of vectors per thread, rows that end inside one, layouts
that leave them for the general form, quotients beside the ties, and values and scales at the ends of fp32 - against
Eq. 1 with IEEE division in numpy, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2505_20932_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TINY = np.float32(np.finfo(np.float32).tiny)


def rows_want(x, bits=8):
    qmax = np.float32(2 ** (bits - 1) - 1)
    with np.errstate(all="ignore"):
        s = (np.fmax.reduce(np.abs(x), axis=1, initial=np.float32(0)) / qmax).astype(np.float32)
        s = np.where(s >= TINY * np.float32(256), s, TINY * np.float32(256)).astype(np.float32)
        v = np.rint(x / s[:, None])
        return np.fmin(np.fmax(v, -qmax), qmax).astype(np.int32).astype(np.int8), s


def act_want(x, s, z, bits=8):
    half, levels = 2 ** (bits - 1), np.float32(2 ** bits - 1)
    with np.errstate(all="ignore"):
        v = np.rint(x / np.float32(s)) + np.float32(z + half)
        return (np.fmin(np.fmax(v, np.float32(0)), levels).astype(np.int32) - half).astype(np.int8)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def run_rows(x, bits=8, pad=0):
    m, k = x.shape
    full = torch.full((m, k + pad), 3.0e38, dtype=torch.float32, device=DEV)
    full[:, :k] = dev(x)
    q = torch.full((m + 1, k + pad), 77, dtype=torch.int8, device=DEV)
    s = torch.full((m + 1,), -1.0, dtype=torch.float32, device=DEV)
    P.cwac_quantize_rows_sym_bits(full[:, :k], bits, s[:m], q[:m, :k])
    torch.cuda.synchronize()
    assert (q[m] == 77).all() and (q[:, k:] == 77).all() and s[m] == -1.0
    return q[:m, :k].cpu().numpy(), s[:m].cpu().numpy()


@pytest.mark.parametrize("m,k,pad", [(1, 4, 0), (5, 256, 0), (7, 260, 4), (9, 512, 0), (3, 516, 8), (6, 1024, 0), (2, 1028, 0),
                                     (3, 2048, 0), (2, 2052, 4), (3, 4096, 0), (2, 4100, 0), (3, 8192, 0), (2, 8196, 4), (2, 11008, 0),
                                     (2, 12292, 0), (2, 16384, 0), (2, 16388, 0), (3, 770, 0), (3, 768, 3), (511, 772, 0), (512, 516, 8), (513, 1024, 0)])
def test_row_quantizer_every_form(m, k, pad):
    rng = np.random.default_rng(m + k + pad)
    x = (rng.standard_normal((m, k)) * np.exp(3 * rng.standard_normal((m, 1)))).astype(np.float32)
    for bits in (8, 4):
        q, s = run_rows(x, bits, pad)
        wq, ws = rows_want(x, bits)
        np.testing.assert_array_equal(s, ws)
        np.testing.assert_array_equal(q, wq)


def beside_ties(rng, s, count, top):
    """Values whose quotient by s is a half-integer, or a few units in the last place from one."""
    half = rng.integers(-top, top, count).astype(np.float64) + 0.5
    x = (half * np.float64(s)).astype(np.float32)
    for _ in range(3):
        x = np.where(rng.random(count) < 0.6, np.nextafter(x, np.float32(np.inf) * rng.choice([-1, 1], count).astype(np.float32)), x)
    return x.astype(np.float32)


@pytest.mark.parametrize("exponent", [0, -20, 40, -88, 99, -101, 110, -125])
def test_quotients_beside_the_ties(exponent):
    """Scales over the whole range, inside and outside the one that the short division covers."""
    rng = np.random.default_rng(exponent + 200)
    rows = []
    for _ in range(64):
        amax = np.float32(np.ldexp(1.0 + rng.random(), exponent + 6))
        s = np.float32(max(amax / np.float32(127), TINY * np.float32(256)))
        x = beside_ties(rng, s, 1024, 126)
        x = np.where(np.abs(x) > amax, np.float32(0), x)
        x[int(rng.integers(1024))] = amax
        rows.append(x)
    x = np.stack(rows)
    q, s = run_rows(x)
    wq, ws = rows_want(x)
    np.testing.assert_array_equal(s, ws)
    np.testing.assert_array_equal(q, wq)
    for z in (-128, 5, 127):
        sa = float(ws[z % 64])
        xa = beside_ties(rng, ws[z % 64], 64 * 1024, 300).reshape(64, 1024)
        qa = torch.empty(64, 1024, dtype=torch.int8, device=DEV)
        P.cwac_quantize_act(dev(xa), sa, z, qa)
        np.testing.assert_array_equal(qa.cpu().numpy(), act_want(xa, np.float32(sa), z))


@pytest.mark.parametrize("m,k,pad", [(1, 4, 0), (1, 1028, 0), (300, 900, 0), (1030, 1024, 0), (1031, 1020, 0), (40, 128, 4), (40, 126, 0)])
@pytest.mark.parametrize("s", [0.03, 1e-30, 2e31])
def test_activation_quantizer_forms_and_extreme_values(m, k, pad, s):
    rng = np.random.default_rng(m + k + pad)
    x = (rng.standard_normal((m, k)) * 60 * s).astype(np.float32)
    x.flat[:4] = [np.inf, -np.inf, np.nan, 3.4e38]
    x.flat[-4:] = [-3.4e38, 1e-45, -0.0, np.nan]
    full = torch.full((m, k + pad), 1.0, dtype=torch.float32, device=DEV)
    full[:, :k] = dev(x)
    q = torch.full((m + 1, k + pad), 77, dtype=torch.int8, device=DEV)
    for z, bits in ((7, 8), (-128, 8), (3, 4)):
        P.cwac_quantize_act_bits(full[:, :k], s, z, bits, q[:m, :k])
        torch.cuda.synchronize()
        assert (q[m] == 77).all() and (q[:, k:] == 77).all()
        np.testing.assert_array_equal(q[:m, :k].cpu().numpy(), act_want(x, s, z, bits))


def test_row_quantizer_special_rows():
    """All zeros, all subnormal, NaN among numbers, an infinity (an infinite scale: codes 0, the infinity's own is the
    lower bound as 0 * inf has no number)."""
    x = np.zeros((5, 1024), dtype=np.float32)
    rng = np.random.default_rng(0)
    x[1] = rng.standard_normal(1024).astype(np.float32) * np.float32(1e-40)
    x[2:] = rng.standard_normal((3, 1024)).astype(np.float32)
    x[3, 5] = np.nan
    x[4, 9] = np.inf
    q, s = run_rows(x)
    wq, ws = rows_want(x)
    np.testing.assert_array_equal(s, ws)
    np.testing.assert_array_equal(q, wq)


@pytest.mark.parametrize("m,k,edge", [(2 ** 25 + 5, 4, 2 ** 25), (2 ** 23 + 3, 1, 2 ** 23), (2 ** 24 + 2, 3, 2 ** 24)])
def test_row_quantizer_of_more_rows_than_one_launch_holds(m, k, edge):
    """Rows around the end of a launch, the first and the last, against Eq. 1; and every scale."""
    print(f"row quantizer {m} x {k}", flush=True)
    x = torch.randn(m, k, device=DEV, generator=torch.Generator(device=DEV).manual_seed(k))
    q, s = torch.full((m + 1, k), 77, dtype=torch.int8, device=DEV), torch.full((m + 1,), -7.0, device=DEV)
    P.cwac_quantize_rows_sym(x, s[:m], q[:m])
    torch.cuda.synchronize()
    assert (q[m] == 77).all() and s[m] == -7.0
    for at in (0, edge - 600, m - 1000):
        rows = slice(at, min(at + 1000, m))
        wq, ws = rows_want(x[rows].cpu().numpy())
        np.testing.assert_array_equal(q[rows].cpu().numpy(), wq)
        np.testing.assert_array_equal(s[rows].cpu().numpy(), ws)
    want = (x.abs().amax(1) / 127.0).clamp_min(float(TINY) * 256)  # (a row of zeros has the smallest scale)
    assert torch.allclose(s[:m], want, rtol=1e-6, atol=0)
