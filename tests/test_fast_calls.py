"""The binding's native calls: taken for what a call documents, and only for that; everything else goes on to the ctypes
form and is refused or accepted as that one does."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import paper_2505_20932_amd as P
from paper_2505_20932_amd import binding as B

DEV = "cuda:0"


def test_what_does_not_fit_is_left_to_the_ctypes_form():
    calls = B._fast_calls()
    x, q, s = torch.zeros(4, 32), torch.zeros(4, 32, dtype=torch.int8), torch.zeros(4)
    assert calls.quantize_act(x, 0.1, 0, q, None) is False             # not on a device
    assert calls.quantize_rows_sym(x, s, q, None) is False
    assert calls.quantize_act(x, 0.1, 0, q) is False                   # too few arguments
    assert calls.forward(*[None] * 10) is False and calls.w4a16(*[3] * 8) is False and calls.conv2d(*["x"] * 11) is False
    for call in (lambda: P.cwac_quantize_act(x, 0.1, 0, q), lambda: P.cwac_quantize_rows_sym(x, s, q),
                 lambda: P.cwac_quantize_act(x.double(), 0.1, 0, q)):
        with pytest.raises(AssertionError):
            call()
    with pytest.raises(KeyError):
        calls.bind(B.cwac_qparams, {}, B._check)
    assert B._fast_calls() is calls


def test_without_the_extension_module_the_ctypes_form_serves_every_call(monkeypatch):
    """Not built, or built for another Python or torch: the import fails, and the library is usable all the same."""
    import sys
    monkeypatch.delattr(P, "_fast_calls", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2505_20932_amd._fast_calls", None)
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_calls", None)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        B.lib()
    assert B.cwac_forward_kernel_for(197, 768, 768, 768, 768) == B.CWAC_KERNEL_SPLIT_K
    x, q = torch.zeros(4, 32), torch.zeros(4, 32, dtype=torch.int8)
    assert B._fast_calls().quantize_act(x, 0.1, 0, q, None) is False
    with pytest.raises(AssertionError):                                # the ctypes form's own refusal
        P.cwac_quantize_act(x, 0.1, 0, q)


def layer(seed=0, m=5, n=48, k=64):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randint(-128, 128, (m, k), dtype=torch.int8, device=DEV, generator=g)
    w = torch.randint(-127, 128, (n, k), dtype=torch.int8, device=DEV, generator=g)
    mult = torch.rand(n, device=DEV, generator=g) * 1e-3 + 1e-4
    off = torch.randint(-500, 500, (n,), dtype=torch.int32, device=DEV, generator=g)
    return x, w, mult, off, B.make_qparams(z_r=3), torch.empty(m, n, dtype=torch.int8, device=DEV)


def by_ctypes(x, w, mult, off, qp, stream=None):
    out = torch.empty(x.shape[0], w.shape[0], dtype=torch.int8, device=DEV)
    P.qlinear_cwac_forward(x, w, qp, mult, off, None, None, P.CWAC_OUT_INT8, out, stream, tuning=B.make_tuning())
    return out


@pytest.mark.gpu
def test_native_and_ctypes_forms_agree():
    calls = B._fast_calls()
    x, w, mult, off, qp, out = layer()
    want = by_ctypes(x, w, mult, off, qp)
    assert calls.forward(x, w, qp, mult, off, None, None, P.CWAC_OUT_INT8, out, None) is True
    assert torch.equal(out, want)
    wide = torch.zeros(5, 64, dtype=torch.int8, device=DEV)            # a pitch of its own, and a parameter
    assert calls.forward(x, torch.nn.Parameter(w, requires_grad=False), qp, mult, off, None, None, 0, wide[:, :48], None) is True
    assert torch.equal(wide[:, :48], want) and (wide[:, 48:] == 0).all()
    tab = torch.arange(127, -129, -1, device=DEV).to(torch.int8)
    assert calls.forward_table(x, w, qp, mult, off, tab, out, None) is True
    assert torch.equal(out, tab[want.long() + 128])
    m0 = torch.full((48,), 1 << 30, dtype=torch.int32, device=DEV)
    sh = torch.full((48,), 41, dtype=torch.int32, device=DEV)
    fixed = torch.empty_like(out)
    assert calls.forward_fixed_point(x, w, qp, m0, sh, off, out, None) is True
    P.qlinear_cwac_forward_fixed_point(x, w, qp, m0, sh, off, fixed, tuning=B.make_tuning())
    assert torch.equal(out, fixed)
    img, fil = x[:4].view(1, 4, 1, 64).contiguous(), w.view(48, 1, 1, 64)
    img = img.expand(2, 4, 1, 64).contiguous()
    conv, conv_c = torch.empty(8, 48, dtype=torch.int8, device=DEV), torch.empty(8, 48, dtype=torch.int8, device=DEV)
    assert calls.conv2d(img, fil, 1, 0, qp, mult, off, None, 0, conv, None) is True
    P.qconv2d_cwac_forward(img, fil, 1, 0, qp, mult, off, None, 0, conv_c, tuning=B.make_tuning())
    assert torch.equal(conv, conv_c) and torch.equal(conv[:4], want[:4])
    xf = torch.randn(3, 256, device=DEV).half()
    pw = torch.randint(0, 256, (B.cwac_w4_packed_w_bytes(256, 256),), dtype=torch.uint8, device=DEV)
    sz = torch.full((2 * 256,), 0x3C00 | (7 << 16), dtype=torch.int32, device=DEV)
    for dt in (torch.float16, torch.float32):
        a, b = torch.empty(3, 256, dtype=dt, device=DEV), torch.empty(3, 256, dtype=dt, device=DEV)
        assert calls.w4a16(xf, pw, sz, 256, None, None, a, None) is True
        P.qlinear_w4a16_cwac_forward(xf, pw, sz, 256, None, None, b, tuning=B.make_tuning())
        assert torch.equal(a, b)
    f = torch.randn(1, 64, device=DEV)
    q, s = torch.empty(1, 64, dtype=torch.int8, device=DEV), torch.empty(1, device=DEV)
    assert calls.quantize_rows_sym(f, s, q, None) is True and calls.quantize_act(f, 0.1, 3, q, None) is True


@pytest.mark.gpu
def test_misfits_are_refused_as_before():
    calls = B._fast_calls()
    x, w, mult, off, qp, out = layer()
    bad = [((x.float(), w, qp, mult, off, None, None, 0, out), AssertionError), ((x, w[:, :32], qp, mult, off, None, None, 0, out), AssertionError),
           ((x, w, qp, mult, off, None, None, 1, out), AssertionError), ((x, w, qp, mult.cpu(), off, None, None, 0, out), AssertionError),
           ((x, w, qp, mult, off, None, None, 0, out[:4]), AssertionError), ((x, w, qp, None, off, None, None, 0, out), B.CwacError),
           ((x, w, None, mult, off, None, None, 0, out), B.CwacError), ((x, w, qp, mult, off, None, mult, 0, out), B.CwacError),
           ((x[:, 8:40], w[:, 8:40], qp, mult, off, None, None, 0, out), B.CwacError)]          # 8-byte aligned rows
    for args, error in bad:
        assert calls.forward(*args, None) is False
        with pytest.raises(error):
            P.qlinear_cwac_forward(*args)
    with pytest.raises(AssertionError):
        P.cwac_quantize_act(torch.zeros(4, 8, device=DEV).t(), 0.1, 0, torch.zeros(8, 4, dtype=torch.int8, device=DEV))
    with pytest.raises(B.CwacError):
        P.cwac_quantize_act(torch.zeros(4, 8, device=DEV), -1.0, 0, torch.zeros(4, 8, dtype=torch.int8, device=DEV))
    q = torch.zeros(4, 8, dtype=torch.int8, device=DEV)
    P.cwac_quantize_act(torch.ones(4, 8, device=DEV), np.float32(0.5), np.int64(1), q)                 # numbers of other types
    assert (q == 3).all()


@pytest.mark.gpu
def test_a_failed_launch_raises_at_once():
    """The status of a refused launch comes with the runtime's error, which a second call would not see."""
    calls, made = B._fast_calls(), []
    x, q = torch.ones(4, 8, device=DEV), torch.zeros(4, 8, dtype=torch.int8, device=DEV)
    refuse = ctypes.CFUNCTYPE(ctypes.c_int32, *B.lib().cwac_quantize_act.argtypes)(lambda *a: made.append(1) or -6)
    names = ("cwac_quantize_act", "cwac_quantize_rows_sym", "qlinear_cwac_forward", "qlinear_cwac_forward_table",
             "qlinear_cwac_forward_fixed_point", "qconv2d_cwac_forward", "qlinear_w4a16_cwac_forward")
    real = {n: ctypes.cast(getattr(B.lib(), n), ctypes.c_void_p).value for n in names}
    calls.bind(B.cwac_qparams, dict(real, cwac_quantize_act=ctypes.cast(refuse, ctypes.c_void_p).value), B._check)
    try:
        with pytest.raises(B.CwacError, match="cwac_quantize_act"):
            P.cwac_quantize_act(x, 0.5, 1, q)
    finally:
        calls.bind(B.cwac_qparams, real, B._check)
    assert len(made) == 1
    P.cwac_quantize_act(x, 0.5, 1, q)
    assert (q == 3).all()


@pytest.mark.gpu
def test_streams_and_threads():
    x, w, mult, off, qp, out = layer(3, 200, 512, 512)
    want = by_ctypes(x, w, mult, off, qp)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):                                          # the current stream ...
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):                             # ... or the call would not be in the capture
            P.qlinear_cwac_forward(x, w, qp, mult, off, None, None, 0, out)
    out.zero_()
    torch.cuda.synchronize()
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        out.zero_()
        torch.cuda.synchronize()
    P.qlinear_cwac_forward(x, w, qp, mult, off, None, None, 0, out, s)   # a stream given
    s.synchronize()
    assert torch.equal(out, want)
    outs = [torch.zeros_like(out) for _ in range(4)]
    torch.cuda.synchronize()

    def work(i):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(50):
                P.qlinear_cwac_forward(x, w, qp, mult, off, None, None, 0, outs[i])
        st.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(torch.equal(o, want) for o in outs)
