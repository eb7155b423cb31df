"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a dict of plain values; its "kind" names one of the five paths:

  linear     one W8A8 layer of a vision model as an engine calls it: the activation quantizer on the fp32
             input, then the int8 layer with the compensation in its epilogue
  decoder    the five linear layers of one LLM decoder layer (qkv, o, up, gate, down), with int8 weights
             and per-token activation codes ("w8") or with 4-bit weights and fp16 activations ("w4"); a
             few tokens are a decoding step, thousands a prefill
  encoder    a stack of W8A8 Vision Transformer blocks from residual stream to residual stream, over
             images or over windows with a relative position bias
  calibrate  a layer's preparation: weight quantizer, calibration forward, statistics, fit and fold, for
             int8 weights or for 4-bit ones
  conv       the three convolutions of a residual network's bottleneck in int8 codes

Inputs and weights are drawn from the seed with the statistics of the models these shapes belong to: a few
strong activation channels, weights of small variance, post-ReLU images."""
from __future__ import annotations

import math
import random

import torch
import torch.nn.functional as F

from paper_2505_20932_amd import binding as B

_DEV = "cuda:0"


# ------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # one image through the qkv layer of a small vision transformer: the smallest call there is
        dict(name="linear_deit_s_1_image", kind="linear", m=197, n=1152, k=384, epilogue="float"),
        # a decoding step of a 7B language model for a batch of 16 sequences, W8A8 with per-token scales
        dict(name="decoder_w8_16_tokens", kind="decoder", bits="w8", tokens=16, width=4096, hidden=11008),
        # its prefill, 8 sequences of 2048 tokens: the largest matrix products
        dict(name="decoder_w8_16384_tokens", kind="decoder", bits="w8", tokens=16384, width=4096, hidden=11008),
        # weight-only INT4: one user's decoding step, a ragged batch of 45 users, one prompt of 2048 tokens
        dict(name="decoder_w4_1_token", kind="decoder", bits="w4", tokens=1, width=4096, hidden=11008),
        dict(name="decoder_w4_45_tokens", kind="decoder", bits="w4", tokens=45, width=4096, hidden=11008),
        dict(name="decoder_w4_2048_tokens", kind="decoder", bits="w4", tokens=2048, width=4096, hidden=11008),
        # the encoder of ViT-B/16 for a single image (latency) and for a batch (throughput)
        dict(name="encoder_vit_b_1_image", kind="encoder", batch=1, tokens=197, heads=12, head_dim=64, hidden=3072,
             blocks=12, bias=False),
        dict(name="encoder_vit_b_128_images", kind="encoder", batch=128, tokens=197, heads=12, head_dim=64,
             hidden=3072, blocks=12, bias=False),
        # the same model at 384 x 384: sequences longer than one workgroup's keys
        dict(name="encoder_vit_b_384_8_images", kind="encoder", batch=8, tokens=577, heads=12, head_dim=64,
             hidden=3072, blocks=12, bias=False),
        # Swin-B's third stage, 37 images of four 7 x 7 windows: heads of 32, a relative position bias
        dict(name="encoder_swin_b_37_images", kind="encoder", batch=148, tokens=49, heads=16, head_dim=32,
             hidden=2048, blocks=18, bias=True),
        # the preparation of ViT-B's first MLP layer on 256 calibration images in batches of 64
        dict(name="calibrate_vit_b_fc1", kind="calibrate", bits="w8", per_token=False, fused=False, n=3072, k=768,
             rows=50432, batches=4),
        # a bottleneck of ResNet-50's fourth stage, 32 images
        dict(name="conv_resnet50_s4_32_images", kind="conv", batch=32, size=14, c_in=1024, c_mid=256, stride=1),
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(("linear", "decoder", "decoder", "encoder", "encoder", "calibrate", "conv"))
    if kind == "linear":
        # the layers of the DeiT / ViT / Swin families and a classifier head, any number of rows
        n, k = rng.choice(((1152, 384), (384, 1536), (768, 768), (2304, 768), (3072, 768), (768, 3072), (1000, 768),
                           (1536, 512), (512, 2048), (4096, 1024), (96, 384)))
        return dict(kind=kind, m=_log(rng, 1, 50432), n=n, k=k, epilogue=rng.choice(("float", "float", "fixed")))
    if kind == "decoder":
        width, hidden = rng.choice(((2048, 5504), (4096, 11008), (4096, 14336), (5120, 13824)))
        most = int(16384 * (4096 * 4096 * 4 + 3 * 4096 * 11008) / (width * width * 4 + 3 * width * hidden))
        bits = rng.choice(("w8", "w4"))
        return dict(kind=kind, bits=bits, tokens=_log(rng, 1, min(most, 16384 if bits == "w8" else 8192)),
                    width=width, hidden=hidden)
    if kind == "encoder":
        heads, head_dim, hidden, blocks, windows = rng.choice((
            (6, 64, 1536, 12, False), (12, 64, 3072, 12, False), (16, 64, 4096, 12, False), (20, 64, 5120, 8, False),
            (16, 32, 2048, 18, True), (8, 32, 1024, 2, True)))
        tokens = rng.choice((49, 144)) if windows else rng.choice((50, 197, 257, 577))
        rows = int(128 * 197 * 12 * 768 * 768 / (blocks * (heads * head_dim) ** 2 * max(1.0, tokens / 288)))
        return dict(kind=kind, batch=_log(rng, 1, max(1, min(rows, 25216) // tokens)), tokens=tokens, heads=heads,
                    head_dim=head_dim, hidden=hidden, blocks=blocks, bias=windows)
    if kind == "calibrate":
        bits = rng.choice(("w8", "w8", "w4"))
        per_token = bits == "w8" and rng.random() < 0.4
        n, k = ((rng.choice(((4096, 4096), (11008, 4096), (4096, 11008))) if per_token or bits == "w4" else
                 rng.choice(((1152, 384), (2304, 768), (768, 768), (3072, 768), (768, 3072), (2048, 512), (512, 2048)))))
        rows = _log(rng, 1024, min(50432, int(50432 * 3072 / n)))
        return dict(kind=kind, bits=bits, per_token=per_token, fused=bits == "w8" and rng.random() < 0.5, n=n, k=k,
                    rows=rows, batches=rng.randint(1, 3))
    size, c_in, c_mid = rng.choice(((56, 256, 64), (28, 512, 128), (14, 1024, 256), (7, 2048, 512)))
    stride = rng.choice((1, 1, 1, 2)) if size > 7 else 1
    return dict(kind=kind, batch=_log(rng, 1, 128), size=size, c_in=c_in, c_mid=c_mid, stride=stride)


# ------------------------------------------------------------------------------------------ inputs
class _Draw:
    """Seeded tensors on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device=_DEV).manual_seed(int(seed))
        self.r = random.Random(int(seed))

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.empty(*shape, dtype=torch.float32, device=_DEV).normal_(mean, std, generator=self.g)

    def activations(self, rows, k, share, gain):
        """N(0, 1) rows with a share of the channels scaled up by about `gain`."""
        x = self.normal(rows, k)
        ch = torch.tensor(self.r.sample(range(k), max(1, int(round(share * k)))), device=_DEV)
        x[:, ch] *= gain * torch.exp(0.5 * self.normal(len(ch)))
        return x


def _empty(*shape, dtype):
    return torch.empty(*shape, dtype=dtype, device=_DEV)


def _params_of_range(t):
    """Scale and signed zero-point of the 8-bit codes of a tensor (Eq. 2)."""
    mn, mx = (float(v) for v in torch.aminmax(t))
    s, z = B.cwac_qparams_from_range(mn, mx, 8)
    return s, z - 128


def _fold(d, w_q, s_w, bias, qp, n, fixed=False):
    """Engine parameters of a compensated int8 layer (alpha near 1, beta small)."""
    alpha, beta = d.normal(n, std=0.03, mean=1.0), d.normal(n, std=0.01)
    colsum, offset = _empty(n, dtype=torch.int32), _empty(n, dtype=torch.int32)
    B.cwac_colsum(w_q, colsum)
    if fixed:
        m0, shift = _empty(n, dtype=torch.int32), _empty(n, dtype=torch.int32)
        B.cwac_fold_fixed_point(alpha, beta, s_w, bias, colsum, qp, m0, shift, offset)
        return dict(m0=m0, shift=shift, offset=offset)
    mult, fbias = _empty(n, dtype=torch.float32), None
    if qp.mode == B.CWAC_EPI_FP_BIAS:
        fbias = _empty(n, dtype=torch.float32)
    B.cwac_fold(alpha, beta, s_w, bias, colsum, qp, mult, offset, fbias)
    return dict(mult=mult, offset=offset, fbias=fbias)


def _quantized(w):
    w_q, s_w = _empty(*w.shape, dtype=torch.int8), _empty(w.shape[0], dtype=torch.float32)
    B.cwac_quantize_rows_sym(w, s_w, w_q)
    return w_q, s_w


def _prepare_linear(c, d):
    m, n, k = c["m"], c["n"], c["k"]
    x = d.activations(m, k, 0.01, 20.0)
    w, bias = d.normal(n, k, std=0.02), d.normal(n, std=0.02)
    s_x, z_x = _params_of_range(x)
    s_r, z_r = _params_of_range(x[:256] @ w.t() + bias)
    w_q, s_w = _quantized(w)
    qp = B.make_qparams(s_x=s_x, z_x=z_x, s_r=s_r, z_r=z_r)
    return dict(x=x, w_q=w_q, qp=qp, x_q=_empty(m, k, dtype=torch.int8), out=_empty(m, n, dtype=torch.int8),
                **_fold(d, w_q, s_w, bias, qp, n, c["epilogue"] == "fixed"))


def _run_linear(s):
    qp = s["qp"]
    B.cwac_quantize_act(s["x"], qp.s_x, qp.z_x, s["x_q"])
    if "m0" in s:
        B.qlinear_cwac_forward_fixed_point(s["x_q"], s["w_q"], qp, s["m0"], s["shift"], s["offset"], s["out"])
    else:
        B.qlinear_cwac_forward(s["x_q"], s["w_q"], qp, s["mult"], s["offset"], None, None, B.CWAC_OUT_INT8, s["out"])
    return s["out"]


def _decoder_layers(c):
    """(layer, output channels, input channels, which activation it reads)"""
    w, h = c["width"], c["hidden"]
    return (("qkv", 3 * w, w, 0), ("o", w, w, 1), ("up", h, w, 2), ("gate", h, w, 2), ("down", w, h, 3))


def _w4(w):
    n, k = w.shape
    codes = _empty(n, k, dtype=torch.uint8)
    scales, zeros = _empty(n, k // 128, dtype=torch.float16), _empty(n, k // 128, dtype=torch.uint8)
    B.cwac_w4_quantize_groupwise(w, codes, scales, zeros)
    pw, sz = _empty(B.cwac_w4_packed_w_bytes(n, k), dtype=torch.uint8), _empty(n * (k // 128), dtype=torch.int32)
    B.cwac_w4_pack(codes, scales, zeros, pw, sz)
    return pw, sz


def _prepare_decoder(c, d):
    m = c["tokens"]
    widths = (c["width"], c["width"], c["width"], c["hidden"])
    xs = [d.activations(m, k, 0.002, 100.0 if c["bits"] == "w8" else 20.0) for k in widths]
    layers = []
    for name, n, k, which in _decoder_layers(c):
        w = d.normal(n, k, std=0.02)
        if c["bits"] == "w4":
            pw, sz = _w4(w)
            mult, fbias = _empty(n, dtype=torch.float32), _empty(n, dtype=torch.float32)
            B.cwac_fold_weight_only(d.normal(n, std=0.03, mean=1.0), d.normal(n, std=0.01), None, mult, fbias)
            layers.append(dict(n=n, which=which, pw=pw, sz=sz, mult=mult, fbias=fbias,
                               out=_empty(m, n, dtype=torch.float16)))
        else:
            s_r, z_r = _params_of_range(xs[which][:256] @ w.t())
            w_q, s_w = _quantized(w)
            qp = B.make_qparams(mode=B.CWAC_EPI_FP_BIAS, act_per_token=True, s_r=s_r, z_r=z_r)
            layers.append(dict(which=which, w_q=w_q, qp=qp, out=_empty(m, n, dtype=torch.int8),
                               **_fold(d, w_q, s_w, None, qp, n)))
    if c["bits"] == "w4":
        return dict(w4=True, xs=[x.half() for x in xs], layers=layers)
    return dict(w4=False, xs=xs, xq=[_empty(m, k, dtype=torch.int8) for k in widths],
                sx=[_empty(m, dtype=torch.float32) for _ in widths], layers=layers)


def _run_decoder(s):
    if s["w4"]:
        for L in s["layers"]:
            B.qlinear_w4a16_cwac_forward(s["xs"][L["which"]], L["pw"], L["sz"], L["n"], L["mult"], L["fbias"], L["out"])
    else:
        ready = -1
        for L in s["layers"]:
            i = L["which"]
            if i != ready:          # up and gate read the same codes
                B.cwac_quantize_rows_sym(s["xs"][i], s["sx"][i], s["xq"][i])
                ready = i
            B.qlinear_cwac_forward(s["xq"][i], L["w_q"], L["qp"], L["mult"], L["offset"], L["fbias"], s["sx"][i],
                                   B.CWAC_OUT_INT8, L["out"])
    return [L["out"] for L in s["layers"]]


def _prepare_encoder(c, d):
    batch, tokens, heads, hd, hidden = c["batch"], c["tokens"], c["heads"], c["head_dim"], c["hidden"]
    width, m = heads * hd, batch * tokens
    h = d.normal(m, width)
    h[:, torch.tensor(d.r.sample(range(width), max(1, width // 100)), device=_DEV)] *= 8.0
    h = h.half()
    # the floating-point model on a few images gives the ranges of the tensors that are quantized
    few = min(batch, max(1, 788 // tokens))
    t = h[:few * tokens].float()
    blocks, keep = [], []
    for _ in range(c["blocks"]):
        g1, b1 = d.normal(width, std=0.1, mean=1.0), d.normal(width, std=0.05)
        g2, b2 = d.normal(width, std=0.1, mean=1.0), d.normal(width, std=0.05)
        bias = pos = None
        if c["bias"]:
            pos = torch.zeros(heads, tokens, (tokens + 31) // 32 * 32, dtype=torch.float16, device=_DEV)
            pos[:, :, :tokens] = d.normal(heads, tokens, tokens, std=0.5).half()
            bias = pos[None, :, :, :tokens].float()
        shapes = ((3 * width, width), (width, width), (hidden, width), (width, hidden))
        # the two layers that end in the residual stream add little to it, as in a trained deep stack
        gain = (1.0, 1.0 / math.sqrt(2 * c["blocks"]), 1.0, 1.0 / math.sqrt(2 * c["blocks"]))
        ws = [d.normal(n, k, std=g / math.sqrt(k)) for (n, k), g in zip(shapes, gain)]
        bs = [d.normal(n, std=0.02) for n, _ in shapes]
        x1 = F.layer_norm(t, (width,), g1, b1, 1e-6)
        r1 = x1 @ ws[0].t() + bs[0]
        q, k_, v = (r1[:, j * width:(j + 1) * width].reshape(few, tokens, heads, hd).transpose(1, 2).contiguous()
                    for j in range(3))
        logits = torch.matmul(q, k_.transpose(2, 3).contiguous()) / math.sqrt(hd)
        a = torch.matmul(torch.softmax(logits if bias is None else logits + bias, -1), v)
        a = a.transpose(1, 2).reshape(few * tokens, width)
        r2 = a @ ws[1].t() + bs[1]
        t = t + r2
        x2 = F.layer_norm(t, (width,), g2, b2, 1e-6)
        r3 = x2 @ ws[2].t() + bs[2]
        g = F.gelu(r3)
        r4 = g @ ws[3].t() + bs[3]
        t = t + r4
        layers = []
        ins, outs = [_params_of_range(v) for v in (x1, a, x2, g)], [_params_of_range(v) for v in (r1, r2, r3, r4)]
        for w, bia, (s_x, z_x), (s_r, z_r) in zip(ws, bs, ins, outs):
            w_q, s_w = _quantized(w)
            qp = B.make_qparams(s_x=s_x, z_x=z_x, s_r=s_r, z_r=z_r)
            f = _fold(d, w_q, s_w, bia, qp, w.shape[0])
            layers.append(dict(w_q=w_q, mult=f["mult"], offset=f["offset"], s_x=s_x, z_x=z_x, s_r=s_r, z_r=z_r))
        table = _empty(256, dtype=torch.int8)
        B.vit_gelu_table(outs[2][0], outs[2][1], ins[3][0], ins[3][1], table)
        blocks.append(B.make_block_params(batch, tokens, heads, hidden, 1e-6, (g1, b1), (g2, b2), layers, table, hd, pos))
        keep.append((g1, b1, g2, b2, layers, table, pos))
    ws = _empty(B.vit_block_workspace(batch, tokens, heads, hidden), dtype=torch.uint8)
    return dict(blocks=blocks, keep=keep, h=h, out=torch.empty_like(h), ws=ws)


def _run_encoder(s):
    B.vit_encoder_w8a8_forward(s["blocks"], s["h"], s["out"], s["ws"])
    return s["out"]


def _batches(c):
    """First row and number of rows of each calibration batch."""
    rows, n = c["rows"], c["batches"]
    at = [rows * i // n for i in range(n + 1)]
    return [(a, b - a) for a, b in zip(at, at[1:])]


def _prepare_calibrate(c, d):
    n, k, rows = c["n"], c["k"], c["rows"]
    llm = c["per_token"] or c["bits"] == "w4"
    w, bias = d.normal(n, k, std=0.02), None if llm else d.normal(n, std=0.02)
    x = d.activations(rows, k, 0.002 if llm else 0.01, 100.0 if c["per_token"] else 20.0)
    y = x @ w.t() if bias is None else torch.addmm(bias, x, w.t())
    most = max(r for _, r in _batches(c))
    f32, i32 = torch.float32, torch.int32
    s = dict(c=c, w=w, bias=bias, x=x.half() if c["bits"] == "w4" else x, y=y,
             stats=_empty(B.cwac_stats_bytes(n), dtype=torch.uint8), alpha=_empty(n, dtype=f32),
             beta=_empty(n, dtype=f32), mult=_empty(n, dtype=f32), fbias=_empty(n, dtype=f32))
    s["ws"] = _empty(max(B.cwac_calibrate_stats_workspace(most, n), B.cwac_calibrate_fused_workspace(most, n)),
                     dtype=torch.uint8)
    if not c["fused"]:
        s["y_q"] = _empty(most, n, dtype=f32)
    if c["bits"] == "w4":
        s.update(codes=_empty(n, k, dtype=torch.uint8), scales=_empty(n, k // 128, dtype=torch.float16),
                 zeros=_empty(n, k // 128, dtype=torch.uint8),
                 pw=_empty(B.cwac_w4_packed_w_bytes(n, k), dtype=torch.uint8), sz=_empty(n * (k // 128), dtype=i32))
        return s
    s_x, z_x = (1.0, 0) if c["per_token"] else _params_of_range(x)
    s_r, z_r = _params_of_range(y)
    mode = B.CWAC_EPI_FP_BIAS if c["per_token"] else B.CWAC_EPI_INT_OFFSET
    s.update(w_q=_empty(n, k, dtype=torch.int8), s_w=_empty(n, dtype=f32), colsum=_empty(n, dtype=i32),
             offset=_empty(n, dtype=i32), d_mult=_empty(n, dtype=f32), d_fbias=_empty(n, dtype=f32),
             d_offset=_empty(n, dtype=i32), x_q=_empty(most, k, dtype=torch.int8), s_x=_empty(most, dtype=f32),
             qp_deq=B.make_qparams(mode=B.CWAC_EPI_FP_BIAS, act_per_token=c["per_token"], s_x=s_x, z_x=z_x),
             qp=B.make_qparams(mode=mode, act_per_token=c["per_token"], s_x=s_x, z_x=z_x, s_r=s_r, z_r=z_r))
    return s


def _run_calibrate(s):
    c, n = s["c"], s["c"]["n"]
    w4 = c["bits"] == "w4"
    if w4:
        B.cwac_w4_quantize_groupwise(s["w"], s["codes"], s["scales"], s["zeros"])
        B.cwac_w4_pack(s["codes"], s["scales"], s["zeros"], s["pw"], s["sz"])
    else:
        B.cwac_quantize_rows_sym(s["w"], s["s_w"], s["w_q"])
        B.cwac_colsum(s["w_q"], s["colsum"])
        B.cwac_fold(None, None, s["s_w"], s["bias"], s["colsum"], s["qp_deq"], s["d_mult"], s["d_offset"], s["d_fbias"])
    if c["fused"]:
        B.cwac_stats_reset(s["stats"], n)
    for i, (a, rows) in enumerate(_batches(c)):
        x, y = s["x"][a:a + rows], s["y"][a:a + rows]
        if w4:
            y_q = s["y_q"][:rows]
            B.qlinear_w4a16_cwac_forward(x, s["pw"], s["sz"], n, None, None, y_q)
        else:
            x_q, s_x = s["x_q"][:rows], None
            if c["per_token"]:
                s_x = s["s_x"][:rows]
                B.cwac_quantize_rows_sym(x, s_x, x_q)
            else:
                B.cwac_quantize_act(x, s["qp"].s_x, s["qp"].z_x, x_q)
            if c["fused"]:
                B.qlinear_cwac_calibrate_fused(x_q, s["w_q"], s["d_mult"], s["d_offset"], s["d_fbias"], s_x, y,
                                               s["stats"], s["ws"])
                continue
            y_q = s["y_q"][:rows]
            B.qlinear_cwac_forward(x_q, s["w_q"], None, s["d_mult"], s["d_offset"], s["d_fbias"], s_x,
                                   B.CWAC_OUT_FP32, y_q)
        B.cwac_calibrate_stats(y, y_q, s["stats"], s["ws"], first=i == 0)
    B.cwac_solve(s["stats"], n, s["alpha"], s["beta"])
    if w4:
        B.cwac_fold_weight_only(s["alpha"], s["beta"], s["bias"], s["mult"], s["fbias"])
        return [s["pw"], s["sz"], s["alpha"], s["beta"], s["mult"], s["fbias"]]
    fbias = s["fbias"] if c["per_token"] else None
    B.cwac_fold(s["alpha"], s["beta"], s["s_w"], s["bias"], s["colsum"], s["qp"], s["mult"], s["offset"], fbias)
    return [s["w_q"], s["s_w"], s["alpha"], s["beta"], s["mult"], s["offset"]] + ([fbias] if c["per_token"] else [])


def _conv_layers(c):
    """(filter [c_out, kh, kw, c_in], stride, padding, input size)"""
    mid, c_in, size, st = c["c_mid"], c["c_in"], c["size"], c["stride"]
    return (((mid, 1, 1, c_in), 1, 0, size), ((mid, 3, 3, mid), st, 1, size),
            ((4 * mid, 1, 1, mid), 1, 0, (size + 2 - 3) // st + 1))


def _prepare_conv(c, d):
    batch, size = c["batch"], c["size"]
    x = d.activations(batch * size * size, c["c_in"], 0.01, 4.0).abs_().view(batch, size, size, c["c_in"])
    s_x, z_x = _params_of_range(x)
    x_q = _empty(batch * size * size, c["c_in"], dtype=torch.int8)
    B.cwac_quantize_act(x.view(-1, c["c_in"]), s_x, z_x, x_q)
    t, layers = x[:4], []
    for i, (shape, stride, pad, hw) in enumerate(_conv_layers(c)):
        n, kh, kw, ci = shape
        w, bias = d.normal(*shape, std=1.0 / math.sqrt(kh * kw * ci)), d.normal(n, std=0.02)
        patches = F.unfold(t.permute(0, 3, 1, 2), (kh, kw), padding=pad, stride=stride).transpose(1, 2)
        wf = w.permute(0, 3, 1, 2).reshape(n, -1)
        oh = (hw + 2 * pad - kh) // stride + 1
        y = (patches.reshape(-1, wf.shape[1]) @ wf.t() + bias).view(t.shape[0], oh, oh, n)
        if i < 2:                     # the activation of these two is folded into their output range
            y = torch.relu(y)
        s_r, z_r = _params_of_range(y)
        w_q, s_w = _quantized(w.view(n, -1))
        qp = B.make_qparams(s_x=s_x, z_x=z_x, s_r=s_r, z_r=z_r)
        layers.append(dict(w_q=w_q.view(shape), stride=stride, pad=pad, qp=qp,
                           out=_empty(batch * oh * oh, n, dtype=torch.int8), view=(batch, oh, oh, n),
                           **_fold(d, w_q, s_w, bias, qp, n)))
        t, s_x, z_x = y, s_r, z_r
    return dict(x_q=x_q.view(batch, size, size, c["c_in"]), layers=layers)


def _run_conv(s):
    x = s["x_q"]
    for L in s["layers"]:
        B.qconv2d_cwac_forward(x, L["w_q"], L["stride"], L["pad"], L["qp"], L["mult"], L["offset"], None,
                               B.CWAC_OUT_INT8, L["out"])
        x = L["out"].view(L["view"])
    return [L["out"] for L in s["layers"]]


_PREPARE = dict(linear=_prepare_linear, decoder=_prepare_decoder, encoder=_prepare_encoder,
                calibrate=_prepare_calibrate, conv=_prepare_conv)
_RUN = dict(linear=_run_linear, decoder=_run_decoder, encoder=_run_encoder, calibrate=_run_calibrate, conv=_run_conv)


def prepare(case, seed):
    return case["kind"], _PREPARE[case["kind"]](case, _Draw(seed))


def run(state):
    return _RUN[state[0]](state[1])


# ------------------------------------------------------------------------------------------ the measure
def work(case):
    """Bytes and operations of one pass: inputs once, outputs once, weights at their stored width."""
    c, kind = case, case["kind"]
    if kind == "linear":
        m, n, k = c["m"], c["n"], c["k"]
        return dict(bytes=4.0 * m * k + n * k + m * n + 8.0 * n, flops=2.0 * m * n * k)
    if kind == "decoder":
        m, w4 = c["tokens"], c["bits"] == "w4"
        by = (2.0 if w4 else 4.0) * m * (3 * c["width"] + c["hidden"])
        fl = 0.0
        for _, n, k, _ in _decoder_layers(c):
            by += n * k * (0.5 + 4.0 / 128 if w4 else 1.0) + m * n * (2.0 if w4 else 1.0) + 8.0 * n
            fl += 2.0 * m * n * k
        return dict(bytes=by, flops=fl)
    if kind == "encoder":
        width, m = c["heads"] * c["head_dim"], c["batch"] * c["tokens"]
        by = 4.0 * m * width
        per = 4.0 * width * width + 2.0 * width * c["hidden"]
        bias = 2.0 * c["heads"] * c["tokens"] * ((c["tokens"] + 31) // 32 * 32) if c["bias"] else 0.0
        by += c["blocks"] * (per + bias + 8.0 * (5 * width + c["hidden"]) + 16.0 * width)
        return dict(bytes=by, flops=c["blocks"] * (2.0 * m * per + 4.0 * m * c["tokens"] * width))
    if kind == "calibrate":
        n, k, rows = c["n"], c["k"], c["rows"]
        w4 = c["bits"] == "w4"
        return dict(bytes=(2.0 if w4 else 4.0) * rows * k + 4.0 * rows * n + n * k * (4.5 if w4 else 5.0),
                    flops=2.0 * rows * n * k)
    by, fl = 1.0 * c["batch"] * c["size"] ** 2 * c["c_in"], 0.0
    for (n, kh, kw, ci), stride, pad, hw in _conv_layers(c):
        oh = (hw + 2 * pad - kh) // stride + 1
        by += n * kh * kw * ci + c["batch"] * oh * oh * n + 8.0 * n
        fl += 2.0 * c["batch"] * oh * oh * n * kh * kw * ci
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """Integer paths are exact.  The others were compared with fp64 evaluations of the same definitions: the
    weight-only layer (fp32 sums, a few fp16 roundings at ties) was off by rel 2e-5, max 1e-3; the encoders by
    rel 0.008 to 0.016, max 0.06 to 0.08 - a code of an attention's or a layer norm's output that sits at a tie
    moves everything behind it; statistics, fit and fold agree to the last fp32 digit or two."""
    if case["kind"] == "decoder" and case["bits"] == "w4":
        return dict(rel=7e-5, max=4e-3)
    if case["kind"] == "encoder":
        return dict(rel=0.03, max=0.3)
    if case["kind"] == "calibrate":
        # fit and fold of fp64 sums; with 4-bit weights of fp32 outputs whose sums have no fixed order
        return dict(rel=2e-5, max=1e-4, differ=1e-3) if case["bits"] == "w4" else dict(rel=1e-6, max=1e-5, differ=1e-3)
    return "exact"
