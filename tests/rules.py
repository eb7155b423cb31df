"""The library's HIP-free dispatch rules (paper_2505_20932_amd/csrc/*_rules.h), compiled with g++ for the CPU tests."""
import ctypes as C
import os
import subprocess
import tempfile

_ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_CSRC = os.path.join(_ROOT, "paper_2505_20932_amd", "csrc")

_SHIM = r"""
#include "attention_rules.h"
#include "fast_rules.h"
#include "quantize_rules.h"
#include "splitk_rules.h"
#include "w4_rules.h"
using namespace cwac;
// the weight-streaming kernel's tile for the layer, -1 where the tiled kernel takes it
extern "C" int w4_tile(long long m, int n, int k) {
  const int tile = w4_stream_tile(m, n, k);
  return w4_stream_pays(m, n, k, tile) ? tile : -1;
}
extern "C" int w4_tile16(long long m, int n, int k) { return w4_stream16_pays(m, n, k); }
// the direct-to-LDS kernel's tile shape for a linear layer of n >= 256 channels
extern "C" int fast_shape(long long m, int n, int k, int out_bytes) { return fast_linear_shape(m, n, k, out_bytes); }
// the small-problem kernel's tile, 0 where the tile kernels take the layer
extern "C" int split_tile(long long m, int n, int k) { return splitk_tile(m, n, k); }
extern "C" int table(long long m, int n, int k) { return table_form(m, n, k); }
extern "C" void split_shape(int tile, int *out) {
  const SplitkTile &t = kSplitk[tile];
  out[0] = t.tn, out[1] = t.tm, out[2] = t.w, out[3] = t.d;
}
extern "C" int attention(int tokens, long long pairs, int head_dim, int bias) { return attention_form(tokens, pairs, head_dim, bias); }
extern "C" int row_threads(long long rows, int k, int vec) { return quantize_row_threads(rows, k, vec); }
extern "C" long long rows_per_launch(long long rows, int k, int vec) { return quantize_rows_per_launch(rows, k, vec); }
extern "C" int w4_cut(long long tiles) { return w4_pieces(tiles); }
extern "C" int w4_tiles() { return kW4StreamTiles; }
extern "C" void w4_shape(int tile, int *out) {
  const W4StreamTile &t = kW4Stream[tile];
  out[0] = t.nb, out[1] = t.mp, out[2] = t.nw, out[3] = t.depth;
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
            with open(src, "w") as f:
                f.write(_SHIM)
            subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", _CSRC, "-I", os.path.join(_ROOT, "include"), src, "-o", so],
                           check=True)
            _lib = C.CDLL(so)
        _lib.w4_tile.argtypes = [C.c_longlong, C.c_int, C.c_int]
        _lib.split_tile.argtypes = [C.c_longlong, C.c_int, C.c_int]
        _lib.split_shape.argtypes = [C.c_int, C.POINTER(C.c_int)]
        _lib.fast_shape.argtypes = [C.c_longlong, C.c_int, C.c_int, C.c_int]
        _lib.w4_shape.argtypes = [C.c_int, C.POINTER(C.c_int)]
    return _lib


def w4_tile(m, n, k):
    return lib().w4_tile(m, n, k)


def w4_tile16(m, n, k):
    """Whether up to 16 tokens stream in tiles of 16 channels."""
    return bool(lib().w4_tile16(C.c_longlong(m), n, k))


def fast_shape(m, n, k, out_bytes):
    """CWAC_SHAPE_* the direct-to-LDS kernel picks for a linear layer of at least 256 channels."""
    return lib().fast_shape(m, n, k, out_bytes)


ATTN_SPLIT, ATTN_CHUNKS, ATTN_CHUNKS_WIDE = 0, 8, 9


def attention_form(batch, heads, tokens, head_dim, bias):
    """ATTN_*, or 1 .. 7: the number of key tiles that a workgroup holds."""
    return lib().attention(tokens, C.c_longlong(batch * heads), head_dim, bool(bias))


def quantize_grid(rows, k, vec):
    """(rows of one launch of the row quantizer, threads per row)."""
    lib().rows_per_launch.restype = C.c_longlong
    return lib().rows_per_launch(C.c_longlong(rows), k, vec), lib().row_threads(C.c_longlong(rows), k, vec)


def split_tile(m, n, k):
    return lib().split_tile(m, n, k)


def table_form(m, n, k):
    """What a layer with a code table takes instead of the 64 x 64 tile: 0 nothing, 1 split-K, 2 direct-to-LDS."""
    return lib().table(C.c_longlong(m), n, k)


def split_shape(tile):
    """(16-channel blocks, 16-token blocks, wavefronts, ring depth) of the small-problem kernel's tile."""
    out = (C.c_int * 4)()
    lib().split_shape(tile, out)
    return tuple(out)


def w4_pieces(m, n):
    """Pieces to a tile of the last round of 512-channel tiles (1: whole)."""
    return lib().w4_cut(C.c_longlong(-(-m // 128) * -(-n // 512)))


def w4_shape(tile):
    """(blocks of 32 channels, tokens, wavefronts, ring depth) of the weight-streaming kernel's tile."""
    out = (C.c_int * 4)()
    lib().w4_shape(tile, out)
    return tuple(out)
