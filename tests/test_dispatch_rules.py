"""Dispatch rules on the CPU: which kernel and tile a layer's sizes pick."""
import ctypes as C

import pytest

import rules
from test_gpu_small_problem import MAIN_LOOP as SPLIT_MAIN_LOOP
from test_gpu_w4_mid_batch import MAIN_LOOP as W4_MAIN_LOOP
from paper_2505_20932_amd import binding as B

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


# microseconds measured with cold weights: the tiled kernel's 128-token tiles, the streaming kernel with its tile
MEASURED = [(384, 12288, 128, 7.0, 16.3), (200, 24576, 128, 7.3, 16.8), (100, 49152, 128, 7.4, 16.2), (64, 65536, 128, 7.3, 14.5),
            (384, 12288, 384, 10.8, 20.3), (256, 24576, 256, 10.2, 18.3), (33, 65536, 384, 11.3, 16.8), (512, 8192, 512, 12.3, 15.4),
            (128, 32768, 768, 16.4, 19.5), (128, 4096, 4096, 55.0, 10.0), (400, 4096, 4096, 55.5, 24.1),
            (256, 4096, 11008, 119.0, 34.1), (200, 12288, 4096, 56.7, 41.3)]


@pytest.mark.parametrize("m,n,k,tiled,streaming", MEASURED)
def test_weight_only_mid_batch_takes_the_kernel_that_measured_faster(m, n, k, tiled, streaming):
    """A wide layer with a short K is one round of the tiled kernel and several of the streaming one's."""
    assert (rules.w4_tile(m, n, k) >= 0) == (streaming < tiled)


# microseconds measured with cold weights: the persistent 256 x 256 tile, 128 x 128 tiles
@pytest.mark.parametrize("m,n,k,out_bytes,persistent,quarter",
                         [(1979, 3952, 1280, 1, 21.1, 16.2), (16337, 448, 1664, 1, 23.4, 18.2), (3193, 2416, 384, 1, 12.7, 9.2),
                          (1310, 5600, 384, 4, 13.6, 10.4), (1863, 4064, 128, 1, 9.5, 6.8), (8031, 816, 128, 4, 12.6, 9.2),
                          (7107, 1072, 128, 1, 9.2, 6.4), (3106, 2656, 128, 1, 9.1, 8.2), (1517, 6256, 128, 4, 13.8, 11.8),
                          (12608, 2304, 384, 4, 34.5, 31.5), (25216, 1152, 512, 4, 39.9, 32.0), (12608, 2304, 768, 4, 44.7, 39.2),
                          (50432, 2304, 768, 4, 134.9, 139.8), (25216, 2304, 768, 4, 76.8, 79.4), (20000, 2304, 768, 4, 62.7, 64.8),
                          (16000, 3072, 768, 4, 65.4, 67.6), (7252, 4096, 1024, 4, 49.1, 50.6), (30000, 1024, 1024, 4, 49.4, 51.6), (20000, 1536, 384, 4, 35.9, 32.9),
                          (7252, 4096, 512, 4, 37.9, 33.8), (12608, 1024, 1024, 4, 24.2, 26.1), (3152, 4096, 512, 4, 20.0, 20.9), (9000, 1536, 384, 4, 18.9, 19.7),
                          (5000, 2560, 896, 4, 22.8, 24.5), (9000, 1152, 512, 4, 17.9, 16.2), (12608, 1000, 768, 4, 39.5, 37.1), (3152, 3840, 640, 4, 20.0, 17.7), (25216, 1152, 1024, 4, 51.8, 46.9), (25216, 2304, 1024, 4, 87.7, 92.7),
                          (20000, 1536, 1536, 4, 61.5, 73.4), (2000, 3072, 768, 1, 13.6, 10.0), (3152, 3072, 768, 1, 14.3, 15.2), (12608, 768, 3072, 4, 39.4, 45.7)])
def test_half_a_round_of_large_tiles_takes_the_tile_that_measured_faster(m, n, k, out_bytes, persistent, quarter):
    want = B.CWAC_SHAPE_128_128 if quarter < persistent else B.CWAC_SHAPE_256_PERSIST
    assert rules.fast_shape(m, n, k, out_bytes) == want


# microseconds measured with cold weights: the 64 x 64 tile kernel, the split-K kernel with its tile
@pytest.mark.parametrize("m,n,k,tile,split", [(350, 3040, 1776, 11.8, 12.9), (547, 2352, 3472, 20.1, 23.4), (481, 2912, 3280, 20.2, 23.0),
                                              (286, 5120, 8944, 62.5, 72.4), (2655, 544, 9504, 49.2, 57.9), (1348, 832, 4720, 25.5, 27.5),
                                              (296, 4096, 2000, 13.5, 14.6), (197, 768, 768, 5.7, 3.5), (197, 768, 3072, 16.7, 5.0),
                                              (1576, 768, 3072, 18.0, 15.8), (16, 4096, 4096, 29.2, 6.7), (200, 11008, 4096, 33.4, 41.0)])
def test_small_layers_take_the_kernel_that_measured_faster(m, n, k, tile, split):
    assert (rules.split_tile(m, n, k) != 0) == (split < tile)


# microseconds measured with cold weights: eight and four wavefronts to a workgroup of the weight-streaming kernel
@pytest.mark.parametrize("m,n,k,eight,four", [(16, 24576, 128, 5.1, 3.8), (16, 24576, 256, 5.4, 4.0), (12, 131072, 512, 22.8, 13.8),
                                              (16, 131072, 1024, 30.9, 22.1), (1, 131072, 256, 15.1, 9.8), (8, 131072, 1024, 23.8, 20.2),
                                              (8, 4096, 2048, 4.5, 4.8), (1, 49152, 2048, 14.1, 15.1), (1, 8192, 4096, 6.7, 8.1)])
def test_weight_only_decode_of_a_short_k_takes_the_wavefronts_that_measured_faster(m, n, k, eight, four):
    assert (rules.w4_shape(rules.w4_tile(m, n, k))[2] == 4) == (four < eight)


def shares(units, wavefronts):
    return {units // wavefronts, -(-units // wavefronts)}


def test_gpu_shapes_run_the_main_loop_of_every_split_k_tile():
    """The ring-refill loop runs for the units of a wavefront beyond its ring; the GPU test's shapes give every tile two
    such units or more, and every remainder behind the last whole unit (none, one and two 64-byte steps)."""
    loops, tails = {}, {}
    for m, n, k in SPLIT_MAIN_LOOP:
        tile = rules.split_tile(m, n, k)
        assert tile > 0 and B.cwac_forward_kernel_for(m, n, k, k, k) == B.CWAC_KERNEL_SPLIT_K, (m, n, k)
        _, _, waves, depth = rules.split_shape(tile)
        loops.setdefault(tile, []).append(min(shares(k // 128, waves)) - depth)
        tails.setdefault(tile, set()).add(-(-(k % 128) // 64))
    assert set(loops) == {1, 2, 3, 4}
    assert all(min(v) >= 2 for v in loops.values()), loops
    assert all(tails[t] == {0, 1, 2} for t in loops), tails
    assert any(rules.split_tile(m, n, k) == 4 and n % 16 == 0 for m, n, k in SPLIT_MAIN_LOOP)    # its code-table epilogue


def test_gpu_shapes_run_the_main_loop_of_every_weight_streaming_tile():
    loops = {}
    for m, n, k in W4_MAIN_LOOP:
        tile = rules.w4_tile(m, n, k)
        assert tile >= 0, (m, n, k)
        _, _, waves, depth = rules.w4_shape(tile)
        share = shares(k // 64, waves)
        loops.setdefault(tile, []).append((min(share) - depth, len(share)))
    assert set(loops) == set(range(rules.lib().w4_tiles()))
    assert all(max(v)[0] >= 2 for v in loops.values()), loops
    assert all(max(c for _, c in v) == 2 for v in loops.values()), loops      # wavefronts with shares of unequal length


def test_random_shapes_lie_on_both_sides_of_the_weight_streaming_kernels_limit():
    for m, n, k in ((256, 4096, 128), (512, 2048, 256), (1632, 640, 256)):
        assert rules.w4_tile(m, n, k) >= 0 and rules.w4_tile(m + 1, n, k) == -1


# microseconds measured with cold weights: the 64 x 64 tile kernel, the split-K kernel, 128 x 128 direct-to-LDS tiles
@pytest.mark.parametrize("m,n,k,tile,split,lds", [(640, 2048, 512, 6.64, 7.5, 6.26), (788, 1536, 512, 6.58, 7.39, 5.99),
                                                  (256, 3072, 768, 7.14, 5.92, 7.5), (788, 1280, 1280, 9.9, 8.2, 9.7),
                                                  (256, 5504, 2048, 13.19, 12.3, 11.73), (577, 2048, 2048, 13.2, 11.2, 11.7),
                                                  (2000, 512, 512, 6.0, 7.1, 6.5), (300, 2304, 768, 7.2, 6.0, 7.4),
                                                  (450, 2304, 768, 7.2, 7.6, 7.3), (1280, 1000, 768, 7.62, 8.15, 8.11), (1280, 1024, 768, 7.68, 8.13, 7.55)])
def test_layers_between_the_kernels_take_the_one_that_measured_fastest(m, n, k, tile, split, lds):
    want = min((tile, B.CWAC_KERNEL_GENERIC_64), (split, B.CWAC_KERNEL_SPLIT_K), (lds, B.CWAC_KERNEL_DIRECT_LDS))[1]
    assert B.cwac_forward_kernel_for(m, n, k, k, k) == want


# microseconds measured with cold weights: tiles of 32 and of 16 channels of the weight-streaming kernel
@pytest.mark.parametrize("m,n,k,wide,narrow", [(1, 4096, 11008, 12.0, 8.1), (16, 4096, 4096, 7.0, 5.6), (12, 256, 8192, 8.5, 5.6),
                                               (8, 12288, 4096, 11.2, 9.2), (9, 12288, 4096, 10.9, 12.4), (16, 5120, 2048, 4.7, 5.7),
                                               (8, 5120, 8192, 9.8, 10.7), (4, 6144, 512, 3.5, 3.3), (1, 24576, 1024, 5.8, 7.0),
                                               (8, 14336, 256, 3.5, 4.3), (4, 11008, 4096, 9.8, 8.2), (1, 6144, 2048, 4.57, 4.74), (4, 8192, 4096, 6.05, 6.39),
                                               (4, 5504, 2048, 4.62, 4.71), (8, 4128, 4096, 5.94, 5.76), (1, 4608, 4096, 5.85, 5.76), (8, 8192, 1024, 4.15, 3.91),
                                               (4, 7168, 512, 3.60, 3.36), (8, 11008, 2048, 6.11, 5.35)])
def test_weight_only_decode_takes_the_tile_that_measured_faster(m, n, k, wide, narrow):
    assert rules.w4_tile16(m, n, k) == (narrow < wide)


def test_gpu_shapes_reach_both_tile_widths_of_a_decoding_step():
    from test_gpu_w4_mid_batch import TILES16, WIDE_MAIN_LOOP
    assert all(rules.w4_tile16(*s) for s in TILES16)
    assert not any(rules.w4_tile16(*s) for s in WIDE_MAIN_LOOP)
    assert {rules.w4_tile(*s) for s in WIDE_MAIN_LOOP} == {0, 1, 7}
    # a wavefront's share of the groups exceeds its two slots by a round at least, in shares of two lengths
    assert any(min(shares(k // 128, 8)) >= 3 and len(shares(k // 128, 8)) == 2 and m > 8 for m, n, k in TILES16)
    assert any(min(shares(k // 128, 8)) >= 2 and len(shares(k // 128, 8)) == 2 and m <= 8 for m, n, k in TILES16)


# microseconds per call of a replayed graph: blocks of 128 queries, wide blocks
@pytest.mark.parametrize("batch,heads,tokens,head_dim,narrow,wide",
                         [(8, 12, 257, 64, 11.9, 10.9), (8, 12, 289, 64, 13.0, 11.8), (8, 12, 400, 64, 16.6, 14.3), (4, 12, 785, 64, 26.1, 22.5),
                          (4, 12, 1025, 64, 33.1, 28.7), (1, 12, 4096, 64, 110.1, 94.5), (8, 12, 1025, 64, 58.2, 53.5),
                          (8, 12, 577, 64, 21.1, 32.2), (8, 12, 785, 64, 36.1, 42.2), (32, 12, 400, 64, 39.8, 40.7), (128, 12, 257, 64, 78.7, 103.4),
                          (3, 12, 257, 64, 8.5, 10.1), (2, 12, 1025, 64, 22.6, 27.6), (32, 16, 400, 32, 39.0, 32.9), (1, 16, 4096, 32, 76.4, 67.9),
                          (32, 16, 785, 32, 120.9, 97.0), (128, 16, 400, 32, 141.4, 118.4), (128, 16, 257, 32, 73.0, 71.8),
                          (8, 16, 577, 32, 20.0, 20.2), (32, 16, 257, 32, 21.7, 22.6)])
def test_long_attention_takes_the_query_blocks_that_measured_faster(batch, heads, tokens, head_dim, narrow, wide):
    want = rules.ATTN_CHUNKS_WIDE if wide < narrow else rules.ATTN_CHUNKS
    assert rules.attention_form(batch, heads, tokens, head_dim, False) == want
    assert rules.attention_form(batch, heads, tokens, head_dim, True) == rules.ATTN_CHUNKS


# ... a workgroup per head (or 128 queries), the keys split over a workgroup's wavefronts
@pytest.mark.parametrize("batch,heads,tokens,head_dim,bias,whole,split",
                         [(3, 12, 197, 64, False, 7.6, 5.9), (8, 3, 257, 64, False, 8.4, 6.8), (1, 12, 577, 64, False, 13.4, 9.2),
                          (1, 12, 144, 64, False, 5.9, 5.3), (1, 12, 128, 64, False, 4.6, 4.8), (1, 16, 257, 64, True, 10.2, 7.3),
                          (1, 16, 144, 32, True, 6.0, 4.8), (1, 4, 128, 32, True, 4.83, 4.53), (1, 16, 100, 32, True, 4.75, 4.67),
                          (1, 16, 112, 64, True, 5.32, 5.41), (1, 16, 128, 32, False, 3.87, 4.19)])
def test_attention_of_few_heads_takes_the_form_that_measured_faster(batch, heads, tokens, head_dim, bias, whole, split):
    assert (rules.attention_form(batch, heads, tokens, head_dim, bias) == rules.ATTN_SPLIT) == (split < whole)


def test_row_quantizer_launches_fewer_than_2_to_the_32_threads():
    for k in (1, 3, 4, 256, 512, 516, 1024, 1028, 4096, 4100, 16384, 16388, 100000):
        for vec in (0, 1):
            for asked in (1, 511, 512, 2 ** 24, 2 ** 31 - 1):
                rows, threads = rules.quantize_grid(asked, k, vec)
                assert rows > 0 and (rows + 3) * threads < 2 ** 32, (asked, k, vec)


# microseconds per call of a replayed graph: one wavefront to a row, four
@pytest.mark.parametrize("rows,k,one,four", [(8, 1000, 3.19, 3.03), (64, 1024, 3.30, 3.11), (197, 896, 3.35, 3.16), (197, 640, 3.18, 3.15),
                                             (512, 640, 3.24, 3.33), (1000, 1000, 3.80, 3.90), (4096, 772, 5.21, 6.73)])
def test_row_quantizer_takes_the_wavefronts_that_measured_faster(rows, k, one, four):
    assert (rules.quantize_grid(rows, k, 1)[1] == 256) == (four < one)


# microseconds measured with cold weights: the last round of 512-channel tiles whole, in halves, in quarters of a tile
@pytest.mark.parametrize("m,n,whole,halves,quarters", [(1400, 12288, 190, 169, 164), (3000, 12288, 298, 276, 273), (2048, 11008, 189, 174, 999),
                                                       (2048, 12288, 200, 189, 999)])
def test_weight_only_prefill_cuts_the_last_round_as_measured_fastest(m, n, whole, halves, quarters):
    assert rules.w4_pieces(m, n) == min((whole, 1), (halves, 2), (quarters, 4))[1]


def test_weight_only_prefill_keeps_whole_tiles_in_full_rounds():
    assert [rules.lib().w4_cut(C.c_longlong(t)) for t in (1, 128, 255, 256, 257, 320, 321, 384, 385, 511, 512, 513)] == \
        [1, 1, 1, 1, 4, 4, 2, 2, 1, 1, 1, 4]


def tile_of_block(pid, tiles_m, tiles_n):
    """The kernels' order of tiles (qlinear_common.h): a contiguous range to each of 8 dies, in bands of 8 tile rows."""
    per, rem = divmod(tiles_m * tiles_n, 8)
    at = pid % 8 * per + min(pid % 8, rem) + pid // 8
    band = 8 * tiles_n
    rows = min(tiles_m - at // band * 8, 8)
    return at // band * 8 + at % band % rows, at % band // rows


def test_gpu_shapes_reach_every_piece_of_the_cut_last_round():
    """Halves and quarters; among the cut tiles the last rows' (whole, partial and empty pieces) and the last channels'."""
    from test_gpu_w4_mid_batch import HALVES, QUARTERS
    seen = set()
    for pieces, shapes in ((4, QUARTERS), (2, HALVES)):
        for m, n, k in shapes:
            assert rules.w4_tile(m, n, k) == -1 and rules.w4_pieces(m, n) == pieces
            tiles_m, tiles_n = -(-m // 128), -(-n // 512)
            tiles = tiles_m * tiles_n
            cut = [tile_of_block(i, tiles_m, tiles_n) for i in range(tiles - tiles % 256, tiles)]
            for tm, tn in cut:
                for piece in range(pieces):
                    rows = m - tm * 128 - piece * (128 // pieces)
                    seen.add((pieces, "empty" if rows <= 0 else "partial" if rows < 128 // pieces else "whole"))
                if tn == tiles_n - 1 and n % 512:
                    seen.add((pieces, "shifted"))
    assert seen == {(p, what) for p in (2, 4) for what in ("whole", "partial", "empty", "shifted")}


def test_gpu_shapes_reach_every_attention_form():
    from test_gpu_block import FORMS
    seen = {(rules.attention_form(batch, heads, tokens, d, bias), d, bias) for batch, heads, tokens, d, bias in FORMS}
    assert seen == {(form, d, bias) for form in range(10) for d in (64, 32) for bias in (False, True)
                    if not (bias and form == rules.ATTN_CHUNKS_WIDE)}


# microseconds measured with cold weights: the 64 x 64 tile kernel and a lookup pass, the split-K kernel, 128-token direct-to-LDS tiles
@pytest.mark.parametrize("m,n,k,tile,split,lds", [(591, 1536, 384, 7.3, 5.2, 5.4), (788, 1536, 384, 7.8, 6.6, 5.5), (592, 2048, 512, 8.6, 7.0, 5.8),
                                                  (160, 6656, 768, 10.0, 7.6, 8.3), (250, 5120, 768, 10.1, 8.5, 8.3), (250, 5120, 1024, 11.2, 8.9, 9.3),
                                                  (224, 6656, 1024, 11.3, 9.6, 9.3), (197, 5120, 1280, 12.2, 9.7, 10.8), (250, 6144, 1280, 12.5, 10.8, 10.9),
                                                  (224, 6144, 1536, 13.5, 11.0, 10.2), (255, 8192, 256, 8.3, 8.6, 5.7)])
def test_a_code_table_moves_a_layer_off_the_register_staged_tile_as_measured(m, n, k, tile, split, lds):
    assert rules.table_form(m, n, k) == min((tile, 0), (split, 1), (lds, 2))[1]
