"""Bit-exact GEMM parity: Eq. (3) and Eq. (10) on operands whose every partial sum is exact.

Weights are non-zero integers of magnitude at most 15 (stored exactly in bf16 / fp32) and every token
row holds at most four non-zero entries from {-2, -1, 1, 2}, placed so that over the tokens every
contraction index is hit.  Every product is an integer, every sum of at most four of them has magnitude
at most 120, so fp32 accumulation in any order is exact and the bf16 output (integers up to 256) is
exact: the kernels' outputs must EQUAL the float64 oracle, element for element.  One dropped, doubled
or misplaced product -- a wrong index nibble, a wrong slot, a wrong column of g(Y)[:, P], a row tile or
stage read from the wrong place -- changes some output by at least 1.

The shapes select every GEMM kernel family of the library in both directions (named beside each case),
with the permutation and with the identity.
"""
import numpy as np
import pytest

import oracle
import paper_2302_06058_amd as bm
from paper_2302_06058_amd import synth
from helpers import to_dev, i32_dev, words, from_dev_f64

pytestmark = pytest.mark.gpu


def int_weights(I, J, rng):
    mag = rng.integers(1, 16, size=(I, J))
    sign = rng.integers(0, 2, size=(I, J)) * 2 - 1
    return (mag * sign).astype(np.float32)


def sparse_rows(T, C, rng):
    """T x C, four non-zeros from {-2, -1, 1, 2} per row; the rows walk over all C columns in an order
    drawn once, so with 4 T >= C every column is non-zero in some row."""
    a = np.zeros((T, C), dtype=np.float32)
    order = rng.permutation(C)
    vals = np.array([-2, -1, 1, 2], dtype=np.float32)
    for q in range(4):
        cols = order[(4 * np.arange(T) + q) % C]
        a[np.arange(T), cols] = vals[rng.integers(0, 4, size=T)]
    return a


def exact_layer(I, J, T, N, M, dtype, seed, perm=True):
    import torch
    rng = np.random.default_rng(seed)
    Wh = synth.store(int_weights(I, J, rng), dtype)
    W64 = synth.to_f64(Wh, dtype)
    Xh = synth.store(sparse_rows(T, J, rng), dtype)
    dYh = synth.store(sparse_rows(T, I, rng), dtype)
    assert (Xh != 0).any(axis=0).all() and (dYh != 0).any(axis=0).all()      # every contraction index is exercised
    P_h = rng.permutation(I).astype(np.int32) if perm else None
    W, X, dY = to_dev(Wh, dtype), to_dev(Xh, dtype), to_dev(dYh, dtype)
    P = i32_dev(P_h) if perm else None
    B, vals, index = bm.bimask_forward_mask_compress(W, N, M)
    Bbar, vb, ib = bm.bimask_backward_mask_compress(W, N, M, B, P)
    B_o = oracle.forward_mask(W64, N, M)
    Bbar_o, _ = oracle.backward_mask(W64, B_o, P_h, N, M)
    assert (words(B) == oracle.pack_bits(B_o)).all() and (words(Bbar) == oracle.pack_bits(Bbar_o)).all()
    Y = bm.bimask_sparse_gemm_fwd(X, vals, index, I, J, N, M)
    dX = bm.bimask_sparse_gemm_bwd(dY, P, vb, ib, I, J, N, M)
    torch.cuda.synchronize()
    Y_o = oracle.gemm_fwd(synth.to_f64(Xh, dtype), W64, B_o)
    dX_o = oracle.gemm_bwd(synth.to_f64(dYh, dtype), W64, Bbar_o, P_h)
    assert np.abs(Y_o).max() <= 120 and np.abs(dX_o).max() <= 120 and np.abs(Y_o).max() > 0 and np.abs(dX_o).max() > 0
    gy, gx = from_dev_f64(Y, dtype), from_dev_f64(dX, dtype)
    bad_y, bad_x = np.argwhere(gy != Y_o), np.argwhere(gx != dX_o)
    assert bad_y.shape[0] == 0, f"forward: {bad_y.shape[0]} wrong outputs, first at (t, i) = {bad_y[0].tolist()}"
    assert bad_x.shape[0] == 0, f"backward: {bad_x.shape[0]} wrong outputs, first at (t, j) = {bad_x[0].tolist()}"


# (I, J, T): forward kernel, backward kernel with a permutation (checked without a GPU in test_dispatch.py).  "a x b": the streaming kernel
# with tiles of a weight rows x b tokens, "split": its contraction split over groups of wavefronts
SP24_SHAPES = {
    (64, 148, 300): ("narrow", "narrow"),                                           # 296-byte rows both ways
    (256, 64, 300): ("narrow_rows", "coltile"),                                     # two sibling wavefronts forward
    (224, 64, 150): ("narrow_rows", "coltile"),                                     # 7 row tiles over 2 x 4
    (64, 512, 600): ("narrow_rows", "resident 256 x 64"),
    (160, 128, 200): ("narrow_rows", "coltile"),                                    # 5 row tiles
    (128, 256, 700): ("128 x 64", "narrow_rows"),                                   # two sibling wavefronts with the fused gather
    (64, 128, 200): ("narrow_rows", "narrow_rows"),
    (32, 128, 200): ("narrow_rows", "narrow_rows"),
    (32, 256, 200): ("narrow_rows", "narrow_rows"),
    (32, 384, 200): ("narrow_rows", "resident 256 x 64"),                           # 3 stages
    (32, 512, 200): ("narrow_rows", "resident 256 x 64"),                           # 4 stages
    (96, 128, 200): ("narrow_rows", "narrow_rows"),
    (512, 128, 300): ("resident 256 x 64", "coltile"),                              # one stage / 4 stages
    (1024, 192, 300): ("split 64 x 32", "coltile"),                                 # contraction ends inside a stage
    (256, 124, 300): ("narrow", "resident 128 x 32"),                               # 124 columns
    (124, 128, 300): ("narrow", "resident 128 x 32"),                               # contraction 124
    (512, 128, 16400): ("resident 256 x 64", "coltile"),
    (512, 256, 16400): ("wide", "coltile"),
    (384, 384, 16400): ("wide", "coltile"),
    (512, 512, 16400): ("wide", "coltile"),
    (1536, 384, 400): ("split 64 x 64", "coltile"),                                 # 12 stages
    (2048, 512, 600): ("128 x 64", "coltile"),                                      # 16 stages
    (64, 576, 500): ("split 64 x 32", "resident 256 x 64"),                         # contraction ends inside a stage
    (64, 576, 66000): ("64 x 64", "resident 256 x 64 persistent"),                  # contraction ends inside a stage
    (64, 640, 9000): ("64 x 64", "resident 256 x 64"),
    (64, 644, 9000): ("64 x 64", "resident 256 x 64"),                              # 4-byte rows
    (256, 576, 66000): ("256 x 128", "wide"),                                       # contraction ends inside a stage
    (256, 2304, 2400): ("split 64 x 64", "coltile"),
    (384, 640, 700): ("split 64 x 32", "coltile"),
    (384, 640, 2800): ("128 x 64", "coltile"),                                      # 384 rows = 1.5 tiles of 256
    (384, 648, 2800): ("128 x 64", "coltile"),                                      # ... contraction ends inside a stage
    (384, 644, 2800): ("128 x 64", "resident 256 x 64"),                            # ... 4-byte rows
    (256, 640, 12500): ("256 x 64", "coltile"),
    (256, 648, 12500): ("256 x 64", "coltile"),                                     # contraction ends inside a stage
    (256, 644, 12500): ("256 x 64", "resident 256 x 64"),                           # 4-byte rows
    (512, 644, 12200): ("256 x 128", "resident 256 x 64"),                          # 4-byte rows
    (2100, 64, 600): ("resident 256 x 64", "gather, split 64 x 32"),                # 4-byte rows, 17 stages
    (1024, 1028, 300): ("split 64 x 32", "gather, split 64 x 32"),                  # 4-byte rows
    (2560, 1024, 2600): ("256 x 128", "gather, 256 x 64"),
    (4096, 2048, 8200): ("big", "gather, 256 x 128"),                               # 8 x 65 tiles, the last token tile ragged
    (3200, 1152, 22037): ("big", "gather, big"),                                    # 6.25 and 2.25 weight tiles, ragged last token tile
    (1024, 1152, 65600): ("big", "coltile"),                                        # two weight tiles, 513 token tiles (65 per XCD, the last run shorter)
    (4352, 256, 2051): ("resident 256 x 64", "gather, split 64 x 64"),              # four token rows interleaved per gather tile (8.5 KB rows), ragged last tile
    (8704, 128, 2305): ("resident 256 x 64", "gather, split 64 x 32"),              # two token rows per gather tile (17 KB rows), one row in the last tile
    (4224, 1024, 11200): ("big", "gather, 256 x 128"),                              # nine weight tiles (the last with 128 rows) x 88 token tiles, 99 per XCD on 32 workgroups
}


@pytest.mark.parametrize("I,J,T", list(SP24_SHAPES))
@pytest.mark.parametrize("perm", [True, False], ids=["perm", "identity"])
def test_sparse_core_gemms_are_exact_on_integer_operands(I, J, T, perm):
    exact_layer(I, J, T, 2, 4, synth.BF16, 7000 + I + J + T, perm=perm)


OTHER_RATIOS, OTHER_RATIO_SHAPES = [(1, 4), (2, 8), (1, 16)], [(256, 384, 500), (64, 128, 200)]


@pytest.mark.parametrize("N,M", OTHER_RATIOS)
def test_other_ratios_on_the_sparse_cores_are_exact(N, M):
    for q, (I, J, T) in enumerate(OTHER_RATIO_SHAPES):
        exact_layer(I, J, T, N, M, synth.BF16, 7100 + 100 * q + M + N)


# dense operand: streaming tiles 64 x 64, 128 x 64 and 256 x 128 with whole and ragged stages (the split tiles are below); column tiles
# with contractions of 2 to 9 stages
DENSE_SHAPES = [(384, 384, 500), (1536, 384, 600), (384, 1536, 1600), (136, 1032, 1100), (64, 72, 80), (1152, 384, 16400),
                (64, 640, 9000), (64, 648, 9000), (384, 640, 2800), (384, 648, 2800), (512, 640, 12200), (512, 648, 12200),
                (256, 128, 300), (384, 256, 700), (520, 512, 300), (648, 256, 300)]


@pytest.mark.parametrize("I,J,T", DENSE_SHAPES)
@pytest.mark.parametrize("perm", [True, False], ids=["perm", "identity"])
def test_dense_core_gemms_4of8_are_exact(I, J, T, perm):
    exact_layer(I, J, T, 4, 8, synth.BF16, 7300 + I + J, perm=perm)


# few output tiles: the contraction split over groups of wavefronts (64 x 32 tiles by 4, 64 x 64 by 2): two stages and three, whole and
# partial last steps, ragged rows, tokens and stages, token rows of 16-byte pitch and of 8-byte pitch
SPLIT_SHAPES = [(68, 132, 35), (64, 260, 70), (136, 136, 37), (192, 648, 165), (512, 1152, 290), (1000, 520, 251),
                (64, 4096, 1030), (1024, 1024, 1000), (960, 904, 1001), (900, 908, 1023)]


@pytest.mark.parametrize("I,J,T", SPLIT_SHAPES)
@pytest.mark.parametrize("perm", [True, False], ids=["perm", "identity"])
def test_split_contractions_are_exact(I, J, T, perm):
    exact_layer(I, J, T, 2, 4, synth.BF16, 7700 + I + J, perm=perm)
    if I % 8 == 0 and J % 8 == 0:
        exact_layer(I, J, T, 4, 8, synth.BF16, 7800 + I + J, perm=perm)


# Backward on column tiles: 1, 2, 3 row tiles per wavefront, up to 32 and up to 64 tokens, few and many pieces per fetching thread;
# contractions of 2 (136 terms) to 16 stages, even and odd, ragged in the last one; one tile per workgroup and up to seven, the
# last one short; a last workgroup and a last row of four tokens that are not full; pieces of weight rows over the grid; 8 outputs
COLTILE_SHAPES = [(136, 8, 37), (136, 8, 8200), (136, 136, 8200), (136, 264, 8200), (160, 392, 2049), (144, 136, 5001), (160, 264, 5001),
                  (264, 264, 5001), (264, 264, 8200), (384, 136, 1101), (640, 64, 2050), (648, 8, 12301), (648, 520, 5001), (648, 776, 5001),
                  (1000, 264, 3000), (1152, 384, 16390), (1536, 264, 3000), (1536, 776, 2049), (1800, 136, 2049), (2048, 512, 8203), (512, 128, 60001)]


@pytest.mark.parametrize("I,J,T", COLTILE_SHAPES)
@pytest.mark.parametrize("N,M", [(2, 4), (4, 8)])
def test_column_tiles_are_exact(I, J, T, N, M):
    exact_layer(I, J, T, N, M, synth.BF16, 7950 + I + J)


# Wavefront-private tiles: rows in 16-byte pieces, 1 to 5 row tiles (6 to 8 on two wavefronts), 1 to 4 stages, every piece and row tile
# whole or ragged (whole ones with constant steps over the pieces: 64, 128, 256 terms on multiples of 32 columns); rows that are no multiple of 16 bytes; three token rows in the last tile; more tiles than wavefronts on the chip
NARROW_SHAPES = [(24, 56, 67), (56, 24, 67), (64, 88, 131), (88, 64, 131), (48, 120, 99), (120, 48, 99), (56, 152, 163), (152, 56, 163),
                 (24, 120, 99), (120, 24, 99), (88, 120, 131), (120, 88, 131), (152, 120, 163), (120, 152, 163), (176, 56, 195), (56, 248, 259),
                 (24, 248, 259), (24, 376, 387), (56, 376, 387), (24, 504, 515), (56, 504, 515), (104, 200, 16403),
                 (64, 64, 99), (128, 64, 131), (64, 128, 131), (128, 128, 131), (64, 256, 259), (256, 64, 32771),
                 (28, 64, 99), (28, 256, 259), (28, 384, 387), (28, 512, 515), (60, 256, 259), (60, 384, 387), (60, 512, 515), (92, 128, 131), (156, 128, 163),
                 (60, 64, 99), (56, 24, 140003), (88, 120, 140003), (64, 64, 140003),
                 (32, 64, 99), (64, 32, 99), (96, 64, 131), (64, 96, 131), (64, 160, 163), (160, 64, 163), (64, 192, 195), (96, 128, 131), (128, 96, 131),
                 (160, 128, 163), (128, 160, 163), (128, 192, 195), (32, 128, 99), (128, 32, 99), (32, 256, 259), (256, 32, 3103), (64, 256, 3075), (256, 64, 3075),
                 (160, 32, 65539), (136, 8, 65539), (128, 256, 16387), (96, 256, 98307)]


@pytest.mark.parametrize("I,J,T", NARROW_SHAPES)
@pytest.mark.parametrize("perm", [True, False], ids=["perm", "identity"])
def test_wavefront_private_tiles_are_exact(I, J, T, perm):
    exact_layer(I, J, T, 2, 4, synth.BF16, 8050 + I + J, perm=perm)


# Wide outputs: tiles of 64 and of 128 tokens, one piece of weight rows and several, contractions that end inside a stage (1 to 4
# stages), row tiles and wavefront tiles that are not full, a last token tile of a few rows, fewer wavefront tiles than wavefronts
WIDE_SHAPES = [(1032, 264, 4099), (1536, 384, 25003), (1096, 392, 9001), (2056, 504, 5003), (392, 1544, 17003), (504, 1096, 20011), (512, 4608, 3139),
               (640, 136, 5003), (288, 136, 16401), (160, 544, 16403),
               (264, 136, 65500), (192, 992, 16200), (384, 448, 16700)]     # just outside: resident (many tokens; rows that end inside a line), streaming
WIDE_DENSE_SHAPES = [(264, 104, 4099), (1032, 200, 9001), (1536, 384, 25003), (104, 520, 4101), (320, 1032, 9001), (136, 1096, 30011),
                     (1056, 64, 2051), (72, 544, 4100)]


@pytest.mark.parametrize("I,J,T,N,M", [(*s, 2, 4) for s in WIDE_SHAPES] + [(*s, 4, 8) for s in WIDE_DENSE_SHAPES])
def test_wide_outputs_are_exact(I, J, T, N, M):
    exact_layer(I, J, T, N, M, synth.BF16, 8150 + I + J)


def test_tiles_of_256_x_64_stay_exact_where_the_tiles_fill_the_chip():
    exact_layer(256, 640, 12500, 2, 4, synth.BF16, 7900)


F32_SMALL = [(64, 128, 40), (136, 264, 300)]


@pytest.mark.parametrize("N,M", [(2, 4), (4, 8)])
def test_fp32_gemms_are_exact(N, M):
    for q, (I, J, T) in enumerate(F32_SMALL):
        exact_layer(I, J, T, N, M, synth.F32, 7400 + 100 * q + M)


# 16 x 16 tiles; 1 / 2 / 4 / 8 / 16 wavefronts by contraction length and tile count; gather in the token loads or as a pass; 64 weight
# rows per workgroup where there are many tiles (the last workgroup with 1 and 3 row tiles, the last row tile half filled)
F32_SHAPES = [(8, 8, 5), (16, 136, 37), (40, 264, 70), (520, 24, 131), (264, 520, 1040), (24, 136, 16400),
              (136, 56, 37), (72, 40, 50), (104, 48, 20000), (72, 136, 33000), (24, 136, 60000)]


@pytest.mark.parametrize("I,J,T", F32_SHAPES)
@pytest.mark.parametrize("N,M", [(2, 4), (4, 8)])
@pytest.mark.parametrize("perm", [True, False], ids=["perm", "identity"])
def test_fp32_tiles_and_contraction_splits_are_exact(I, J, T, N, M, perm):
    exact_layer(I, J, T, N, M, synth.F32, 7600 + I + J, perm=perm)


BOTH = (True, False)                                     # with a permutation, with the identity


def exact_products():
    """(I, J, T, N, M, dtype, permutations) of every layer above: one forward product, a backward product for each entry of the last."""
    for shapes, ratios, dtype, perms in (
            (SP24_SHAPES, [(2, 4)], synth.BF16, BOTH), (OTHER_RATIO_SHAPES, OTHER_RATIOS, synth.BF16, BOTH[:1]), (DENSE_SHAPES, [(4, 8)], synth.BF16, BOTH),
            (SPLIT_SHAPES, [(2, 4)], synth.BF16, BOTH), ([s for s in SPLIT_SHAPES if s[0] % 8 == 0 and s[1] % 8 == 0], [(4, 8)], synth.BF16, BOTH),
            (COLTILE_SHAPES, [(2, 4), (4, 8)], synth.BF16, BOTH[:1]), (NARROW_SHAPES, [(2, 4)], synth.BF16, BOTH), (WIDE_SHAPES, [(2, 4)], synth.BF16, BOTH[:1]),
            (WIDE_DENSE_SHAPES, [(4, 8)], synth.BF16, BOTH[:1]), (F32_SMALL, [(2, 4), (4, 8)], synth.F32, BOTH[:1]), (F32_SHAPES, [(2, 4), (4, 8)], synth.F32, BOTH)):
        for shape in shapes:
            for ratio in ratios:
                yield *shape, *ratio, dtype, perms


@pytest.mark.parametrize("I,J,T", [(40, 72, 37), (72, 40, 50), (264, 136, 300), (136, 72, 33000)])
@pytest.mark.parametrize("N,M", [(2, 4), (4, 8)])
def test_fp32_rows_at_any_pitch(I, J, T, N, M):
    """Token rows that start on 16 bytes and on 4, in wider buffers: what the packed call gives, and the padding untouched."""
    import torch
    rng = np.random.default_rng(7670 + I)
    W = to_dev(synth.store(int_weights(I, J, rng), synth.F32), synth.F32)
    X = to_dev(synth.store(sparse_rows(T, J, rng), synth.F32), synth.F32)
    dY = to_dev(synth.store(sparse_rows(T, I, rng), synth.F32), synth.F32)
    P = i32_dev(rng.permutation(I).astype(np.int32))
    B, v, x = bm.bimask_forward_mask_compress(W, N, M)
    Y = bm.bimask_sparse_gemm_fwd(X, v, x, I, J, N, M)
    for perm in (P, None):
        _, vb, xb = bm.bimask_backward_mask_compress(W, N, M, B, perm)
        dX = bm.bimask_sparse_gemm_bwd(dY, perm, vb, xb, I, J, N, M)
        for at, extra in ((4, 8), (1, 3)):
            wide = lambda a, fill: torch.full((T, a + extra), fill, dtype=torch.float32, device=W.device)
            Xw, dYw, Yw, dXw = wide(J, float("nan")), wide(I, float("nan")), wide(I, 3.0), wide(J, 3.0)
            Xw[:, at:at + J], dYw[:, at:at + I] = X, dY
            bm.bimask_sparse_gemm_fwd(Xw[:, at:at + J], v, x, I, J, N, M, Y=Yw[:, at:at + I])
            bm.bimask_sparse_gemm_bwd(dYw[:, at:at + I], perm, vb, xb, I, J, N, M, dX=dXw[:, at:at + J])
            for out, want, c in ((Yw, Y, I), (dXw, dX, J)):
                assert torch.equal(out[:, at:at + c], want)
                assert bool((out[:, :at] == 3.0).all()) and bool((out[:, at + c:] == 3.0).all())


# fp32 with the gather in the token loads and dense bf16 weights in natural order read dY itself while dX is written: dX on top of
# dY (in place, and one row further down in the same buffer) has to give what a separate output gives
@pytest.mark.parametrize("C,T,N,M,dtype", [(64, 70, 2, 4, synth.F32), (40, 100, 4, 8, synth.F32), (64, 200, 4, 8, synth.BF16),
                                           (128, 1000, 3, 4, synth.BF16), (2056, 2300, 4, 8, synth.BF16)])
def test_backward_product_in_place(C, T, N, M, dtype):
    import torch
    rng = np.random.default_rng(7660 + C)
    W = to_dev(synth.store(int_weights(C, C, rng), dtype), dtype)
    dY = to_dev(synth.store(sparse_rows(T, C, rng), dtype), dtype)
    P = i32_dev(rng.permutation(C).astype(np.int32))
    B = bm.bimask_forward_mask(W, N, M)
    _, vb, ib = bm.bimask_backward_mask_compress(W, N, M, B, P)
    want = bm.bimask_sparse_gemm_bwd(dY, P, vb, ib, C, C, N, M)
    assert float(want.float().abs().max()) > 0
    for down in (0, 1):
        buf = torch.zeros((T + 1, C), dtype=dY.dtype, device=dY.device)
        buf[:T] = dY
        bm.bimask_sparse_gemm_bwd(buf[:T], P, vb, ib, C, C, N, M, dX=buf[down:T + down])
        assert torch.equal(buf[down:T + down], want), (C, T, down)


def test_fp32_outputs_beyond_2_to_the_32_elements():
    """2^24 output tiles of 16 x 16 and more (256 work-items each: beyond what one dimension of a launch counts): the first and
    the last token rows and the ones around the 2^32nd output equal the product of these rows alone."""
    import torch
    I, J, T = 4096, 8, (1 << 20) + 21
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of free device memory")
    rng = np.random.default_rng(7650)
    W = to_dev(synth.store(int_weights(I, J, rng), synth.F32), synth.F32)
    X = to_dev(synth.store(sparse_rows(T, J, rng), synth.F32), synth.F32)
    _, vals, index = bm.bimask_forward_mask_compress(W, 2, 4)
    Y = bm.bimask_sparse_gemm_fwd(X, vals, index, I, J, 2, 4, Y=torch.full((T, I), -777.0, device=X.device))
    for a, b in ((0, 64), ((1 << 19) - 32, (1 << 19) + 32), ((1 << 20) - 48, (1 << 20) + 16), (T - 40, T)):
        part = bm.bimask_sparse_gemm_fwd(X[a:b].contiguous(), vals, index, I, J, 2, 4)
        assert float(part.abs().max()) > 0 and torch.equal(Y[a:b], part), (a, b)
    assert bool((Y != -777.0).all())
    del Y
    torch.cuda.empty_cache()


def test_large_shapes_with_padded_leading_dimensions():
    """The 512 x 128 forward kernel and the row-interleaved gather of the backward pass on activations whose rows
    are longer than the matrices (ldx > J, lddy > I, ldy > I, lddx > J): the outputs must equal those of the
    packed call (which the exact tests above compare with the oracle), and the padding must stay untouched."""
    import torch
    I, J, T, pad = 4096, 1024, 16400, 8
    rng = np.random.default_rng(515)
    Wh = synth.store(int_weights(I, J, rng), synth.BF16)
    Xh = synth.store(sparse_rows(T, J, rng), synth.BF16)
    dYh = synth.store(sparse_rows(T, I, rng), synth.BF16)
    W, X, dY = to_dev(Wh, synth.BF16), to_dev(Xh, synth.BF16), to_dev(dYh, synth.BF16)
    P = i32_dev(rng.permutation(I).astype(np.int32))
    B, vals, index = bm.bimask_forward_mask_compress(W, 2, 4)
    _, vb, ib = bm.bimask_backward_mask_compress(W, 2, 4, B, P)
    Y = bm.bimask_sparse_gemm_fwd(X, vals, index, I, J, 2, 4)
    dX = bm.bimask_sparse_gemm_bwd(dY, P, vb, ib, I, J, 2, 4)
    fill = -3.0
    Xp = torch.full((T, J + pad), fill, dtype=torch.bfloat16, device=X.device)
    dYp = torch.full((T, I + pad), fill, dtype=torch.bfloat16, device=X.device)
    Xp[:, :J], dYp[:, :I] = X, dY
    Yp = torch.full((T, I + pad), fill, dtype=torch.bfloat16, device=X.device)
    dXp = torch.full((T, J + pad), fill, dtype=torch.bfloat16, device=X.device)
    bm.bimask_sparse_gemm_fwd(Xp[:, :J], vals, index, I, J, 2, 4, Y=Yp[:, :I])
    bm.bimask_sparse_gemm_bwd(dYp[:, :I], P, vb, ib, I, J, 2, 4, dX=dXp[:, :J])
    torch.cuda.synchronize()
    assert torch.equal(Yp[:, :I], Y) and torch.equal(dXp[:, :J], dX)
    assert bool((Yp[:, I:] == fill).all()) and bool((dXp[:, J:] == fill).all())
    assert float(Y.float().abs().max()) > 0 and float(dX.float().abs().max()) > 0


# dX on dY, same first element and pitch, in calls that need no workspace: no workgroup may write a token row that another one still
# has to read (few tokens, where the weight rows are cut over the grid otherwise; wavefront-private tiles; more columns than dY has)
IN_PLACE_SHAPES = [(384, 384, 9001, 2, 4), (384, 384, 17003, 2, 4), (384, 384, 9001, 4, 8), (264, 264, 5003, 4, 8), (512, 512, 9001, 4, 8),
                   (1032, 456, 5003, 2, 4), (520, 392, 9001, 2, 4), (384, 384, 5000, 2, 4), (512, 512, 8192, 2, 4), (264, 264, 8000, 2, 4),
                   (64, 256, 3000, 2, 4), (128, 176, 777, 2, 4), (256, 64, 40000, 2, 4), (260, 388, 1000, 2, 4), (512, 2304, 100, 2, 4)]


@pytest.mark.parametrize("I,J,T,N,M", IN_PLACE_SHAPES)
def test_fused_gather_in_place(I, J, T, N, M):
    import torch
    rng = np.random.default_rng(7665 + I + T)
    W = to_dev(synth.store(int_weights(I, J, rng), synth.BF16), synth.BF16)
    dY = to_dev(synth.store(sparse_rows(T, I, rng), synth.BF16), synth.BF16)
    P = i32_dev(rng.permutation(I).astype(np.int32))
    _, vb, ib = bm.bimask_backward_mask_compress(W, N, M, bm.bimask_forward_mask(W, N, M), P)
    want = bm.bimask_sparse_gemm_bwd(dY, P, vb, ib, I, J, N, M)
    buf = torch.full((T, max(I, J)), 3.0, dtype=torch.bfloat16, device=W.device)
    buf[:, :I] = dY
    bm.bimask_sparse_gemm_bwd(buf[:, :I], P, vb, ib, I, J, N, M, dX=buf[:, :J])
    assert torch.equal(buf[:, :J], want) and torch.equal(buf[:, J:], dY[:, J:])


# dX beside dY in the rows of one buffer: no byte in common, so the way of separate buffers
@pytest.mark.parametrize("I,J,T,N,M", [(384, 384, 17003, 2, 4), (256, 64, 40000, 2, 4), (1152, 384, 5003, 2, 4), (384, 1536, 5003, 4, 8), (128, 256, 3000, 2, 4)])
def test_backward_product_beside_its_input(I, J, T, N, M):
    import torch
    rng = np.random.default_rng(7680 + I + T)
    W = to_dev(synth.store(int_weights(I, J, rng), synth.BF16), synth.BF16)
    dY = to_dev(synth.store(sparse_rows(T, I, rng), synth.BF16), synth.BF16)
    P = i32_dev(rng.permutation(I).astype(np.int32))
    _, vb, ib = bm.bimask_backward_mask_compress(W, N, M, bm.bimask_forward_mask(W, N, M), P)
    want = bm.bimask_sparse_gemm_bwd(dY, P, vb, ib, I, J, N, M)
    buf = torch.full((T, I + J), float("nan"), dtype=torch.bfloat16, device=W.device)
    buf[:, :I] = dY
    bm.bimask_sparse_gemm_bwd(buf[:, :I], P, vb, ib, I, J, N, M, dX=buf[:, I:])
    assert torch.equal(buf[:, I:], want) and torch.equal(buf[:, :I], dY)
