"""Which kernels a product takes (chosen on the host from sizes, types and
alignment; no GPU needed), and the helper that the GPU tests use to make sure
that they run the kernel they are written for."""
import ctypes

import pytest

from paper_2608_01528_amd import gramspace as gsm

FEW, SPLIT, TILES256, SWEEP256, TILES128, SWEEP128 = range(6)
F32, BF16 = gsm.GS_F32, gsm.GS_BF16
PROJECT, RESTORE, BIND, SCORES, WEIGHTS, WINNER = "project", "restore", "bind", "scores", "weights", "winner"
# epilogue, B stored K x N, scores written, argmax asked for
FORMS = {PROJECT: (0, 0, 0, 0), RESTORE: (0, 1, 0, 0), BIND: (1, 1, 0, 0), SCORES: (2, 0, 1, 1),
         WEIGHTS: (3, 0, 0, 0), WINNER: (2, 0, 0, 1)}


def route(form, rows, cols, K, t=F32, out=None, ld=None):
    """Of out (rows x cols) = A (rows x K) B, leading dimensions rounded up to
    16 bytes, or `ld` for the rows of A."""
    epi, b_nn, write, argmax = FORMS[form]
    f = gsm.lib().gs_test_product_route
    f.argtypes = [ctypes.c_int] * 4 + [ctypes.c_int64] * 5 + [ctypes.c_int] * 2
    per = 4 if t == F32 else 8
    up = lambda n: (n + per - 1) // per * per
    return f(t, t if out is None else out, b_nn, epi, rows, cols, K, ld or up(K), up(cols if b_nn else K), write,
             argmax)


@pytest.mark.parametrize("t,short", [(F32, (1, 3)), (BF16, (1, 4, 7))], ids=["f32", "bf16"])
def test_less_than_16_bytes_of_k(t, short):
    """Nothing to share out: 128 x 128 tiles while they fit one round, and for
    bf16 output with cut columns until a round of the large ones fills the CUs."""
    for K in short:
        for form in (PROJECT, RESTORE, SCORES, WEIGHTS):
            assert route(form, 1000, 300, K, t) == TILES128
            assert route(form, 8 * 256, 8 * 256 - 1, K, t, out=F32) == TILES128
            assert route(form, 8 * 256 + 1, 8 * 256 - 1, K, t, out=F32) == TILES256
            assert route(form, 16 * 256, 16 * 256 - 1, K, t) == TILES256
            assert route(form, 16 * 256, 16 * 256, K, t, ld=K + 1 + K % 2) == TILES128      # odd rows
        for form in (PROJECT, RESTORE):
            assert route(form, 256, 512, K, t, out=BF16) == TILES256
            assert route(form, 257, 512, K, t, out=BF16) == TILES128
            assert route(form, 20000, 256, K, t, out=BF16) == TILES256
            assert route(form, 9000, 1000, K, t, out=BF16) == TILES128
    assert route(PROJECT, 1000, 300, 16, t) == SPLIT


@pytest.mark.parametrize("t", [F32, BF16], ids=["f32", "bf16"])
def test_rows_that_the_large_tiles_cannot_take(t):
    for form in (PROJECT, RESTORE, BIND, SCORES, WEIGHTS):
        for rows in (100, 16384, 262144):
            assert route(form, rows, 1000, 901, t, ld=901) == SPLIT         # no 16-byte alignment
    assert route(BIND, 65536, 4096, 1000, t, out=BF16) == SPLIT             # factors rounded once only
    assert route(PROJECT, 100, 300, 512, t, ld=1 << 22) == TILES128         # beyond 32-bit offsets
    assert route(WINNER, 100, 300, 512, t) == SWEEP128
    assert route(WINNER, 65536, 300, 512, t) == SWEEP256
    assert route(WINNER, 65536, 256, 512, t) == TILES256
    assert route(SCORES, 16, 100, 512, t) == FEW


@pytest.mark.parametrize("t", [F32, BF16], ids=["f32", "bf16"])
def test_full_batches_take_the_large_tiles(t):
    assert route(PROJECT, 65536, 256, 8192, t) == TILES256
    assert route(RESTORE, 65536, 4096, 1000, t) == TILES256
    assert route(SCORES, 65536, 256, 256, t) == TILES256
    assert route(WEIGHTS, 262144, 2048, 1843, t) == TILES256
    assert route(BIND, 16384, 4096, 1000, t, out=F32) == TILES256
    assert route(PROJECT, 777, 203, 4096, t) == SPLIT
