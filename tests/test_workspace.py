"""The context's workspace as a function of the batch: more rows never ask for less, so one call at the largest batch is
enough before calls are recorded into a graph.  The library's own size functions, called without a GPU."""
import ctypes as C

import pytest

from paper_2605_13907_amd import binding as B


def sizes():
    lib = B._lib()
    logprob = lib["_ZN3ais21lm_head_logprob_bytesExii"]          # lm_head_logprob_bytes(rows, vocab, compute units)
    dlogits = lib["_ZN3ais21lm_grad_dlogits_bytesExxxi"]         # lm_grad_dlogits_bytes(rows, vocab, asked chunk, units)
    chunk = lib["_ZN3ais13lm_grad_chunkExxxi"]
    logprob.argtypes, logprob.restype = [C.c_longlong, C.c_int, C.c_int], C.c_size_t
    dlogits.argtypes, dlogits.restype = [C.c_longlong, C.c_longlong, C.c_longlong, C.c_int], C.c_size_t
    chunk.argtypes, chunk.restype = [C.c_longlong, C.c_longlong, C.c_longlong, C.c_int], C.c_longlong
    return logprob, dlogits, chunk


def chunks(rows, vocab, n_cus):
    """Most chunks that a batch of so many rows is split into: at least 64, two work items per compute unit."""
    blocks = (rows + 255) // 256
    return min((vocab + 255) // 256, max(64, (2 * n_cus + blocks - 1) // blocks))


@pytest.mark.parametrize("n_cus", [256, 64, 304])
@pytest.mark.parametrize("vocab", [1, 3000, 20_000, 50_257, 151_936])
def test_more_rows_never_need_less(vocab, n_cus):
    logprob, dlogits, _ = sizes()
    rows = list(range(1, 5200, 1 if vocab > 50_257 else 7)) + [8191, 8192, 8193, 41_643, 1 << 20]
    last = 0, 0
    for n in rows:
        now = logprob(n, vocab, n_cus), dlogits(n, vocab, 0, n_cus)
        assert now[0] >= 4 * n * (2 * chunks(n, vocab, n_cus) + 3) + 256, (n, "what the call itself lays out")
        assert now[0] >= last[0] and now[1] >= last[1], (n, last, now)
        last = now


@pytest.mark.parametrize("vocab", [1, 8192, 50_257, 151_936])
def test_dlogits_hold_whole_chunks(vocab):
    _, dlogits, chunk = sizes()
    for n in (1, 255, 256, 700, 2000, 4095, 4096, 41_643):
        for asked in (0, 256, 8192, 65_536):
            width = chunk(n, vocab, asked, 256)
            assert width % 256 == 0 and 0 < width < vocab + 256 and (asked == 0 or width <= asked)
            assert dlogits(n, vocab, asked, 256) >= 2 * n * width
            if asked:
                assert dlogits(n, vocab, asked, 256) == 2 * n * width
    assert chunk(4096, 151_936, 0, 256) == 8192 and chunk(700, 151_936, 0, 256) == 170 * 256


@pytest.mark.parametrize("n_cus", [256, 64])
def test_wide_chunks_fill_one_round(n_cus):
    """Where few rows take wide chunks, the recomputation has at most a work item of two tiles per compute unit."""
    _, _, chunk = sizes()
    for rows in range(1, 5000, 61):
        tiles, blocks = chunk(rows, 1 << 20, 0, n_cus) // 256, (rows + 255) // 256
        assert tiles == 32 or (blocks <= 12 and blocks * ((tiles + 1) // 2) <= n_cus), (rows, tiles)
