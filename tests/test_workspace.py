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


class Room(C.Structure):
    _fields_ = [("chunk", C.c_longlong), ("w", C.c_int), ("h", C.c_int)] + [(n, C.c_size_t) for n in (
        "plan", "mask", "index", "pos", "hidden", "dhidden", "dweight", "end", "all")]


def room():
    f = B._lib()["_ZN3ais12lm_grad_roomExxxxxii"]        # lm_grad_room(rows, rows gone through, d_model, vocab, asked chunk, units, roomy)
    f.argtypes, f.restype = [C.c_longlong] * 5 + [C.c_int] * 2, Room
    return f


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


@pytest.mark.parametrize("n_cus", [256, 64, 304])
@pytest.mark.parametrize("asked", [0, 256, 1024, 1536, 1792, 4096, 8192, 65_536])
def test_gradient_arrays_lie_inside_what_is_asked_for(asked, n_cus):
    """Every array of the gradient call begins where the one before it ends or later and ends inside the workspace, the
    parts of both sums among them, over many rows, widths, vocabularies and chunks, with and without a row list."""
    f = room()
    split = 0
    for rows in (1, 64, 300, 2000, 3000, 4096, 5000, 12_000, 16_384, 41_643):
        for d in (32, 64, 512, 1024, 1056, 2048, 3584, 4096, 8192):
            for vocab in (1, 700, 2048, 8192, 8193, 32_000, 50_257, 151_936):
                for m in (rows, max(1, rows // 3)):
                    for roomy in (1, 0):
                        r = f(rows, m, d, vocab, asked, n_cus, roomy)
                        width = min(r.chunk, vocab)
                        listed = m < rows
                        assert r.chunk % 256 == 0 and 0 < r.chunk < vocab + 256 and r.w >= 1 and r.h >= 1
                        assert roomy or (r.w, r.h) == (1, 1)
                        ends = [(0, 2 * m * r.chunk), (r.plan, 2 * 32), (r.mask, rows * listed), (r.index, 4 * rows * listed),
                                (r.pos, 4 * rows * listed), (r.hidden, 2 * m * d * listed),
                                (r.dhidden, 4 * r.h * m * d if listed or r.h > 1 else 0),
                                (r.dweight, 4 * r.w * width * d if r.w > 1 else 0), (r.end, 0)]
                        case = (rows, m, d, vocab, roomy, r.chunk, r.w, r.h)
                        assert all(a + n <= b for (a, n), (b, _) in zip(ends, ends[1:])), case
                        assert all(a % 256 == 0 for a, _ in ends) and r.end <= r.all, case
                        split += r.w > 1 and vocab > 8192 and d >= 1024
    if 0 < asked < 8192 and n_cus == 256:
        assert split > 0                # sizes where it is the chunk that has dweight split, not the vocabulary or the model


@pytest.mark.parametrize("n_cus", [256, 64])
@pytest.mark.parametrize("asked", [0, 1024, 8192])
@pytest.mark.parametrize("d,vocab", [(64, 700), (512, 2048), (1024, 50_257), (2304, 128_256), (4096, 20_000), (4096, 151_936)])
def test_more_rows_never_need_less_for_the_gradient(d, vocab, asked, n_cus):
    f = room()
    for roomy in (1, 0):
        last = [0, 0]
        for n in list(range(1, 5200, 97)) + [6000, 8191, 8192, 8193, 12_000, 16_384, 30_000, 41_643, 65_537, 1 << 20]:
            now = [f(n, n, d, vocab, asked, n_cus, roomy).all, f(1 << 21, n, d, vocab, asked, n_cus, roomy).all]
            assert now[0] >= last[0] and now[1] >= last[1], (n, roomy, last, now)
            last = now


def test_bytes_asked_for_by_the_gradient():
    """What the header says of the call's workspace: the chunk's dlogits, with an explicit chunk at most 96 MiB of parts beside
    them; with the library's choice at most 1 GiB of dlogits (or those of 8,192 entries) and 256 MiB of parts, and parts only
    where some number of rows up to this one has them."""
    f, mib = room(), 1 << 20
    for rows in (1, 300, 2000, 4096, 12_000, 41_643, 100_000):
        for d in (64, 512, 1024, 4096):
            for vocab in (700, 8192, 50_257, 151_936):
                for asked in (256, 1024, 8192):
                    r = f(rows, rows, d, vocab, asked, 256, 1)
                    assert r.all <= 2 * rows * r.chunk + 96 * mib + 4096
                r = f(rows, rows, d, vocab, 0, 256, 1)
                assert r.all <= max(1024 * mib, 2 * rows * min(vocab + 255, 8192)) + 256 * mib + 4096
    # two parts of dhidden fit 128 MiB up to 4,096 rows of 4,096: these and their dlogits need less than 41,643 rows' dlogits
    assert f(41_643, 41_643, 4096, 151_936, 0, 256, 1).all == 1024 * mib + 256


class Layout(C.Structure):
    _fields_ = [(n, C.c_size_t) for n in ("tile_off", "partial", "g", "total")]


def test_partials_of_the_scalar_kernels_fit():
    """Between the tiling and the row coefficients there is room for the tiles of a planned batch (6 words each) and for what the
    workgroups of any other leave (14 words and a count each, a count per response; or 16 words of the loss), whatever the device,
    and more rows or responses never move an offset down."""
    f = B._lib()["_ZN3ais16workspace_layoutExi"]
    f.argtypes, f.restype = [C.c_longlong, C.c_int], Layout
    rows = [0, 1, 2048, 2049, 2304, 2305, 8192, 8193, 32_768, 32_769, 262_144, 262_145, 4_000_000, 2**31 - 1]
    for n_resp in (1, 8, 1023, 1024, 1025, 20_000):
        last = Layout()
        for n in rows:
            w, fewer = f(n, n_resp), f(n, max(1, n_resp - 1))
            if n_resp <= 1024:
                groups = 1 if n <= 2048 else min(256, max(min(-(-n // 256), 32), -(-n // 1024)))
                assert w.g - w.partial >= max(8 * 14 * groups + 4 * (n_resp + groups), 8 * 16 * groups), (n, n_resp)
            else:
                assert w.partial - w.tile_off >= 4 * (n_resp + 1)
                assert w.g - w.partial >= 8 * 6 * (-(-n // 1024) + n_resp), (n, n_resp)
            assert w.total - w.g >= 4 * n
            assert w.partial >= last.partial and w.g >= last.g and w.total >= last.total and w.total >= fewer.total
            last = w
