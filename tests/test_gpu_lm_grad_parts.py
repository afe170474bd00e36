"""The hidden-state gradient's products where their sums are split into parts: few rows (the hidden gradient), a narrow model or
a small vocabulary (the embedding gradient), both, with a row list, over several chunks, and with outputs whose rows are not
16-byte aligned.  Every element against float64 on the dlogits' own rounding."""
import ctypes as C
import time

import pytest
import torch

from paper_2605_13907_amd import binding as B
from tests.test_workspace import room

pytestmark = pytest.mark.gpu


class Parts(C.Structure):
    _fields_ = [("w", C.c_int), ("h", C.c_int)]


# rows, d, vocab, rows with a gradient (None: all), chunk (0: the library's choice), sums that are split
CASES = [
    (300, 4096, 20_000, None, 0, "h"),           # two blocks of rows, one chunk
    (65, 96, 3000, None, 1024, "h"),             # one tile, three chunks, the last one of 952 entries
    (257, 64, 70_001, 130, 0, "h"),              # two chunks, a row list
    (6001, 512, 2048, None, 0, "wh"),            # a long sum over rows, a last step of 49
    (5000, 64, 700, None, 256, "w"),             # three chunks, the last one narrower
    (9000, 128, 1500, 4097, 0, "wh"),            # a row list shorter than its bound would be
    (64, 32, 64, None, 0, ""),                   # one step each
    (1024, 512, 2048, None, 0, "h"),             # the longest sum over rows that stays whole, and one row more
    (1025, 512, 2048, None, 0, "wh"),
    (3000, 3584, 9000, None, 1024, "w"),         # dweight split because the chunk is narrow, not the vocabulary or the model
]


def operands(rows, d, vocab, live, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    w = (torch.randn(vocab, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    h = (torch.randn(rows, d, generator=g, device="cuda") * 2.0).bfloat16()
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda").to(torch.int32)
    c = torch.randn(rows, generator=g, device="cuda")
    if live is not None:
        c[torch.randperm(rows, generator=torch.Generator().manual_seed(seed))[live:].cuda()] = 0.0
    return h, w, y, c


def check(h, w, y, c, dh, dw):
    z = h.double() @ w.double().t()
    ds = torch.softmax(z, dim=1)
    ds.scatter_add_(1, y.long().unsqueeze(1), torch.full((h.shape[0], 1), -1.0, dtype=torch.float64, device="cuda"))
    ds *= c.double().unsqueeze(1)
    # a dlogit is rounded to bf16 once: up to 2^-8 of itself (eight significant bits), and the product's error is at most
    # that of all its terms; the fp32 lse and exponential and the fp32 sums add about 1e-5 of the same
    for got, a, b in ((dh, ds, w.double()), (dw, ds.t(), h.double())):
        a, b = a.contiguous(), b.contiguous()
        tol = (2.0 ** -8 + 1e-4) * (a.abs() @ b.abs()) + 1e-9
        err = (got.double() - a @ b).abs()
        assert bool((err <= tol).all()), float((err / tol).max())


@pytest.mark.parametrize("k", range(len(CASES)))
def test_parts(k):
    rows, d, vocab, live, chunk, split = CASES[k]
    print("rows", rows, "d", d, "vocab", vocab, "live", live, "chunk", chunk, flush=True)
    ctx = B.AisContext()
    choose = B._lib()["_ZN3ais13lm_grad_partsEixxx"]              # lm_grad_parts(compute units, rows, d_model, chunk)
    choose.argtypes, choose.restype = [C.c_int] + [C.c_longlong] * 3, Parts
    parts = choose(torch.cuda.get_device_properties(0).multi_processor_count, rows if live is None else live, d,
                   min(vocab, chunk or 65_536))
    assert (parts.w > 1, parts.h > 1) == ("w" in split, "h" in split), (parts.w, parts.h)
    h, w, y, c = operands(rows, d, vocab, live, 31 + k)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    bound = -1 if live is None else live
    dh, dw = ctx.lm_head_grad(h, w, y, lse, logp, c, chunk_vocab=chunk, n_live_max=bound)
    check(h, w, y, c, dh, dw)
    if live is not None:
        assert bool((dh[c == 0] == 0).all())
    again = ctx.lm_head_grad(h, w, y, lse, logp, c, chunk_vocab=chunk, n_live_max=bound)
    assert torch.equal(dh, again[0]) and torch.equal(dw, again[1])
    # outputs that begin four bytes after a 16-byte boundary: the same bits, and nothing beside them is touched
    at = {n: torch.full((t.numel() + 8,), 7.0, device="cuda") for n, t in (("h", dh), ("w", dw))}
    rc = B._lib().ais_lm_head_grad(ctx._h, h.data_ptr(), d, w.data_ptr(), d, B.AIS_BF16, rows, d, vocab, y.data_ptr(),
                                   lse.data_ptr(), logp.data_ptr(), c.data_ptr(), 1.0, chunk, bound,
                                   at["h"].data_ptr() + 4, at["w"].data_ptr() + 4)
    torch.cuda.synchronize()
    assert rc == 0
    for n, t in (("h", dh), ("w", dw)):
        assert torch.equal(at[n][1:-7].view_as(t), t) and bool((at[n][:1] == 7).all()) and bool((at[n][-7:] == 7).all())
    assert ctx.status() == 0
    ctx.close()


def test_recorded_in_a_workspace_without_room_for_parts():
    """A call that is being recorded can allocate nothing: with a workspace that holds the narrow chunks and no more it
    takes those, and its replays are right."""
    ctx = B.AisContext()
    h, w, y, c = operands(8192, 32, 8192, None, 77)          # sizes the workspace: 2 * 8192 * 8192 bytes and 42 MB, and a quarter
    logp, lse = ctx.lm_head_logprob(h, w, y)
    ctx.lm_head_grad(h, w, y, lse, logp, c, chunk_vocab=8192)
    small = operands(64, 256, 64, None, 78)
    logp, lse = ctx.lm_head_logprob(*small[:3])
    ctx.lm_head_grad(*small[:3], lse, logp, small[3])
    # 67 MB of dlogits in chunks of 8,192; 166 MB in one chunk and 134 + 67 MB of parts
    h, w, y, c = operands(4096, 256, 20_000, None, 79)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            dh, dw = ctx.lm_head_grad(h, w, y, lse, logp, c)
    torch.cuda.synchronize()
    for scale in (1.0, -0.5):
        c.mul_(scale)
        dh.fill_(7.0)
        dw.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(h, w, y, c, dh, dw)
    assert ctx.status() == 0
    ctx.close()


def free_bytes():
    """Free device memory, once it has stopped changing: what is freed shows with a delay."""
    torch.cuda.synchronize()
    last = torch.cuda.mem_get_info()[0]
    for _ in range(100):
        time.sleep(0.05)
        now = torch.cuda.mem_get_info()[0]
        if now == last:
            break
        last = now
    return last


@pytest.mark.parametrize("first", ["gradient", "diagnostics"])
def test_a_recorded_workspace_stays(first):
    """After a call has been recorded, an eager gradient call that the workspace holds in narrow chunks and one part leaves it
    where it is, although it would like a larger one: the graph still writes there.  Nothing is allocated, and replays before and
    after it are right."""
    ctx = B.AisContext()
    big = operands(8192, 32, 8192, None, 81)                 # sizes the workspace
    logp, lse = ctx.lm_head_logprob(*big[:3])
    ctx.lm_head_grad(*big[:3], lse, logp, big[3], chunk_vocab=8192)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    held = room()(8192, 8192, 32, 8192, 8192, units, 1).all * 1.25
    assert room()(4096, 4096, 256, 40_000, 0, units, 0).all < held < room()(4096, 4096, 256, 40_000, 0, units, 1).all
    h, w, y, c = operands(4096, 256, 40_000, None, 82)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    ctx.lm_head_grad(*operands(64, 256, 64, None, 83)[:3], lse[:64], logp[:64], c[:64])        # (kernel attributes)
    small = torch.rand(4096, device="cuda") - 2.0
    cu, rewards, params = torch.tensor([0, 4096], device="cuda"), torch.ones(1, device="cuda"), B.default_params()
    ctx.diagnostics(small, small, None, cu, rewards, 1, params)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        if first == "gradient":
            dh, dw = ctx.lm_head_grad(h, w, y, lse, logp, c)
        else:
            adv, count, diag = ctx.diagnostics(small, small * 0.5, None, cu, rewards, 1, params)
    eager = [torch.empty(4096, 256, device="cuda"), torch.empty(40_000, 256, device="cuda")]
    torch.cuda.synchronize()
    for scale in (1.0, -0.5, 3.0):
        c.mul_(scale)
        small.sub_(0.125)
        free = free_bytes()
        ctx._sync_stream()
        rc = B._lib().ais_lm_head_grad(ctx._h, h.data_ptr(), 256, w.data_ptr(), 256, B.AIS_BF16, 4096, 256, 40_000, y.data_ptr(),
                                       lse.data_ptr(), logp.data_ptr(), c.data_ptr(), 1.0, 0, -1, eager[0].data_ptr(),
                                       eager[1].data_ptr())
        assert rc == 0 and free_bytes() == free
        check(h, w, y, c, *eager)
        graph.replay()
        torch.cuda.synchronize()
        if first == "gradient":
            assert torch.equal(dh, eager[0]) and torch.equal(dw, eager[1])
        else:
            ref = ctx.diagnostics(small, small * 0.5, None, cu, rewards, 1, params)
            assert all(torch.equal(a, b) for a, b in zip((adv, count, diag), ref))
    assert ctx.status() == 0
    ctx.close()


def test_a_recorded_workspace_that_holds_the_parts():
    """A workspace that stays because a recorded call uses it, and holds another gradient call's chunks and parts although not what
    that call would ask for (room for calls over fewer rows): the call has its parts, and nothing is allocated."""
    ctx = B.AisContext()
    big = operands(4096, 32, 16_384, None, 85)               # sizes the workspace
    logp, lse = ctx.lm_head_logprob(*big[:3])
    ctx.lm_head_grad(*big[:3], lse, logp, big[3], chunk_vocab=8192)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    held = room()(4096, 4096, 32, 16_384, 8192, units, 1).all * 1.25
    now = room()(2000, 2000, 512, 10_000, 0, units, 1)
    assert now.end < held < now.all and now.h > 1
    h, w, y, c = operands(2000, 512, 10_000, None, 86)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    small = torch.rand(2000, device="cuda") - 2.0
    cu, rewards, params = torch.tensor([0, 2000], device="cuda"), torch.ones(1, device="cuda"), B.default_params()
    ctx.diagnostics(small, small, None, cu, rewards, 1, params)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        adv, count, diag = ctx.diagnostics(small, small * 0.5, None, cu, rewards, 1, params)
    fresh = B.AisContext()
    want = fresh.lm_head_grad(h, w, y, lse, logp, c)
    dh, dw = torch.empty(2000, 512, device="cuda"), torch.empty(10_000, 512, device="cuda")
    for _ in range(3):
        free = free_bytes()
        ctx._sync_stream()
        rc = B._lib().ais_lm_head_grad(ctx._h, h.data_ptr(), 512, w.data_ptr(), 512, B.AIS_BF16, 2000, 512, 10_000, y.data_ptr(),
                                       lse.data_ptr(), logp.data_ptr(), c.data_ptr(), 1.0, 0, -1, dh.data_ptr(), dw.data_ptr())
        assert rc == 0 and free_bytes() == free
        check(h, w, y, c, dh, dw)
        assert torch.equal(dh, want[0]) and torch.equal(dw, want[1])
        graph.replay()
        torch.cuda.synchronize()
        ref = ctx.diagnostics(small, small * 0.5, None, cu, rewards, 1, params)
        assert all(torch.equal(a, b) for a, b in zip((adv, count, diag), ref))
    assert ctx.status() == 0 and fresh.status() == 0
    ctx.close()
    fresh.close()


def test_no_room_for_wide_chunks_now_and_room_later():
    """While the device is full, calls take narrow chunks and keep the workspace they have; the first call after that takes wide
    ones again."""
    ctx = B.AisContext()
    h, w, y, c = operands(8192, 64, 65_536, None, 84)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    wide, narrow = (int(room()(8192, 8192, 64, 65_536, 0, units, roomy).all * 1.25) for roomy in (1, 0))
    left = (wide + narrow) // 2
    assert narrow + (64 << 20) < left < wide - (64 << 20)
    out = [[torch.empty(8192, 64, device="cuda"), torch.empty(65_536, 64, device="cuda")] for _ in range(4)]

    def call(k):
        rc = B._lib().ais_lm_head_grad(ctx._h, h.data_ptr(), 64, w.data_ptr(), 64, B.AIS_BF16, 8192, 64, 65_536, y.data_ptr(),
                                       lse.data_ptr(), logp.data_ptr(), c.data_ptr(), 1.0, 0, -1, out[k][0].data_ptr(),
                                       out[k][1].data_ptr())
        assert rc == 0
        return free_bytes()

    torch.cuda.empty_cache()
    full = torch.empty(free_bytes() - left, dtype=torch.uint8, device="cuda")
    before = free_bytes()
    print("free", before, "wide", wide, "narrow", narrow, flush=True)
    assert narrow + (64 << 20) < before < wide - (64 << 20)
    first = call(0)
    assert abs(before - first - narrow) <= 16 << 20
    assert call(1) == first                              # nothing is given back, nothing asked for
    del full
    torch.cuda.empty_cache()
    free = free_bytes()
    third = call(2)
    assert abs(free - third - (wide - narrow)) <= 16 << 20
    assert call(3) == third
    assert all(torch.equal(a, b) for k in (0, 2) for a, b in zip(out[k], out[k + 1]))
    for a, b in zip(out[0], out[2]):                     # the same bf16 dlogits; fp32 sums in another order
        assert (a - b).norm() < 1e-5 * b.norm()
    assert ctx.status() == 0
    ctx.close()
