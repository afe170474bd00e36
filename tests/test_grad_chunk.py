"""The library's choice of the gradient call's chunk by d_model: the library's own size function on the CPU, and on the GPU the
results against those of an explicit chunk."""
import ctypes as C

import pytest
import torch

from paper_2605_13907_amd import binding as B


def choose():
    f = B._lib()["_ZN3ais17lm_grad_chunk_forExxxi"]              # lm_grad_chunk_for(chunk, vocab, d_model, compute units)
    f.argtypes, f.restype = [C.c_longlong, C.c_longlong, C.c_longlong, C.c_int], C.c_longlong
    return f


@pytest.mark.parametrize("n_cus", [256, 64, 304])
def test_chunk_fills_the_rounds(n_cus):
    f = choose()
    for d in range(32, 8193, 32):
        across = (d + 255) // 256

        def fill(tiles):
            return tiles * across / (-(-tiles * across // n_cus) * n_cus)

        chunk = f(8192, 1 << 20, d, n_cus)
        full = [t for t in range(22, 32) if fill(t) >= 0.95]
        want = 32 if fill(32) >= 0.8 or not full else max(full)
        assert chunk == 256 * want                                 # never wider, so it fits what 8,192 entries need
        assert f(8192, 24_575, d, n_cus) == 8192                   # fewer than three chunks
        for other in (256, 7168, 8448, 43_520):                    # only the default is looked at
            assert f(other, 1 << 20, d, n_cus) == other


@pytest.mark.gpu
@pytest.mark.parametrize("rows,vocab,d", [(3073, 25_001, 2304), (3300, 30_001, 2560), (3200, 33_000, 4352)])
def test_same_gradient_as_an_explicit_chunk(rows, vocab, d):
    ctx = B.AisContext()
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    h = torch.randn(rows, d, generator=g, device="cuda").bfloat16()
    w = (torch.randn(vocab, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    c = torch.randn(rows, generator=g, device="cuda")
    for live in (-1, rows - 1):
        c[0] = 0.0
        dh, dw = ctx.lm_head_grad(h, w, y, lse, logp, c, n_live_max=live)
        dh2, dw2 = ctx.lm_head_grad(h, w, y, lse, logp, c, chunk_vocab=4096, n_live_max=live)
        # the same bf16 dlogits; fp32 sums in another order
        assert (dh - dh2).norm() < 1e-5 * dh2.norm() and (dw - dw2).norm() < 1e-5 * dw2.norm()
    assert ctx.status() == 0
    ctx.close()
