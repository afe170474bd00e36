"""The two products of the hidden-state gradient at the sizes where their tiles (256 x 256 outputs, 64 summed elements a
step) end inside the operands, with sums whole and in parts, with one and with several chunks, and with a row list.  Every element against float64 on the dlogits' own rounding."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.AisContext()
    yield c
    c.close()


def case(rows, d, vocab, live, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    w = (torch.randn(vocab, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    h = (torch.randn(rows, d, generator=g, device="cuda") * 2.0).bfloat16()
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda").to(torch.int32)
    c = torch.randn(rows, generator=g, device="cuda")
    if live is not None:
        c[torch.randperm(rows, generator=torch.Generator().manual_seed(seed))[live:].cuda()] = 0.0
    return h, w, y, c


# rows, d, vocab, rows with a gradient (None: all), chunk (0: the library's choice)
CASES = [
    (4096, 4096, 8192, None, 0),           # whole tiles and steps
    (4097, 4064, 8193, None, 8192),        # one row, one entry and half a d block over; a last chunk of one entry
    (4031, 4096, 7937, None, 0),           # a last step of 63 rows, a last tile of one entry
    (3841, 4064, 16_100, None, 8192),      # 16,100 = 8,192 + 7,908: two chunks, the hidden gradient accumulates
    (9000, 4096, 8200, 4000, 0),           # a row list
    (6000, 2080, 8192, 2055, 8192),        # a row list, a last d block of 32, seven rows in the last step
    (16_384, 1024, 3000, None, 0),         # a long sum over rows for few entries
    (300, 4096, 20_000, 7, 0),             # few rows: one wide chunk, a list shorter than a step
    (5000, 64, 700, None, 256),            # one d block of 64, a last chunk of 188 entries
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_products(ctx, k):
    rows, d, vocab, live, chunk = CASES[k]
    print("rows", rows, "d", d, "vocab", vocab, "live", live, "chunk", chunk, flush=True)
    h, w, y, c = case(rows, d, vocab, live, 17 + k)
    logp, lse = ctx.lm_head_logprob(h, w, y)
    dh, dw = ctx.lm_head_grad(h, w, y, lse, logp, c, chunk_vocab=chunk, n_live_max=-1 if live is None else live)
    z = h.double() @ w.double().t()
    ds = torch.softmax(z, dim=1)
    ds.scatter_add_(1, y.long().unsqueeze(1), torch.full((rows, 1), -1.0, dtype=torch.float64, device="cuda"))
    ds *= c.double().unsqueeze(1)
    # a dlogit is rounded to bf16 once: up to 2^-8 of itself (eight significant bits), and the product's error is at most
    # that of all its terms; the fp32 lse and exponential and the fp32 sum add about 1e-5 of the same
    for got, a, b in ((dh, ds, w.double()), (dw, ds.t(), h.double())):
        a, b = a.contiguous(), b.contiguous()
        tol = (2.0 ** -8 + 1e-4) * (a.abs() @ b.abs()) + 1e-9
        err = (got.double() - a @ b).abs()
        assert bool((err <= tol).all()), float((err / tol).max())
    if live is not None:
        assert bool((dh[c == 0] == 0).all())
    again = ctx.lm_head_grad(h, w, y, lse, logp, c, chunk_vocab=chunk, n_live_max=-1 if live is None else live)
    assert torch.equal(dh, again[0]) and torch.equal(dw, again[1])
    assert ctx.status() == 0
