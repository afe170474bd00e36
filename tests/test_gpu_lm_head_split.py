"""How the hidden-state read-out is split over the chip: a few token blocks take many short chunks of the vocabulary
(more than 64), a mask that leaves few of many rows takes more chunks than the whole batch would, and the listing of
evaluated rows works on runs of 64 rows per wavefront.  Every log-prob against float64 on the same bits."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.AisContext()
    yield c
    c.close()


def operands(rows, d, vocab, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    w = (torch.randn(vocab, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    h = (torch.randn(rows, d, generator=g, device="cuda") * 2.0).bfloat16()
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda").to(torch.int32)
    return h, w, y


def reference(h, w, y):
    z = h.double() @ w.double().t()
    lse = torch.logsumexp(z, dim=1)
    return z.gather(1, y.long().unsqueeze(1)).squeeze(1) - lse, lse


# the accumulation of 64 to 256 products in fp32 and the exponentials are good to about 1e-5 (the full-width tests see
# 2e-5 at most over 4,096 products); 2e-4 leaves room for the sum over 100,000 entries
TOL = 2e-4


@pytest.mark.parametrize("d", [64, 96, 72])           # whole, half and ragged last slices of d_model
@pytest.mark.parametrize("rows", [1, 17, 255, 256, 257, 390, 1025, 2049])
def test_few_token_blocks(ctx, rows, d):
    for vocab in (255, 256 * 65 + 1, 90_113):
        print("rows", rows, "d", d, "vocab", vocab, flush=True)
        h, w, y = operands(rows, d, vocab, rows + vocab)
        logp, lse = ctx.lm_head_logprob(h, w, y)
        ref_p, ref_l = reference(h, w, y)
        assert (logp.double() - ref_p).abs().max() <= TOL and (lse.double() - ref_l).abs().max() <= TOL
        assert ctx.status() == 0


@pytest.mark.parametrize("rows,live", [(63, 1), (64, 63), (1024, 3), (1025, 1024), (4097, 257), (5000, 2), (9000, 0)])
def test_few_evaluated_rows(ctx, rows, live):
    vocab, d = 50_261, 64
    h, w, y = operands(rows, d, vocab, rows + live)
    order = torch.randperm(rows, generator=torch.Generator().manual_seed(rows))[:live].cuda()
    valid = torch.zeros(rows, dtype=torch.uint8, device="cuda")
    valid[order] = 1
    y[valid == 0] = -1
    logp, lse = ctx.lm_head_logprob(h, w, y, valid)
    on = valid.bool()
    assert bool((logp[~on] == 0).all()) and bool((lse[~on] == 0).all())
    if live:
        ref_p, ref_l = reference(h[on], w, y[on])
        assert (logp[on].double() - ref_p).abs().max() <= TOL and (lse[on].double() - ref_l).abs().max() <= TOL
    assert ctx.status() == 0


@pytest.mark.parametrize("d", [8, 56, 64, 72, 104, 128, 136, 200, 256, 264])
def test_every_length_of_the_contraction(ctx, d):
    """One step and less, an odd and an even number of steps, last slices of 1 to 8 chunks, with values next to the
    rows that must not enter (the operands are views of wider, NaN-filled arrays)."""
    rows, vocab = 300, 1100
    h, w, y = operands(rows, d, vocab, d)
    wide_h = torch.full((rows, d + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide_w = torch.full((vocab, d + 16), float("nan"), dtype=torch.bfloat16, device="cuda")
    wide_h[:, :d], wide_w[:, :d] = h, w
    logp, lse = ctx.lm_head_logprob(wide_h[:, :d], wide_w[:, :d], y)
    ref_p, ref_l = reference(h, w, y)
    assert (logp.double() - ref_p).abs().max() <= TOL and (lse.double() - ref_l).abs().max() <= TOL
    # an infinite embedding row is that row's logit, and nothing else's
    w[7] = float("-inf")
    h = h.abs() + 0.01
    y[y == 7] = 8
    logp, lse = ctx.lm_head_logprob(h, w, y)
    ref_p, ref_l = reference(h, w, y)
    assert (logp.double() - ref_p).abs().max() <= TOL and (lse.double() - ref_l).abs().max() <= TOL
