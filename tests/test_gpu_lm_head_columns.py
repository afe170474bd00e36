"""The read-out's token blocks: as many rows in each, dealt to the wavefronts in columns of 16, with the copies that so many rows
take; the embedding one step ahead or two (by rows, d_model, vocabulary and mask), with contractions of one, two, three and more
steps."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu


def problem(rows, vocab, d, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    h = torch.randn(rows, d, generator=g, device="cuda").bfloat16()
    w = (torch.randn(vocab, d, generator=g, device="cuda") * 2 / d ** 0.5).bfloat16()
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    return g, h, w, y


def check(ctx, rows, vocab, d, grad=True, masked=False):
    g, h, w, y = problem(rows, vocab, d, rows + 7 * vocab + 13 * d)
    valid = (torch.rand(rows, generator=g, device="cuda") < 0.5).to(torch.uint8) if masked else None
    z = h.double() @ w.double().t()
    lse = torch.logsumexp(z, dim=1)
    want = z.gather(1, y.long().unsqueeze(1)).squeeze(1) - lse
    logp, got_lse = ctx.lm_head_logprob(h, w, y, valid)
    keep = torch.ones(rows, dtype=torch.bool, device="cuda") if valid is None else valid.bool()
    # fp32 accumulation of d products and an fp32 log-sum-exp of results of a few units
    assert (logp.double() - want)[keep].abs().max() < 1e-5 if bool(keep.any()) else True, (rows, vocab, d)
    assert (got_lse.double() - lse)[keep].abs().max() < 1e-5 if bool(keep.any()) else True, (rows, vocab, d)
    assert not logp[~keep].any() and not got_lse[~keep].any()
    if not grad:
        return
    c = torch.randn(rows, generator=g, device="cuda")
    dh, dw = ctx.lm_head_grad(h, w, y, lse.float(), want.float(), c)
    ds = (z - lse.unsqueeze(1)).exp_()
    ds.scatter_(1, y.long().unsqueeze(1), torch.expm1(want).unsqueeze(1))
    ds *= c.double().unsqueeze(1)
    # dlogits are rounded to bf16 (2^-9 of each), independently
    for got, ref in ((dh, ds @ w.double()), (dw, ds.t().contiguous() @ h.double())):
        assert (got.double() - ref).norm() < 4e-3 * ref.norm(), (rows, vocab, d)


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 48, 63, 64, 65, 112, 129, 176, 195, 208, 241, 255, 256, 257, 273, 300, 390,
                                  511, 513, 769])
def test_columns(rows):
    ctx = B.AisContext()
    for vocab, d in ((700, 64), (257, 160), (1500, 224)):
        check(ctx, rows, vocab, d)
        check(ctx, rows, vocab, d, grad=False, masked=True)
    assert ctx.status() == 0
    ctx.close()


@pytest.mark.parametrize("rows,d", [(6144, 64), (6145, 64), (6400, 192), (12_288, 128), (12_290, 128), (600, 1984), (600, 2048),
                                    (300, 2080)])
def test_either_side_of_the_rule(rows, d):
    ctx = B.AisContext()
    check(ctx, rows, 520, d)
    check(ctx, rows, 520, d, grad=False, masked=True)
    ctx.close()


@pytest.mark.parametrize("rows,vocab,d", [(256, 8192, 1024), (257, 8192, 1024), (256, 8191, 1024), (256, 8192, 960), (2049, 8192, 1024),
                                          (2050, 8192, 1024), (4608, 300, 2048), (4609, 300, 2048), (9217, 300, 2048),
                                          (9218, 300, 2048)])
def test_edges_of_two_steps_ahead(rows, vocab, d):
    ctx = B.AisContext()
    check(ctx, rows, vocab, d, grad=False)
    check(ctx, rows, vocab, d, grad=False, masked=True)
    ctx.close()


@pytest.mark.parametrize("rows,d,pitch", [(6145, 72, 72), (6400, 96, 104), (6160, 128, 136), (300, 64, 72), (6200, 200, 256)])
def test_embedding_rows_across_lines(rows, d, pitch):
    """An embedding whose rows do not begin with a 128-byte line is copied two steps ahead at any size: ragged d_model, a pitch
    that is no multiple of 64 elements, a base in the middle of a line."""
    ctx = B.AisContext()
    vocab = 600
    g, h, w, y = problem(rows, vocab, d, rows + d)
    for offset in (0, 8):
        room = torch.zeros(vocab * pitch + offset, device="cuda", dtype=torch.bfloat16)
        wide = room[offset:].view(vocab, pitch)[:, :d]
        wide.copy_(w)
        want = ctx.lm_head_logprob(h, w, y)
        z = h.double() @ w.double().t()
        lse = torch.logsumexp(z, dim=1)
        logp, got_lse = ctx.lm_head_logprob(h, wide, y)
        # fp32 accumulation of d products and an fp32 log-sum-exp of results of a few units
        assert (logp.double() - (z.gather(1, y.long().unsqueeze(1)).squeeze(1) - lse)).abs().max() < 1e-5
        assert torch.equal(logp, want[0]) and torch.equal(got_lse, want[1])
        if d % 32 == 0:
            c = torch.randn(rows, generator=g, device="cuda")
            for a, b in zip(ctx.lm_head_grad(h, wide, y, got_lse, logp, c), ctx.lm_head_grad(h, w, y, got_lse, logp, c)):
                # the same bf16 dlogits; products by one kernel or another
                assert (a - b).norm() < 1e-5 * b.norm()
    assert ctx.status() == 0
    ctx.close()
