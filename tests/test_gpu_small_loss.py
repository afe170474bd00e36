"""Loss and gradient of small batches in one launch, at the edges of the sizes that take it, against the coefficients, weights
and loss that the row-scale call forms in its own kernel."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n_resp", [(1, 1), (2, 2), (63, 4), (511, 8), (512, 64), (512, 65), (513, 16), (1024, 64),
                                         (1025, 64)])
@pytest.mark.parametrize("dtype,vocab", [(torch.float32, 8), (torch.float32, 1024), (torch.float32, 1028),
                                         (torch.float32, 2049), (torch.bfloat16, 4096), (torch.bfloat16, 4104),
                                         (torch.bfloat16, 9001), (torch.bfloat16, 32_776), (torch.float32, 33_000)])
@pytest.mark.parametrize("stale", [False, True])
def test_against_the_row_scale_call(rows, n_resp, dtype, vocab, stale):
    ctx = B.AisContext()
    g = torch.Generator(device="cuda")
    g.manual_seed(rows * 7 + n_resp + vocab)
    z = (torch.randn(rows, vocab, generator=g, device="cuda") * 3).to(dtype)
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    valid = (torch.rand(rows, generator=g, device="cuda") < 0.8).to(torch.uint8) if stale else None
    cuts = torch.randint(0, rows + 1, (n_resp - 1,), generator=g, device="cuda").sort().values     # empty responses among them
    cu = torch.cat([torch.zeros(1, device="cuda"), cuts, torch.full((1,), rows, device="cuda")]).long()
    rewards = (torch.rand(n_resp, generator=g, device="cuda") < 0.5).float()
    p = B.default_params(beta_kl=0.04, inv_temperature=0.8) if stale else B.default_params()
    logp, lse = ctx.token_logprob(z, y, valid, p.inv_temperature)
    roll = logp + 0.2 * torch.randn(rows, generator=g, device="cuda")
    old = logp + 0.3 * torch.randn(rows, generator=g, device="cuda") if stale else None      # some ratios beyond the clip range
    ref = logp - 0.1 if stale else None
    adv, count, diag = ctx.diagnostics(logp if old is None else old, roll, valid, cu, rewards, 1, p)
    adv = adv + torch.linspace(-1, 1, n_resp, device="cuda") + 0.01
    want_loss, want_wt, want_g = ctx.grpo_row_scale(logp, roll, valid, cu, adv, count, diag, p, old, ref)
    for out in (None, z.clone()):
        src = z if out is None else out
        loss, wt, dz = ctx.grpo_loss_grad(src, y, valid, cu, logp, lse, roll, adv, count, diag, p, old, ref, dlogits=out)
        assert torch.equal(wt, want_wt)
        # the same fp64 terms in another order
        scale = want_g.abs().double().sum() + want_loss.abs()
        assert (loss - want_loss).abs() <= 1e-12 * scale
        s = torch.softmax(z.double() * p.inv_temperature, dim=1)
        s.scatter_add_(1, y.long().unsqueeze(1), torch.full((rows, 1), -1.0, dtype=torch.float64, device="cuda"))
        want = s * want_g.double().unsqueeze(1)
        rounding = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
        near_one = 1e-6 * want_g.double().abs().unsqueeze(1)             # p_y - 1 by subtraction in `s`
        assert bool(((dz.double() - want).abs() <= (rounding + 2e-5) * want.abs() + near_one * 1e-6 + 1e-30).all())
        assert not dz[want_g == 0].any()
    _, none, _ = ctx.grpo_loss_grad(z, y, valid, cu, logp, lse, roll, adv, count, diag, p, old, ref, want_wtilde=False)
    assert none is None and ctx.status() == 0
    ctx.close()


@pytest.mark.parametrize("fault", ["first", "last", "order", "range"])
def test_row_offsets_that_are_no_partition(fault):
    ctx = B.AisContext()
    z = torch.randn(64, 512, device="cuda")
    y = torch.zeros(64, device="cuda", dtype=torch.int32)
    cu = torch.tensor([0, 16, 32, 48, 64])
    cu[{"first": 0, "last": 4, "order": 1, "range": 2}[fault]] = {"first": 1, "last": 63, "order": 40, "range": 10 ** 12}[fault]
    logp, lse = ctx.token_logprob(z, y)
    one = torch.ones(4, device="cuda")
    good = torch.tensor([0, 16, 32, 48, 64], device="cuda")
    adv, count, diag = ctx.diagnostics(logp, logp, None, good, one, 1)
    assert ctx.status() == 0
    ctx.grpo_loss_grad(z, y, None, cu.cuda(), logp, lse, logp, one, count, diag)
    assert ctx.status() & B.STATUS_BAD_CU
    ctx.grpo_loss_grad(z, y, None, good, logp, lse, logp, one, count, diag)
    assert ctx.status() == 0
    ctx.close()
