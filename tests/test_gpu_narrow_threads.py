"""Narrow rows in the gradient sweep and the one-sweep call, at the ends of the classes that give a row 64 to 1,024 threads:
aligned and not, masked rows, out of place and in place."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu

VECTORS = [1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049]


@pytest.mark.parametrize("vectors", VECTORS)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_direction_and_gradient(dtype, vectors):
    """Tolerance: one rounding to the output type of a value that fp32 exponentials and an fp32 shift of up to about 20 give
    to a few 1e-6."""
    n = 16 // dtype.itemsize
    ctx, p = B.AisContext(), B.default_params()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vectors)
    rounding = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    for vocab, rows in ((vectors * n, 600), (vectors * n + 1, 601), (vectors * n + n - 1, 40)):
        z = (torch.randn(rows, vocab, generator=gen, device="cuda") * 3.0).to(dtype)
        y = torch.randint(0, vocab, (rows,), generator=gen, device="cuda", dtype=torch.int32)
        y[0], y[1], y[2] = 0, vocab - 1, min(vocab - 1, (vectors - 1) * n)
        valid = (torch.rand(rows, generator=gen, device="cuda") < 0.9).to(torch.uint8)
        ref = torch.log_softmax(z.double(), 1)
        want_logp = ref.gather(1, y.long().unsqueeze(1)).squeeze(1) * valid
        want = ref.exp().scatter_add_(1, y.long().unsqueeze(1), torch.full((rows, 1), -1.0, dtype=torch.float64, device="cuda"))
        want *= valid.unsqueeze(1)
        logp, lse = ctx.token_logprob(z, y, valid)
        roll = logp - 0.1
        cu = torch.tensor([0, rows // 3, rows], device="cuda")
        adv, count, diag = ctx.diagnostics(logp, roll, valid, cu, torch.tensor([1.0, 0.0], device="cuda"), 2, p)
        _, _, g = ctx.grpo_row_scale(logp, roll, valid, cu, adv, count, diag, p)
        _, _, dz = ctx.grpo_loss_grad(z, y, valid, cu, logp, lse, roll, adv, count, diag, p)
        want_dz = want * g.double().unsqueeze(1)
        assert bool(((dz.double() - want_dz).abs() <= (rounding + 1e-5) * want_dz.abs() + 1e-30).all()), vocab
        for out in (None, z):
            got, _, s = ctx.token_logprob_softmax_grad(z, y, valid, sgrad=out)
            assert bool(((got.double() - want_logp).abs() <= 1e-5 * want_logp.abs().clamp_min(1.0)).all()), vocab
            assert bool(((s.double() - want).abs() <= (rounding + 1e-5) * want.abs() + 1e-30).all()), vocab
    assert ctx.status() == 0
    ctx.close()


@pytest.mark.parametrize("vectors", [1024, 1025, 1536, 2047, 2048, 2049])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_many_masked_rows(dtype, vectors):
    """Both sides of the line at which rows of more than 1,024 vectors share other numbers of threads: a mask, and eight rows
    per compute unit."""
    n = 16 // dtype.itemsize
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vectors)
    rounding = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    for vocab in (vectors * n, vectors * n + n - 1):
        for rows in (2047, 2048):
            z = (torch.randn(rows, vocab, generator=gen, device="cuda") * 3.0).to(dtype)
            y = torch.randint(0, vocab, (rows,), generator=gen, device="cuda", dtype=torch.int32)
            valid = (torch.rand(rows, generator=gen, device="cuda") < 0.5).to(torch.uint8)
            logp, lse, s = ctx.token_logprob_softmax_grad(z, y, valid)
            for r in range(0, rows, 256):                                 # a part at a time: fp64
                ref = torch.log_softmax(z[r:r + 256].double(), 1)
                at, on = y[r:r + 256].long().unsqueeze(1), valid[r:r + 256].unsqueeze(1)
                want_logp = (ref.gather(1, at) * on).squeeze(1)
                want = ref.exp().scatter_add_(1, at, torch.full_like(at, -1.0, dtype=torch.float64)) * on
                assert bool(((logp[r:r + 256].double() - want_logp).abs() <= 1e-5 * want_logp.abs().clamp_min(1.0)).all())
                # one rounding to the output type of a value that fp32 exponentials and an fp32 shift of up to about 20 give
                assert bool(((s[r:r + 256].double() - want).abs() <= (rounding + 1e-5) * want.abs() + 1e-30).all())
    assert ctx.status() == 0
    ctx.close()
