"""The log-prob sweep at the edges of the rule that gives a row 64 to 1,024 threads, and of the rounds in which those read
it: every width where the number of vectors left after the last whole round changes class, aligned and not."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu

# bf16 vectors hold 8 elements, fp32 ones 4; rows on both sides of 1, 2 and 8 per compute unit (256 of them)
ROWS = [1, 256, 257, 512, 513, 2047, 2048, 2049]
VECTORS = [1, 63, 64, 65, 128, 129, 192, 193, 256, 257, 511, 512, 513, 895, 896, 1025, 2047, 2048, 2499, 2500, 4097, 8191,
           8192, 8193, 10_241]


@pytest.mark.parametrize("vectors", VECTORS)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_log_probs_at_the_edges_of_the_rule(dtype, vectors):
    n = 16 // dtype.itemsize
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vectors)
    for extra in (0, n // 2 + 1):                       # the second: rows of odd width, unaligned
        vocab = vectors * n + extra
        base = (torch.randn(max(ROWS), vocab, generator=gen, device="cuda") * 4).to(dtype)
        y = torch.randint(0, vocab, (max(ROWS),), generator=gen, device="cuda", dtype=torch.int32)
        y[:4] = torch.tensor([0, vocab - 1, max(0, vocab - extra - 1), min(vocab - 1, (vectors - 1) * n)],
                             dtype=torch.int32)
        ref = torch.cat([torch.logsumexp(base[r:r + 256].double(), dim=1) for r in range(0, max(ROWS), 256)])
        ref_y = base.gather(1, y.long().unsqueeze(1)).squeeze(1).double() - ref
        for rows in ROWS:
            logp, lse = ctx.token_logprob(base[:rows], y[:rows])
            # sums of up to 2^17 fp32 terms in trees of a few hundred: 1e-6 relative, and the rounding of the fp32 results
            assert (lse.double() - ref[:rows]).abs().max() < 4e-6, (vocab, rows)
            assert (logp.double() - ref_y[:rows]).abs().max() < 6e-6, (vocab, rows)
        again = ctx.token_logprob(base[:7], y[:7])
        assert torch.equal(again[0], ctx.token_logprob(base[:7], y[:7])[0])
    assert ctx.status() == 0
    ctx.close()


@pytest.mark.parametrize("vectors", [127, 767, 768, 769, 1535, 1537, 2999, 3000, 3199, 3200, 3499, 3501])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_log_probs_at_the_other_edges(dtype, vectors):
    """The lines that lie elsewhere for few rows and for the two types, and tails of three vectors a thread."""
    test_log_probs_at_the_edges_of_the_rule(dtype, vectors)


@pytest.mark.parametrize("rows", [769, 1280, 1281])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_rows_per_compute_unit(dtype, rows):
    """Three to five rows per compute unit (256 of them), where 2,500 to 8,191 vectors have 256 threads instead of 512."""
    n = 16 // dtype.itemsize
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    for vocab in (3300 * n, 6283 * n, 6283 * n + 1):
        z = (torch.randn(rows, vocab, generator=gen, device="cuda") * 4).to(dtype)
        y = torch.randint(0, vocab, (rows,), generator=gen, device="cuda", dtype=torch.int32)
        ref = torch.cat([torch.logsumexp(z[r:r + 256].double(), dim=1) for r in range(0, rows, 256)])
        ref_y = z.gather(1, y.long().unsqueeze(1)).squeeze(1).double() - ref
        logp, lse = ctx.token_logprob(z, y)
        # sums of up to 2^17 fp32 terms in trees of a few hundred: 1e-6 relative, and the rounding of the fp32 results
        assert (lse.double() - ref).abs().max() < 4e-6 and (logp.double() - ref_y).abs().max() < 6e-6, vocab
    ctx.close()
