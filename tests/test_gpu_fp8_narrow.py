"""FP8 kernels on narrow rows: the streaming kernels with 64 and 256 threads a row, at the ends of their ranges, aligned and not,
with NaNs, infinities and logits of any magnitude, against the kernels that hold a row where those take over."""
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu

MAX = 448.0


def reference(z, aligned_bf16):
    """Codes and scale as the definition gives them; a NaN is -448, in 16-byte aligned bf16 rows the row's largest magnitude
    with its own sign."""
    x = z.float()
    amax = torch.where(x.isnan(), torch.zeros_like(x), x).abs().amax(dim=1)
    s = amax / torch.full_like(amax, MAX)
    s = torch.where(s > 0, s, torch.ones_like(s))
    own = torch.copysign(amax.unsqueeze(1).expand_as(x), x) if aligned_bf16 else -MAX * s.unsqueeze(1)
    q = (torch.where(x.isnan(), own, x) / s.unsqueeze(1)).clamp(-MAX, MAX)
    return q.to(torch.float8_e4m3fn).view(torch.uint8), s


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("vocab", [1, 7, 8, 9, 63, 64, 520, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 4100, 8192, 16_384,
                                   16_391, 16_392])
def test_narrow_rows(dtype, vocab):
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    for rows in (3, 2047, 2048) if vocab <= 4100 else (3, 500):
        z = (torch.randn(rows, vocab, generator=gen, device="cuda") * 3).to(dtype)
        y = torch.randint(0, vocab, (rows,), generator=gen, device="cuda", dtype=torch.int32)
        aligned = dtype == torch.bfloat16 and vocab % 8 == 0
        codes, scale = ctx.fp8_quantize_rows(z)
        want, s = reference(z, aligned)
        assert torch.equal(codes, want) and torch.equal(scale, s), rows
        back = want.view(torch.float8_e4m3fn).float() * s.unsqueeze(1)
        assert torch.equal(ctx.fp8_dequantize_rows(codes, scale, torch.float32), back), rows
        assert torch.equal(ctx.fp8_dequantize_rows(codes, scale, torch.bfloat16), back.bfloat16()), rows
        logp = ctx.fp8_rollout_logprob(z, y)
        ref = torch.log_softmax(back.double(), dim=1).gather(1, y.long().unsqueeze(1)).squeeze(1)
        # fp32 log-sum-exp minus an fp32 logit, both of up to 20: a few ulp of 2^-19
        assert (logp.double() - ref).abs().max() < 8e-6, rows
        # a NaN of either sign in every other row
        z[::2, vocab // 2] = float("nan")
        z[::4, vocab // 2] = -z[::4, vocab // 2]
        want, s = reference(z, aligned)
        codes, scale = ctx.fp8_quantize_rows(z)
        assert torch.equal(scale, s) and torch.equal(codes, want), rows
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("power", [-30, 3, 9, 12, 20, 35])
def test_any_magnitude(dtype, power):
    """The largest term of the sum is 1 at every magnitude."""
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(power + 99)
    for vocab in (64, 65, 4096):
        z = (torch.randn(64, vocab, generator=gen, device="cuda") * 10.0 ** power).to(dtype)
        y = torch.randint(0, vocab, (64,), generator=gen, device="cuda", dtype=torch.int32)
        y[::2] = z[::2].argmax(dim=1).int()
        codes, s = reference(z, False)
        back = codes.view(torch.float8_e4m3fn).double() * s.double().unsqueeze(1)
        ref = torch.log_softmax(back, dim=1).gather(1, y.long().unsqueeze(1)).squeeze(1)
        logp = ctx.fp8_rollout_logprob(z, y).double()
        # products are rounded to fp32: 2^-23 of the largest logit, beside the log-prob itself
        tol = 2.0 ** -22 * z.float().abs().amax(dim=1).double() + 1e-5
        assert ((logp - ref).abs() <= tol).all(), (vocab, (logp - ref).abs().max())
    ctx.close()


@pytest.mark.parametrize("rows,vocab", [(500, 4096), (2048, 1000)])
def test_a_nan_does_not_round_the_products(rows, vocab):
    """A negative NaN in an aligned bf16 row has the code of the row's lowest possible value, so the log-probs are to the bit
    those of the row that holds this value: the products of its ordinary logits are formed as exactly."""
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    z = (torch.randn(rows, vocab, generator=gen, device="cuda") * 3).bfloat16()
    at = z.float().abs().argmin(dim=1, keepdim=True)             # never the largest magnitude
    lowest = z.scatter(1, at, -z.float().abs().amax(dim=1, keepdim=True).bfloat16())
    nan = z.view(torch.int16).scatter(1, at, -64).view(torch.bfloat16)      # 0xffc0
    y = (at.squeeze(1).int() + 1) % vocab
    assert torch.equal(ctx.fp8_rollout_logprob(nan, y), ctx.fp8_rollout_logprob(lowest, y))
    ctx.close()


@pytest.mark.parametrize("dtype,vocab", [(torch.bfloat16, v) for v in (6144, 6152, 8192, 12_792, 12_800, 12_801, 12_808, 14_336, 14_344, 16_384, 16_391)]
                         + [(torch.float32, v) for v in (1020, 1024, 1025, 1028, 3072, 3076, 4096, 4099, 4100)])
def test_rows_with_a_compute_unit_each(dtype, vocab):
    """Up to 256 rows, where kernels that hold a row take narrower ones: both sides of the lines, in rows and in width,
    with NaNs (the two kinds of kernel agree on their codes)."""
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    pitch = -(-vocab // 8) * 8                                # aligned rows, also of odd width
    for rows in (1, 255, 256, 257):
        z = (torch.randn(rows, pitch, generator=gen, device="cuda") * 3).to(dtype)[:, :vocab]
        z[::3, vocab // 3] = float("nan")
        z[::6, vocab // 3] = -z[::6, vocab // 3]
        y = torch.randint(0, vocab // 3, (rows,), generator=gen, device="cuda", dtype=torch.int32)
        # (codes of odd width lie differently from their logits: element by element, where a NaN is -448 in every row)
        want, s = reference(z, dtype == torch.bfloat16 and pitch == vocab)
        codes, scale = ctx.fp8_quantize_rows(z)
        assert torch.equal(scale, s) and torch.equal(codes, want), rows
        back = reference(z, dtype == torch.bfloat16)[0].view(torch.float8_e4m3fn).double() * s.double().unsqueeze(1)
        ref = torch.log_softmax(back, dim=1).gather(1, y.long().unsqueeze(1)).squeeze(1)
        # fp32 log-sum-exp minus an fp32 logit, both of up to 20: a few ulp of 2^-19
        assert (ctx.fp8_rollout_logprob(z, y).double() - ref).abs().max() < 8e-6, rows
        flat = reference(torch.nan_to_num(z), False)
        for out in (torch.float32, torch.bfloat16):
            assert torch.equal(ctx.fp8_dequantize_rows(flat[0], flat[1], out),
                               (flat[0].view(torch.float8_e4m3fn).float() * flat[1].unsqueeze(1)).to(out)), rows
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("vocab", [8, 65, 1000, 4096, 12_808, 16_384, 16_385, 16_392])
def test_rows_with_infinities(dtype, vocab):
    """An infinite scale: infinities and NaNs are -448, everything else a zero of its own sign, in the kernels that stream a row
    and in those that hold it; rows without one, beside them, are as ever."""
    ctx = B.AisContext()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    for rows in (6, 300):
        z = (torch.randn(rows, vocab, generator=gen, device="cuda") * 3).to(dtype)
        plain, _ = reference(z, False)
        z[0::6, vocab // 2] = float("inf")
        z[1::6, vocab // 3] = -float("inf")
        z[2::6, vocab - 1] = float("inf")
        z[2::6, 0] = -float("inf")
        z[3::6, vocab // 2] = float("inf")
        z[3::6, 1] = float("nan")
        z[4::6] = -float("inf")
        codes, scale = ctx.fp8_quantize_rows(z)
        special = z.isnan() | z.isinf()
        want = torch.where(special, 0xFE, torch.signbit(z).to(torch.uint8) << 7)
        want[5::6] = plain[5::6]
        assert torch.equal(codes, want.to(torch.uint8)), rows
        infinite = torch.arange(rows, device="cuda") % 6 != 5
        assert torch.equal(scale.isinf(), infinite) and bool((scale > 0).all())
        y = torch.randint(0, vocab, (rows,), generator=gen, device="cuda", dtype=torch.int32)
        logp = ctx.fp8_rollout_logprob(z, y)
        back = plain.view(torch.float8_e4m3fn).double() * scale.double().unsqueeze(1)
        ref = torch.log_softmax(back, dim=1).gather(1, y.long().unsqueeze(1)).squeeze(1)
        # fp32 log-sum-exp minus an fp32 logit, both of up to 20: a few ulp of 2^-19
        assert (logp.double() - ref)[~infinite].abs().max() < 8e-6, rows
    ctx.close()
