"""The FP8 table kernels find a row's extremes from the bits of its numbers, by the sign: rows with one sign only, with
zeros of either sign, and with a single number of the other sign at the places that different lanes, slots and the
elements outside the vectors hold.  Codes, scales and log-probs; rows without a positive number take no longer; and NaNs
in rows of odd width."""
import pytest
import torch

from paper_2605_13907_amd import binding as B
from tests.test_gpu_unaligned_rows import fp8_reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.AisContext()
    yield c
    c.close()


@pytest.mark.parametrize("vocab", [8, 1000, 16_393, 40_000, 100_352, 151_936, 151_937, 176_000, 184_000, 184_001, 200_064,
                                   210_007, 248_320, 250_007])
def test_signs(ctx, vocab):
    rows = 280 if vocab > 50_000 else 700              # more than the workgroups that are resident
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    z = torch.randn(rows, vocab, generator=g, device="cuda") * 3.0
    z[0::8] = -z[0::8].abs() - 0.5                     # below zero
    z[1::8] = z[1::8].abs() + 0.5                      # above zero
    z[2::8] = -0.0
    z[3::8] = 0.0
    z[4::8] = torch.log_softmax(z[4::8], 1)            # log-probabilities
    for k, r in enumerate(range(5, rows, 8)):          # below zero but for one number, here and there in the row
        z[r] = -z[r].abs() - 0.5
        z[r, (k * 1009 + (0 if k % 2 else vocab - 1)) % vocab] = (0.0, 0.25, 700.0)[k % 3]
    for k, r in enumerate(range(6, rows, 8)):          # above zero but for one
        z[r] = z[r].abs() + 0.5
        z[r, (k * 4099 + (vocab - 1 if k % 2 else 0)) % vocab] = (-0.0, -0.25, -700.0)[k % 3]
    z = z.to(torch.bfloat16)
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    code, scale, zr = fp8_reference(z.float())
    codes, s = ctx.fp8_quantize_rows(z)
    assert torch.equal(s, scale.squeeze(1)) and torch.equal(codes, code)
    logp = ctx.fp8_rollout_logprob(z, y)
    ref = zr.gather(1, y.long().unsqueeze(1)).squeeze(1) - torch.logsumexp(zr, dim=1)
    assert bool(((logp.double() - ref).abs() <= 1e-4 * ref.abs().clamp_min(1.0)).all())
    assert ctx.status() == 0


@pytest.mark.parametrize("vocab", [32_000, 151_936, 248_320])
def test_rows_below_zero_take_no_longer(ctx, vocab):
    rows = 200_000_000 // vocab
    mixed = torch.randn(rows, vocab, device="cuda").mul_(3.0).to(torch.bfloat16)
    below = -mixed.abs() - 1.0
    y = torch.randint(0, vocab, (rows,), device="cuda", dtype=torch.int32)

    def us(which, call):
        times = []
        for _ in range(4):
            call()
            ctx.profile(True)
            for _ in range(10):
                call()
            ms, launches = ctx.profile_read(which)
            ctx.profile(False)
            times.append(ms * 1e3 / launches)
        return min(times)

    for which, call in ((B.AIS_K_FP8_QUANT, ctx.fp8_quantize_rows), (B.AIS_K_FP8_LOGPROB, lambda z: ctx.fp8_rollout_logprob(z, y))):
        # reading the rows again would be half as much again; the second look at the registers is a few per cent (the best of
        # up to three attempts: another process may hold the clocks back)
        a = b = float("inf")
        for _ in range(3):
            a, b = min(a, us(which, lambda: call(mixed))), min(b, us(which, lambda: call(below)))
            print(vocab, which, round(a, 1), round(b, 1), flush=True)
            if b <= 1.2 * a:
                break
        assert b <= 1.2 * a, (which, a, b)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("vocab", [1001, 16_393, 50_257, 100_003, 151_937, 210_007, 250_007])
def test_nan_in_unaligned_rows(ctx, vocab, dtype):
    """A NaN counts as -448 times the scale, which it does not enter, in every kernel that takes rows of odd width."""
    rows = 300
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    z = torch.randn(rows, vocab, generator=g, device="cuda") * 3.0
    z[0::4] = -z[0::4].abs() - 0.5
    nan = torch.zeros(rows, vocab, dtype=torch.bool, device="cuda")
    for r in range(0, rows, 3):
        nan[r, [(r * 997) % vocab, 0 if r % 2 else vocab - 1, vocab // 2]] = True
    nan[5::50] = True                                  # nothing else in the row
    z[::6] = torch.where(nan[::6], -float("nan"), z[::6])
    z = torch.where(nan, torch.where(torch.isnan(z), z, float("nan")), z).to(dtype)
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    y[::9] = (torch.arange(rows, device="cuda")[::9] * 997 % vocab).to(torch.int32)         # some of the NaNs are sampled
    clean = torch.where(nan, 0.0, z.float())
    code, scale, zr = fp8_reference(clean)
    code = torch.where(nan, 0xfe, code)
    zr = torch.where(nan, -448.0 * scale.double(), zr)
    codes, s = ctx.fp8_quantize_rows(z)
    assert torch.equal(s, scale.squeeze(1)) and torch.equal(codes, code)
    logp = ctx.fp8_rollout_logprob(z, y)
    ref = zr.gather(1, y.long().unsqueeze(1)).squeeze(1) - torch.logsumexp(zr, dim=1)
    assert bool(((logp.double() - ref).abs() <= 1e-4 * ref.abs().clamp_min(1.0)).all())
