"""Rows that are not 16-byte aligned: a contiguous tensor of odd width, a view that starts inside a vector, logits and
gradient that lie differently relative to a line.  The kernels take the elements before a row's first 128-byte boundary
one by one and whole vectors from there on; the widths below put the first boundary, the last vector and the row-width
classes (1024 vectors per lane slot) on either side of the row's ends."""
import pytest
import torch

from paper_2605_13907_amd import binding as B
from paper_2605_13907_amd import workloads as W
from tests import parity as P
from tests.test_gpu_one_sweep import check_one_sweep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.AisContext()
    yield c
    c.close()


def batch_at(vocab, dtype, pitch, offset, seed):
    """A small batch whose logits sit `offset` elements into their buffer with rows `pitch` elements apart."""
    shape = W.RolloutShape("unaligned", n_prompts=1, group_size=4, vocab=vocab, logits_dtype=dtype, sigma=2.5, boost=4.0,
                           layout="padded", max_len=3, length_dist=("uniform", 1, 3), reward_p=0.5, seed=seed)
    batch = W.generate(shape, "cuda")
    batch.rewards[:] = torch.tensor([1, 0, 0, 1], dtype=torch.float32)
    rows = batch.n_rows
    room = torch.full((rows * pitch + offset + 64,), 77.0, dtype=batch.logits.dtype, device="cuda")
    view = room[offset:offset + rows * pitch].view(rows, pitch)[:, :vocab]
    view.copy_(batch.logits)
    batch.logits = view
    return batch, room


def edges(dtype):
    line, lane = (64, 8192) if dtype == "bf16" else (32, 4096)      # elements of a line; of one vector per lane
    return [1, 2, line - 1, line + 1, 2 * line + 3, 1001, 4 * lane - 1, 4 * lane + line - 1, 12 * lane + 1,
            12 * lane + line, 20 * lane + 5, 32 * lane + 3, 33 * lane + 1]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k", range(13))
def test_both_paths(ctx, dtype, k):
    vocab = edges(dtype)[k]
    for pitch, offset in ((vocab, 0), (vocab + 1, 3), (vocab + 6, 1)):
        print("vocab", vocab, dtype, "pitch", pitch, "offset", offset, flush=True)
        batch, room = batch_at(vocab, dtype, pitch, offset, vocab + offset)
        P.check(ctx, batch)                          # the gradient's buffer starts on a line: another place than offset
        check_one_sweep(ctx, batch)
        P.check(ctx, batch, in_place=True)
        assert bool((room[:offset] == 77.0).all()) and bool((room[offset + batch.n_rows * pitch:] == 77.0).all())
        if pitch > vocab:
            gap = room[offset:offset + batch.n_rows * pitch].view(batch.n_rows, pitch)[:, vocab:]
            assert bool((gap == 77.0).all()), "elements between the rows were written"


def fp8_reference(z):
    """Codes, scales and round trip of float32 rows by torch's own cast (true fp32 divisions)."""
    scale = z.abs().amax(dim=1, keepdim=True) / torch.full((z.shape[0], 1), 448.0, device=z.device)
    scale = torch.where(scale > 0, scale, torch.ones_like(scale))
    code = (z / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return code.view(torch.uint8), scale, code.double() * scale.double()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k", range(17))
def test_fp8(ctx, dtype, k):
    """Codes, scales and decoded values bit for bit, the log-probs to 1e-4 (the sum of up to 270,000 fp32 terms)."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    # the last two: on either side of where a workgroup of 1,024 threads takes over from one of 256
    vocab = (edges(dtype) + [127, 129] + ([16_391, 16_393] if dtype == "bf16" else [4099, 4101]))[k]
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab)
    rows = 600 if vocab < 40_000 else 5         # more rows than compute units: workgroups that walk several rows
    for pitch, offset in ((vocab, 0), (vocab + 1, 3), (vocab + 2, 6)):
        print("vocab", vocab, dtype, "pitch", pitch, "offset", offset, flush=True)
        room = torch.full((rows * pitch + offset + 64,), 77.0, dtype=dt, device="cuda")
        z = room[offset:offset + rows * pitch].view(rows, pitch)[:, :vocab]
        z.copy_(torch.randn(rows, vocab, generator=g, device="cuda") * 3.0)
        z[1] = -z[1].abs() - 1000.0             # no element above zero: the largest one decides the log-prob
        z[2] = 0.0
        z[3, 0] = 40.0                          # the abs-max outside the vectors, at either end
        z[4, vocab - 1] = -41.0
        y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
        code, scale, zr = fp8_reference(z.float())
        codes, s = ctx.fp8_quantize_rows(z)
        assert torch.equal(s, scale.squeeze(1)) and torch.equal(codes, code)
        for out in (torch.float32, torch.bfloat16):
            assert torch.equal(ctx.fp8_dequantize_rows(codes, s, out), (code.view(torch.float8_e4m3fn).float() * scale).to(out))
        logp = ctx.fp8_rollout_logprob(z, y)
        ref = zr.gather(1, y.long().unsqueeze(1)).squeeze(1) - torch.logsumexp(zr, dim=1)
        assert float((logp.double() - ref).abs().max()) <= 1e-4 * max(1.0, float(ref.abs().max()))
        assert ctx.status() == 0


@pytest.mark.parametrize("lanes", [3, 7, 11, 13, 14, 15, 16, 17, 18, 19, 20, 21, 22, 23, 24, 27, 31])
def test_fp8_many_rows(ctx, lanes):
    """More rows than the chip holds at once, in every class of vectors per lane: the registers (and from 24 vectors on
    the LDS slots) of a workgroup are refilled with its next row while this one is still being summed, and with an odd
    pitch the two rows have different heads, vector counts and rests.  Rows differ in scale by 2^10, so that an element
    of another row shows; one row in five is not evaluated."""
    vocab = lanes * 8192 - 4189
    rows = 600 if lanes > 8 else 1200
    g = torch.Generator(device="cuda")
    g.manual_seed(lanes)
    factor = torch.exp2(10.0 * torch.rand(rows, 1, generator=g, device="cuda") - 6.0)
    y = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    valid = (torch.rand(rows, generator=g, device="cuda") < 0.8).to(torch.uint8)
    for pitch, offset in ((vocab, 0), (vocab + 3, 3)):
        print("vocab", vocab, "rows", rows, "pitch", pitch, "offset", offset, flush=True)
        room = torch.full((rows * pitch + offset + 64,), 77.0, dtype=torch.bfloat16, device="cuda")
        z = room[offset:offset + rows * pitch].view(rows, pitch)[:, :vocab]
        z.copy_(torch.randn(rows, vocab, generator=g, device="cuda") * factor)
        z[5::7] = -z[5::7].abs() - 3.0
        code, scale, zr = fp8_reference(z.float())
        codes, s = ctx.fp8_quantize_rows(z)
        assert torch.equal(s, scale.squeeze(1)) and torch.equal(codes, code)
        logp = ctx.fp8_rollout_logprob(z, y, valid)
        ref = zr.gather(1, y.long().unsqueeze(1)).squeeze(1) - torch.logsumexp(zr, dim=1)
        on = valid.bool()
        err = (logp.double() - ref)[on].abs()
        assert bool((err <= 1e-4 * ref[on].abs().clamp_min(1.0)).all()), float(err.max())
        assert bool((logp[~on] == 0).all()) and ctx.status() == 0
