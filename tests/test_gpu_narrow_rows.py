"""Narrow rows that are not 16-byte aligned, many of them: bound by the number of wavefronts in flight, not by bytes, so a
kernel that gives every row a workgroup of 1,024 threads takes several times as long as it should.  Each call is timed
against another route that the library has for the same rows."""
import pytest
import torch

from paper_2605_13907_amd import binding as B
from tests import parity as P
from tests.test_gpu_one_sweep import check_one_sweep
from tests.test_gpu_unaligned_rows import batch_at

pytestmark = pytest.mark.gpu

ROWS = 8192
SLACK = 1.35            # routes that are equally good differ by less


@pytest.fixture(scope="module")
def ctx():
    c = B.AisContext()
    yield c
    c.close()


def kernel_us(ctx, which, call, n=20):
    """Smallest time of the named kernel over several rounds of n launches."""
    times = []
    for _ in range(4):
        call()
        ctx.profile(True)
        for _ in range(n):
            call()
        ms, launches = ctx.profile_read(which)
        ctx.profile(False)
        times.append(ms * 1e3 / launches)
    return min(times)


def logits(vocab, dtype, offset=0, pitch=None):
    """[ROWS, vocab] of row pitch `pitch`, `offset` elements into its buffer."""
    pitch = pitch or vocab
    room = torch.randn(ROWS * pitch + offset, device="cuda").mul_(3.0).to(dtype)
    return room[offset:].view(ROWS, pitch)[:, :vocab]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("vocab", [1, 63, 501, 1001, 3001])
def test_gradient(ctx, vocab, dtype):
    z, y = logits(vocab, dtype), torch.randint(0, vocab, (ROWS,), device="cuda", dtype=torch.int32)
    logp, lse = ctx.token_logprob(z, y)
    cu, rewards = torch.tensor([0, ROWS], device="cuda"), torch.ones(1, device="cuda")
    adv, count, diag = ctx.diagnostics(logp, logp, None, cu, rewards, 1)
    adv.fill_(1.0)
    beside = torch.empty(ROWS * vocab + 1, dtype=dtype, device="cuda")
    same, other = beside[:-1].view(ROWS, vocab), beside[1:].view(ROWS, vocab)      # other: not the logits' lines

    def time(out):
        return kernel_us(ctx, B.AIS_K_DLOGITS, lambda: ctx.grpo_loss_grad(z, y, None, cu, logp, lse, logp, adv, count, diag,
                                                                          dlogits=out))

    vectors, single = time(same), time(other)
    assert vectors <= SLACK * single, (vectors, single)


# where the routes change: element by element below 2 KiB, up to 1,024 vectors with 256 threads a row, 1,024 beyond
@pytest.mark.parametrize("dtype,vocab", [("bf16", v) for v in (1023, 1025, 1087, 4099, 8191, 8199, 8201)] +
                         [("f32", v) for v in (511, 513, 543, 2051, 4095, 4099, 4101)])
def test_route_edges(ctx, dtype, vocab):
    for pitch, offset in ((vocab, 0), (vocab + 1, 3), (vocab + 6, 1)):
        print("vocab", vocab, dtype, "pitch", pitch, "offset", offset, flush=True)
        batch, room = batch_at(vocab, dtype, pitch, offset, vocab)
        P.check(ctx, batch)
        check_one_sweep(ctx, batch)
        P.check(ctx, batch, in_place=True)
        assert bool((room[:offset] == 77.0).all()) and bool((room[offset + batch.n_rows * pitch:] == 77.0).all())
        if pitch > vocab:
            gap = room[offset:offset + batch.n_rows * pitch].view(batch.n_rows, pitch)[:, vocab:]
            assert bool((gap == 77.0).all()), "elements between the rows were written"
