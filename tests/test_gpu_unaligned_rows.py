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
