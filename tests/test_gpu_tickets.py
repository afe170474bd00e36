"""The counters by which a reduction finds its last workgroup.  The static diagnostics call has counters of its own and
may run beside the other calls of its context; and a count that overlapping launches left behind (the contract forbids
them) costs one call, not every later one."""
import ctypes as C

import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu


def scalars(rows, n_resp, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    logp = -torch.rand(rows, generator=g, device="cuda")
    roll = logp + 0.1 * torch.randn(rows, generator=g, device="cuda")
    cu = torch.linspace(0, rows, n_resp + 1, device="cuda", dtype=torch.float64).long()
    rewards = (torch.rand(n_resp, generator=g, device="cuda") < 0.5).float()
    return logp, roll, None, cu, rewards, n_resp


def bits(*tensors):
    return [t.contiguous().view(torch.uint8).clone() for t in tensors]


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def reduce_both(ctx, args):
    adv, count, diag = ctx.diagnostics(*args)
    loss, wtilde, g = ctx.grpo_row_scale(*args[:4], adv, count, diag)
    return adv, count, diag, loss, wtilde, g


def test_static_call_beside_the_others():
    """A graph that holds the static call is replayed on one stream while the context works on another."""
    ctx = B.AisContext()
    a, b = scalars(400_000, 64, 1), scalars(300_000, 1500, 2)
    reduce_both(ctx, b)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        held = ctx.diagnostics(*a, static_scratch=True)
    graph.replay()
    ref_a, ref_b = bits(*held), bits(*reduce_both(ctx, b))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for it in range(20):
        for t in held:
            t.zero_()
        torch.cuda.synchronize()
        for _ in range(10):
            with torch.cuda.stream(streams[0]):
                graph.replay()
            with torch.cuda.stream(streams[1]):
                out = reduce_both(ctx, b)
        torch.cuda.synchronize()
        assert same(bits(*held), ref_a) and same(bits(*out), ref_b), it
    assert ctx.status() == 0
    ctx.close()


class ContextHead(C.Structure):
    _fields_ = [("device", C.c_int), ("stream", C.c_void_p), ("ws", C.c_void_p), ("ws_bytes", C.c_size_t),
                ("status_dev", C.c_void_p)]


class StatusWords:
    """The context's status allocation (64 words: status, tickets at 32, 33 and 48, 49) as an array that torch can view."""

    def __init__(self, ctx):
        head = C.cast(ctx._h, C.POINTER(ContextHead)).contents
        self.__cuda_array_interface__ = {"shape": (64,), "typestr": "<i4", "data": (head.status_dev, False), "version": 2}


@pytest.mark.parametrize("static", [False, True])
def test_a_count_that_was_left_behind(static):
    ctx = B.AisContext()
    args = scalars(100_000, 16, 3)
    run = (lambda: ctx.diagnostics(*args, static_scratch=True)) if static else (lambda: reduce_both(ctx, args))
    ref = bits(*run())
    words = torch.as_tensor(StatusWords(ctx), device="cuda")
    torch.cuda.synchronize()
    assert bool((words == 0).all())
    for word in (32, 33, 48, 49):
        words[word] = 3
        run()                                       # its results may be lost: nobody is the last of its workgroups
        run()
        got = bits(*run())
        torch.cuda.synchronize()
        mine = word >= 48 if static else word < 48
        assert same(got, ref), word
        assert int(words[word]) == (0 if mine else 3)
        words[word] = 0
    assert bool((words == 0).all()) and ctx.status() == 0
    ctx.close()


@pytest.mark.parametrize("static", [False, True])
def test_a_count_left_behind_with_small_batches_between(static):
    """A batch of few tiles is reduced by one workgroup, which takes no ticket: it must not use up a turn either, or the
    large batches between such ones come to the same ticket every time and nobody clears it."""
    ctx = B.AisContext()
    large, small = scalars(100_000, 16, 3), scalars(512, 8, 4)
    diagnostics = lambda args: ctx.diagnostics(*args, static_scratch=static)
    ref, ref_small = bits(*diagnostics(large)), bits(*diagnostics(small))
    words = torch.as_tensor(StatusWords(ctx), device="cuda")
    torch.cuda.synchronize()
    for word in (48, 49) if static else (32, 33):
        words[word] = 1 << 20                       # more than there are workgroups: nobody is the last one of a launch
        for _ in range(3):                          # the results of one of these may be lost
            diagnostics(large)
            assert same(bits(*diagnostics(small)), ref_small)
        for _ in range(3):
            got = bits(*diagnostics(large))
            assert same(got, ref), word
            assert same(bits(*diagnostics(small)), ref_small)
        assert bool((words == 0).all()), word
    assert ctx.status() == 0
    ctx.close()
