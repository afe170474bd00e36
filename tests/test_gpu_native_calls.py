"""The binding's native calls against the methods' own way: same results to the bit, same refusals."""
import numpy as np
import pytest
import torch

from paper_2605_13907_amd import binding as B
from paper_2605_13907_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture
def both():
    fast, slow = B.AisContext(), B.AisContext()
    assert fast._fast is not None, "the native calls have not been built"
    slow._fast = None
    yield fast, slow
    fast.close()
    slow.close()


def flat(out):
    if out is None:
        return [None]
    if isinstance(out, torch.Tensor):
        return [out]
    return [t for o in (out.values() if isinstance(out, dict) else out) for t in flat(o)]


def same(a, b):
    a, b = flat(a), flat(b)
    torch.cuda.synchronize()
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert (x is None) == (y is None)
        if x is None:
            continue
        assert x.dtype == y.dtype and x.shape == y.shape and x.stride() == y.stride() and x.device == y.device
        assert torch.equal(x.contiguous().view(torch.uint8), y.contiguous().view(torch.uint8))


def calls(ctx, batch, params, stale):
    """Every call, on one batch; a generator, so that both ways go through them side by side."""
    z, y, v = batch.logits, batch.token_ids, batch.valid
    old = ref = None
    logp, lse = ctx.token_logprob(z, y, v, params.inv_temperature)
    yield logp, lse
    if stale:
        old, ref = logp - 0.01, logp - 0.02
    adv, count, diag = ctx.diagnostics(logp if old is None else old, batch.logp_roll, v, batch.cu_rows, batch.rewards,
                                       batch.shape.group_size, params)
    yield adv, count, diag
    args = (adv, count, diag, params, old, ref)
    yield ctx.grpo_loss_grad(z, y, v, batch.cu_rows, logp, lse, batch.logp_roll, *args)
    yield ctx.grpo_loss_grad(z, y, v, batch.cu_rows, logp, lse, batch.logp_roll, *args, dlogits=torch.empty_like(z),
                             want_wtilde=False)
    yield ctx.grpo_loss_grad(z[:, 3:-2], y.clamp(max=z.shape[1] - 6), v, batch.cu_rows, logp, lse, batch.logp_roll, adv, count,
                             diag)[:2]
    yield ctx.grpo_row_scale(logp, batch.logp_roll, v, batch.cu_rows, *args)
    yield ctx.token_logprob_softmax_grad(z, y, v)
    yield ctx.token_logprob_softmax_grad(z.clone(), y, v, 0.5, sgrad=torch.zeros_like(z))
    codes, scale = ctx.fp8_quantize_rows(z)
    yield codes, scale
    yield ctx.fp8_dequantize_rows(codes, scale), ctx.fp8_dequantize_rows(codes[:, 1:], scale, torch.bfloat16)
    yield ctx.fp8_rollout_logprob(z, y, v)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    h = torch.randn(z.shape[0], 64, generator=g, device="cuda").bfloat16()
    w = torch.nn.Parameter(torch.randn(z.shape[1], 64, generator=g, device="cuda").bfloat16(), requires_grad=False)
    logp, lse = ctx.lm_head_logprob(h, w, y, v)
    yield logp, lse
    yield ctx.lm_head_grad(h, w, y, lse, logp, torch.where(v.bool(), 1.0, 0.0))
    yield ctx.lm_head_grad(h, w, y, lse, logp, torch.where(v.bool(), 1.0, 0.0), 1.0, 256, int(v.sum()))
    yield ctx.step(batch, params, old, ref)
    yield ctx.step_one_sweep(batch, params, old, ref)


@pytest.mark.parametrize("config", [1, 3])
@pytest.mark.parametrize("stale", [False, True])
def test_same_results(both, config, stale):
    shape = workloads.config(config)
    if config != 1:
        shape = shape.scaled(vocab=2_000, len_div=64)
    batch = workloads.generate(shape, "cuda")
    params = B.default_params(beta_kl=0.04, inv_temperature=0.9) if stale else B.default_params()
    n = 0
    for a, b in zip(calls(both[0], batch, params, stale), calls(both[1], batch, params, stale)):
        same(a, b)
        n += 1
    assert n == 16


def test_own_stream(both):
    z = torch.randn(300, 5000, device="cuda").bfloat16()
    y = torch.randint(0, 5000, (300,), device="cuda", dtype=torch.int32)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        out = both[0].token_logprob(z, y)
    stream.synchronize()
    same(out, both[1].token_logprob(z, y))


def test_same_refusals(both):
    z = torch.randn(8, 64, device="cuda")
    y = torch.zeros(8, device="cuda", dtype=torch.int32)
    f = torch.zeros(8, device="cuda")
    cu = torch.tensor([0, 8], device="cuda")
    one = torch.ones(1, device="cuda")

    class Sub(torch.Tensor):
        pass

    def outcome(call):
        try:
            out = call()
        except Exception as e:
            return type(e), str(e)
        torch.cuda.synchronize()
        return [None if t is None else t.float().cpu().numpy().tobytes() for t in flat(out)]

    bad = [
        lambda c: c.token_logprob(z.cpu(), y), lambda c: c.token_logprob(z, y.long()), lambda c: c.token_logprob(z, y[:7]),
        lambda c: c.token_logprob(z.t(), y), lambda c: c.token_logprob(z.half(), y), lambda c: c.token_logprob(z, y, f),
        lambda c: c.token_logprob(z, y, None, -1.0), lambda c: c.token_logprob(z, y, None, float("nan")),
        lambda c: c.token_logprob(None, y), lambda c: c.token_logprob(z, None), lambda c: c.token_logprob(z[0], y),
        lambda c: c.token_logprob(z.as_subclass(Sub), y), lambda c: c.token_logprob(z[:, ::2], y),
        lambda c: c.token_logprob(z[::2], y[::2].contiguous()), lambda c: c.token_logprob(z[::2], y[::2]),
        lambda c: c.token_logprob(z[:0], y[:0]), lambda c: c.token_logprob(z[:1], y[:1]),
        lambda c: c.token_logprob_softmax_grad(z, y, sgrad=z[:4]), lambda c: c.token_logprob_softmax_grad(z, y, sgrad=z.bfloat16()),
        lambda c: c.diagnostics(f, f, None, cu, one, 2), lambda c: c.diagnostics(f, f, None, cu, one, 0),
        lambda c: c.diagnostics(f, f, None, cu.int(), one, 1), lambda c: c.diagnostics(f, f[:4], None, cu, one, 1),
        lambda c: c.diagnostics(f, f, None, cu, one, 1, B.default_params(C=0.5)), lambda c: c.diagnostics(f, f, None, cu, one, 1),
        lambda c: c.grpo_row_scale(f, f, None, cu, one, one, one), lambda c: c.fp8_quantize_rows(z.double()),
        lambda c: c.fp8_dequantize_rows(z, f), lambda c: c.fp8_dequantize_rows(torch.zeros(8, 64, device="cuda", dtype=torch.uint8), f, torch.float16),
        lambda c: c.lm_head_logprob(z, z, y), lambda c: c.lm_head_logprob(z.bfloat16(), z.bfloat16()[:, :32], y),
        lambda c: c.lm_head_logprob(z.bfloat16()[:, :60].contiguous(), z.bfloat16()[:, :60].contiguous(), y),
    ]
    for i, call in enumerate(bad):
        a, b = outcome(lambda: call(both[0])), outcome(lambda: call(both[1]))
        assert a == b, (i, a, b)
    both[0].close()
    both[1].close()
    assert outcome(lambda: both[0].token_logprob(z, y)) == outcome(lambda: both[1].token_logprob(z, y))


def bad_forms(t):
    """t on the host, of another type, one element (row) short, and with gaps between its elements."""
    yield t.cpu()
    yield t.to(torch.float64)
    yield t[:-1]
    yield torch.stack([t, t], dim=-1).flatten(-2)[..., ::2]


def test_one_wrong_argument_at_a_time(both):
    """Every array of every call: refused by both ways, before anything is launched, with the same error."""
    n, v, d = 8, 64, 32
    f = torch.zeros(n, device="cuda")
    z, y, valid = torch.randn(n, v, device="cuda"), torch.zeros(n, device="cuda", dtype=torch.int32), torch.ones(n, device="cuda").byte()
    cu, r = torch.tensor([0, 3, 5, 8], device="cuda"), torch.ones(3, device="cuda")
    count, diag = torch.full((3,), 2, device="cuda", dtype=torch.int32), torch.zeros(B.C.sizeof(B.AisDiag), device="cuda", dtype=torch.uint8)
    h, w, codes = torch.randn(n, d, device="cuda").bfloat16(), torch.randn(v, d, device="cuda").bfloat16(), torch.zeros(n, v, device="cuda").byte()
    rows = dict(logp_train=f, logp_roll=f, valid=valid, cu_rows=cu)
    loss = dict(adv=r, count=count, diag=diag, logp_old=f, logp_ref=f)
    calls = {
        "token_logprob": dict(logits=z, token_ids=y, valid=valid),
        "token_logprob_softmax_grad": dict(logits=z, token_ids=y, valid=valid, sgrad=z.clone()),
        "diagnostics": dict(rows, rewards=r, group_size=3),
        "grpo_loss_grad": dict(rows, **loss, logits=z, token_ids=y, lse=f, dlogits=z.clone()),
        "grpo_row_scale": dict(rows, **loss),
        "fp8_quantize_rows": dict(logits=z),
        "fp8_dequantize_rows": dict(codes=codes, scale=f),
        "fp8_rollout_logprob": dict(logits=z, token_ids=y, valid=valid),
        "lm_head_logprob": dict(hidden=h, weight=w, token_ids=y, valid=valid),
        "lm_head_grad": dict(hidden=h, weight=w, token_ids=y, lse=f, logp=f, coeff=f),
    }
    sized_by_others = {("fp8_quantize_rows", "logits"), ("lm_head_logprob", "weight"), ("lm_head_grad", "weight")}
    for name, args in calls.items():
        same(getattr(both[0], name)(**args), getattr(both[1], name)(**args))
        for arg, t in args.items():
            if not isinstance(t, torch.Tensor):
                continue
            for k, wrong in enumerate(bad_forms(t)):
                if k == 2 and (name, arg) in sized_by_others:
                    continue                                   # as many rows as it has
                errors = []
                for ctx in both:
                    with pytest.raises((TypeError, ValueError)) as e:
                        getattr(ctx, name)(**{**args, arg: wrong})
                    errors.append((type(e.value), str(e.value)))
                assert errors[0] == errors[1], (name, arg, k)
    # what only an output can have wrong: other strides, and the logits' type
    wide = torch.zeros(n, v + 8, device="cuda")[:, :v]
    for ctx in both:
        for out in (wide, z.bfloat16()):
            with pytest.raises(ValueError):
                ctx.grpo_loss_grad(**{**calls["grpo_loss_grad"], "dlogits": out})
            with pytest.raises(ValueError):
                ctx.token_logprob_softmax_grad(**{**calls["token_logprob_softmax_grad"], "sgrad": out})


def test_storage_that_refuses_its_address(both):
    """A C++ exception in the middle of a native call: the method's own way raises it, and the interpreter goes on."""
    z, y = torch.randn(8, 64, device="cuda"), torch.zeros(8, device="cuda", dtype=torch.int32)
    h = z.bfloat16()
    f, codes = torch.zeros(8, device="cuda"), torch.zeros(8, 64, device="cuda", dtype=torch.uint8)
    for t in (z, h, codes):
        torch._C._set_throw_on_mutable_data_ptr(t)
    for call in (lambda c: c.token_logprob(z, y), lambda c: c.token_logprob_softmax_grad(z, y), lambda c: c.fp8_quantize_rows(z),
                 lambda c: c.fp8_dequantize_rows(codes, f), lambda c: c.fp8_rollout_logprob(z, y),
                 lambda c: c.lm_head_logprob(h, h, y), lambda c: c.lm_head_grad(h, h, y, f, f, f)):
        for ctx in both:
            with pytest.raises(RuntimeError, match="Cannot access data pointer"):
                call(ctx)
    torch.cuda.synchronize()


def test_outputs_are_new_tensors(both):
    z = torch.randn(64, 1000, device="cuda")
    y = torch.randint(0, 1000, (64,), device="cuda", dtype=torch.int32)
    a, b = both[0].token_logprob(z, y), both[0].token_logprob(z, y)
    ptrs = {t.data_ptr() for t in (*a, *b)}
    assert len(ptrs) == 4 and not any(t.requires_grad for t in a)
    np.testing.assert_array_equal(a[0].cpu().numpy(), b[0].cpu().numpy())
