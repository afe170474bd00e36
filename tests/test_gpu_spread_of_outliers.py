"""Spreads of values that lie close together, far from the one that the sums begin with: the first row of the batch, of every
workgroup or of every thread is truncated, the others have ratios near 1.  Against extended precision."""
import numpy as np
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("every", [0, 64, 1024])                      # outliers: the first row, and every so many
@pytest.mark.parametrize("rows,n_resp", [(2000, 8), (3000, 8), (20_000, 128), (41_643, 16), (1_200_000, 1024), (1_200_000, 1100)])
def test_spread(rows, n_resp, every):
    rng = np.random.default_rng(rows + every)
    roll = -rng.random(rows).astype(np.float32) * 3
    train = (roll + rng.normal(0, 1e-3, rows)).astype(np.float32)
    train[0] = roll[0] + 4
    if every:
        train[::every] = roll[::every] + 4
    cu = np.linspace(0, rows, n_resp + 1).astype(np.int64)
    rewards = np.tile(np.array([1.0, 0.0], np.float32), n_resp // 2)
    ctx = B.AisContext()
    t = lambda a: torch.from_numpy(a).cuda()
    adv, _, diag = ctx.diagnostics(t(train), t(roll), None, t(cu), t(rewards), 2, B.default_params())
    d = ctx.read_diag(diag)
    assert ctx.status() == 0
    a = np.repeat(adv.cpu().numpy().astype(np.longdouble), np.diff(cu))
    ctx.close()
    w = np.minimum(np.exp(train.astype(np.longdouble) - roll.astype(np.longdouble)), np.longdouble(5.0))
    # A spread is taken about a value for which the sum of squares is at most 16 times the spread, by sums of about 40 roundings
    # of 2^-53 in a chain: 16 * 40 * 2^-53 = 7e-14; a ratio is right to about two units of 2^-53, against deviations of 1e-3
    # 2e-13 of each
    for name, x in (("var_w", w), ("std_a", a), ("std_aw", a * w)):
        want = ((x - x.mean()) ** 2).mean()
        want = float(want if name == "var_w" else np.sqrt(want))
        print(name, d[name], "error", abs(d[name] - want) / want, flush=True)
        assert abs(d[name] - want) <= 3e-13 * want, name
