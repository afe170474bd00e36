"""Diagnostics of batches that hold a NaN or an infinity: every statistic that depends on it says so, those that do not are what
they are without it, and batches of up to and of more than 1,024 responses agree, on one workgroup and on several."""
import math

import numpy as np
import pytest
import torch

from paper_2605_13907_amd import binding as B

pytestmark = pytest.mark.gpu

NAN, INF = float("nan"), float("inf")
# what is put where, in a valid row 100 or as reward 3: fields that are NaN then, and mean |dp| where it has a value
FAULTS = {
    "train nan": (dict(train=NAN), {"dbar", "kl_roll_train", "mean_abs_dp"}),
    "roll nan": (dict(roll=NAN), {"dbar", "kl_roll_train", "mean_abs_dp"}),
    "both nan": (dict(train=NAN, roll=NAN), {"dbar", "kl_roll_train", "mean_abs_dp"}),
    "nan and -inf": (dict(train=NAN, roll=-INF), {"dbar", "kl_roll_train", "mean_abs_dp"}),
    "both -inf": (dict(train=-INF, roll=-INF), {"dbar", "kl_roll_train"}),       # two probabilities of 0: no difference
    "train -inf": (dict(train=-INF), set()),
    "roll -inf": (dict(roll=-INF), set()),
    "reward nan": (dict(reward=NAN), {"std_a", "std_aw"}),
    "reward inf": (dict(reward=INF), {"std_a", "std_aw"}),
    "none": (dict(), set()),
}


@pytest.mark.parametrize("n_resp,length", [(8, 40), (8, 256), (16, 300), (256, 80), (1100, 12), (1100, 3)])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("fault", list(FAULTS))
def test_diagnostics(fault, masked, n_resp, length):
    put, nans = FAULTS[fault]
    rng = np.random.default_rng(5)
    n = n_resp * length
    roll = -rng.random(n).astype(np.float32) * 3
    train = (roll + rng.normal(0, 0.05, n)).astype(np.float32)
    rewards = (rng.random(n_resp) < 0.5).astype(np.float32)
    valid = (rng.random(n) < 0.7).astype(np.uint8) if masked else None
    if masked:
        valid[100] = 1
        train[valid == 0] = NAN                     # rows that are not evaluated are not looked at
    train[100], roll[100] = put.get("train", train[100]), put.get("roll", roll[100])
    rewards[100 // length] = put.get("reward", rewards[100 // length])
    ctx = B.AisContext()
    t = lambda a: None if a is None else torch.from_numpy(a).cuda()
    adv, count, diag = ctx.diagnostics(t(train), t(roll), t(valid), t(np.arange(n_resp + 1, dtype=np.int64) * length),
                                       t(rewards), 4, B.default_params())
    d = ctx.read_diag(diag)
    assert ctx.status() == 0
    ctx.close()
    on = np.ones(n, bool) if valid is None else valid != 0
    lt, lr = train[on].astype(np.float64), roll[on].astype(np.float64)
    with np.errstate(all="ignore"):
        diff, dp = lt - lr, np.abs(np.exp(lt) - np.exp(lr))
        w = np.where(diff <= math.log(5.0), np.exp(diff), 5.0)         # a NaN counts as truncated
        want = dict(dbar=np.abs(diff).mean(), kl_roll_train=-diff.mean(), mean_abs_dp=dp.mean(), mean_w=w.mean(), var_w=w.var(),
                    clip_frac=(diff > math.log(5.0)).mean())
    assert d["n_valid"] == int(on.sum())
    for k in ("dbar", "kl_roll_train", "mean_abs_dp", "mean_w", "var_w", "clip_frac", "std_a", "std_aw"):
        assert math.isnan(d[k]) == (k in nans), (k, d[k])
        if k in want and k not in nans:
            assert d[k] == want[k] or abs(d[k] - want[k]) <= 1e-9 * max(abs(want[k]), want["mean_w"] * 1e-3), (k, d[k], want[k])
