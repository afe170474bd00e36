"""The rows of a batch and their responses: rows dealt out evenly, each finding its response, for up to 1,024 responses, tiles laid
out by a kernel of its own beyond that."""
import numpy as np
import pytest
import torch

from paper_2605_13907_amd import binding as B
from tests import test_gpu_scalars_at_scale as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_resp", [1, 2, 3, 5, 31, 64, 129, 255, 256, 257, 1023, 1024, 1025])
def test_number_of_responses(monkeypatch, n_resp):
    # lengths around whole tiles of 1,024 rows, empty responses, and (few responses) chains of many tiles
    recipe = ("uniform", 0, 2_050 if n_resp > 64 else 70_000)
    monkeypatch.setitem(S.CASES, "tiling", (n_resp, 1 if n_resp % 2 else 2, recipe, 0.7))
    S.test_scalars_at_scale("tiling", False)
    S.test_scalars_at_scale("tiling", True)


@pytest.mark.parametrize("n_resp,length", [(1, 1), (1, 3_840), (1, 3_841), (8, 256), (8, 257), (2, 393_216), (2, 393_217),
                                           (1024, 64), (1023, 65)])
def test_edges_of_the_tile_rule(monkeypatch, n_resp, length):
    """One row; responses that end with a run of 64 rows and inside one, over one workgroup and over all; as many responses as a
    workgroup has threads."""
    monkeypatch.setitem(S.CASES, "edge", (n_resp, 1, ("fixed", length), 0.6))
    S.test_scalars_at_scale("edge", False)
    S.test_scalars_at_scale("edge", True)


@pytest.mark.parametrize("n_resp", [2, 512, 1024, 1025])       # 512: one workgroup, the offsets in eight wavefronts
@pytest.mark.parametrize("fault", ["first", "last", "order", "range"])
def test_row_offsets_that_are_no_partition(n_resp, fault):
    """Reported, and nothing is read out of range: the offsets are clamped wherever they point."""
    rows = 4 * n_resp
    cu = torch.arange(0, rows + 1, 4, dtype=torch.int64)
    if fault == "first":
        cu[0] = 1
    elif fault == "last":
        cu[-1] = rows - 1
    elif fault == "order":
        cu[1] = -5
    else:
        cu[1] = 10 ** 12
    ctx = B.AisContext()
    logp = -torch.rand(rows, device="cuda")
    rewards = torch.zeros(n_resp, device="cuda")
    rewards[0] = 1.0
    good = torch.arange(0, rows + 1, 4, dtype=torch.int64, device="cuda")
    assert ctx.status() == 0
    _, _, diag = ctx.diagnostics(logp, logp, None, good, rewards, 1)
    assert ctx.read_diag(diag)["status"] == 0 and ctx.read_diag(diag)["n_valid"] == rows
    _, _, diag = ctx.diagnostics(logp, logp, None, cu.cuda(), rewards, 1)
    assert ctx.read_diag(diag)["status"] & B.STATUS_BAD_CU
    assert ctx.status() & B.STATUS_BAD_CU
    _, _, diag = ctx.diagnostics(logp, logp, None, good, rewards, 1)     # the next call is none the worse for it
    d = ctx.read_diag(diag)
    assert d["status"] == 0 and d["n_valid"] == rows and np.isclose(d["mean_w"], 1.0)
    ctx.close()
