"""The scalar kernels where rows are dealt out evenly to workgroups and wavefronts, whatever responses they belong to: around
the number of rows that one workgroup takes on alone, runs of one to more than eight turns of 64 rows, responses that begin and
end inside a wavefront's 64 rows, empty ones, and one response over most workgroups beside many short ones."""
import numpy as np
import pytest

from tests import test_gpu_scalars_at_scale as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_resp,recipe", [
    (1, ("fixed", 63)), (1, ("fixed", 2_048)), (1, ("fixed", 2_049)), (3, ("fixed", 683)), (683, ("fixed", 3)),
    (1_024, ("uniform", 0, 3)), (1_024, ("uniform", 0, 130)), (33, ("fixed", 64)), (32, ("fixed", 65)),
    (5, ("fixed", 52_429)), (7, ("fixed", 320_001)), (1, ("fixed", 1_048_577)),
    # 10, 32, 32, 33 and 65 workgroups, 256 of them with 1,024 rows each and with one row more
    (128, ("fixed", 19)), (2, ("fixed", 4_096)), (1, ("fixed", 32_768)), (1, ("fixed", 32_769)), (1, ("fixed", 65_537)),
    (4, ("fixed", 65_536)), (1, ("fixed", 262_145)),
])
def test_rows_dealt_out(monkeypatch, n_resp, recipe):
    for share in (1.0, 0.6):
        monkeypatch.setitem(S.CASES, "dealt", (n_resp, 1, recipe, share))
        S.test_scalars_at_scale("dealt", share < 1.0)


@pytest.mark.parametrize("at", [0, 500, 1_000])
def test_one_long_response_among_short_ones(monkeypatch, at):
    """Its valid rows are counted by every workgroup; most others lie with many more in one of them."""
    def lengths(recipe, n, rng):
        out = rng.integers(0, 4, size=n).astype(np.int64)
        out[at] = 400_000
        return out

    monkeypatch.setattr(S, "lengths", lengths)
    monkeypatch.setitem(S.CASES, "skewed", (1_001, 1, ("own",), 0.5))
    S.test_scalars_at_scale("skewed", False)
    S.test_scalars_at_scale("skewed", True)
