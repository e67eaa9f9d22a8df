"""Ranking of a profiled context: both forms, and contexts at the line between them."""
import numpy as np
import pytest
import torch

from oracle import lukv_oracle as O
from paper_2602_08585_amd import lukv
from tests.helpers import dev

pytestmark = pytest.mark.gpu


def _scores(kind, T, rng):
    s = np.exp(1.5 * rng.standard_normal(T))
    if kind == "tie_48":
        s[rng.permutation(T)[:48]] = 0.25
    elif kind == "tie_49":
        s[rng.permutation(T)[:49]] = 0.25
    elif kind == "signed":
        s = rng.standard_normal(T)
        s[::7] = 0.0
        s[3::11] = -0.0
    elif kind == "infinities":
        s[T // 2] = np.inf
        s[T // 3] = -np.inf
    elif kind == "outlier":                 # all but one crowded into a bin, few of them equal
        s = 1.0 + rng.random(T) / 1024
        s[T // 2] = 1e30
    elif kind == "half_zero":
        s[rng.random(T) < 0.5] = 0.0
    elif kind == "equal":
        s[:] = 1.0
    elif kind == "distinct_bits":           # every key in its own bin, in both directions
        s = (np.arange(T, dtype=np.uint32) + 0x3F800000).view(np.float32)[::-1 if T % 2 else 1]
    return np.ascontiguousarray(s, dtype=np.float32)


@pytest.mark.parametrize("T", [1, 2, 63, 127, 129, 1024, 1025, 4095, 4096])
@pytest.mark.parametrize("kind", ["spread", "tie_48", "tie_49", "signed", "infinities", "outlier", "half_zero", "equal",
                                  "distinct_bits"])
def test_profile_ranking(T, kind):
    print("case", T, kind, flush=True)
    rng = np.random.default_rng(T)
    sc = np.stack([_scores(kind, T, rng) for _ in range(2)])
    imp = (rng.random((2, T)) ** 4).astype(np.float32)
    Gp = min(T + 1, 300)
    knots = np.tile((np.arange(Gp) * T // max(1, Gp - 1)).astype(np.int32), (2, 1))
    want = np.stack([O.utility_curve(imp[c], sc[c], knots[c]) for c in range(2)])
    got = torch.full((2, Gp), float("nan"), device="cuda")
    lukv.lukv_profile_curves(2, T, Gp, dev(imp), dev(sc), dev(knots), got)
    # sums of up to 4096 terms in 64 bits, rounded once to 32
    assert np.allclose(got.cpu().numpy(), want, rtol=1.2e-7, atol=0)
