"""Budget phase, list form: sizes around its limits, more live segments than stay in registers, units
on offer beyond 31 bits (64-bit counts), and batches of profile ratios with a remainder."""
import numpy as np
import pytest
import torch

from oracle import lukv_oracle as O
from paper_2602_08585_amd import lukv, synth
from tests.helpers import dev

pytestmark = pytest.mark.gpu


def _problem(seed, n, NH, Gp, L, concave):
    rng = np.random.default_rng(seed)
    inc = rng.gamma(0.5, size=(n, NH, Gp)) if not concave else np.sort(rng.gamma(0.5, size=(n, NH, Gp)), axis=-1)[..., ::-1]
    inc = np.round(inc * 64).astype(np.float32) / 64            # equal gains across heads
    inc[..., 0] = 0
    curves = np.cumsum(inc, axis=-1).astype(np.float32)
    knots = np.tile(synth.make_knots(L, Gp), (n, NH, 1)).astype(np.int32)
    b_min = rng.integers(0, max(1, L // 16), size=(n, NH)).astype(np.int32)
    b_max = (L - rng.integers(0, max(1, L // 16), size=(n, NH))).astype(np.int32)
    return curves, knots, b_min, b_max


@pytest.mark.parametrize("NH,Gp,L,concave,units", [
    (65, 2, 40, False, 900), (128, 8, 40, True, 3000), (100, 10, 40, False, 3500),       # (a segment a thread)
    (65, 16, 200, False, 3000), (33, 32, 500, True, 4000), (1024, 2, 9, True, 2000),
    (1024, 64, 80, True, 3000),          # 65536 knots, all of them vertices: most segments not in registers
    (33, 1980, 1990, True, 3000), (1024, 65, 80, False, 2000),       # 66560 knots: general form
    (70, 16, 1 << 25, False, 3000)])     # 2.3e9 units on offer: 64-bit counts
def test_allocate_list_form(NH, Gp, L, concave, units):
    print("case", NH, Gp, L, concave, flush=True)
    curves, knots, b_min, b_max = _problem(NH + Gp, 1, NH, Gp, L, concave)
    B = [int(b_min.sum()) + units]
    ws = lukv.alloc_workspace(lukv.lukv_allocate_workspace_bytes(1, NH, Gp))
    budgets = torch.full((NH,), -7, dtype=torch.int32, device="cuda")
    offsets = torch.full((NH + 1,), -7, dtype=torch.int64, device="cuda")
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    lukv.lukv_allocate(1, NH, Gp, dev(curves), dev(knots), dev(b_min), dev(b_max), B, budgets, offsets, status, ws)
    want, st = O.allocate(curves[0], knots[0], b_min[0], b_max[0], B[0])
    assert np.array_equal(budgets.cpu().numpy(), want)
    assert np.array_equal(offsets.cpu().numpy(), O.offsets_of(want))
    assert int(status.cpu()[0]) == st == 0


@pytest.mark.parametrize("M,NH,Gp,L,n_rho", [(1, 8, 16, 60, 1), (3, 65, 17, 40, 33), (2, 100, 16, 30, 32),
                                             (2, 9, 8, 50, 65), (1, 1030, 4, 5, 3)])
def test_profile_batches(M, NH, Gp, L, n_rho):
    print("case", M, NH, Gp, L, n_rho, flush=True)
    curves, knots, b_min, b_max = _problem(7 * NH + n_rho, M, NH, Gp, L, False)
    rho = [(i + 0.5) / n_rho for i in range(n_rho)]
    want = O.profile_build(curves, knots, b_min, b_max, L, rho)
    phi = torch.full((n_rho, NH), float("nan"), device="cuda")
    ws = lukv.alloc_workspace(lukv.lukv_profile_workspace_bytes(M, NH, Gp))
    ws.fill_(255)
    lukv.lukv_profile_build(M, NH, Gp, dev(curves.reshape(M * NH, Gp)), dev(knots.reshape(M * NH, Gp)), dev(b_min),
                            dev(b_max), L, rho, phi, ws)
    assert np.array_equal(phi.cpu().numpy(), want)


# The oracle hands units out one by one, so problems of more than 2^31 units are small ones with every
# count multiplied by a power of two: gains are divided by it exactly, so the order of the segments, the
# ties and the shares stay, and the budgets are the small problem's times the same factor.
SCALE = 1 << 20


@pytest.mark.parametrize("NH,Gp,L,units", [(70, 16, 40, 3), (70, 16, 40, 2350), (1024, 9, 12, 5000), (65, 33, 60, 2900),
                                           (100, 10, 40, 3000)])
def test_allocate_many_units(NH, Gp, L, units):
    print("case", NH, Gp, L, units, flush=True)
    curves, knots, b_min, b_max = _problem(NH + units, 1, NH, Gp, L, False)
    offer = int((np.minimum(b_max, knots[..., -1]) - b_min).sum())
    assert offer >= units and offer * SCALE >= 1 << 31
    small, st = O.allocate(curves[0], knots[0], b_min[0], b_max[0], int(b_min.sum()) + units)
    want = small.astype(np.int64) * SCALE
    ws = lukv.alloc_workspace(lukv.lukv_allocate_workspace_bytes(1, NH, Gp))
    ws.fill_(255)
    budgets = torch.full((NH,), -7, dtype=torch.int32, device="cuda")
    offsets = torch.full((NH + 1,), -7, dtype=torch.int64, device="cuda")
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    lukv.lukv_allocate(1, NH, Gp, dev(curves), dev(knots * SCALE), dev(b_min * SCALE), dev(b_max * SCALE),
                       [(int(b_min.sum()) + units) * SCALE], budgets, offsets, status, ws)
    assert np.array_equal(budgets.cpu().numpy(), want)
    assert np.array_equal(offsets.cpu().numpy(), O.offsets_of(want))
    assert int(status.cpu()[0]) == st == 0


def test_profile_many_units():
    M, NH, Gp, L, n_rho = 2, 80, 16, 40, 16
    curves, knots, b_min, b_max = _problem(11, M, NH, Gp, L, False)
    assert all(int((np.minimum(b_max[m], knots[m, :, -1]) - b_min[m]).sum()) * SCALE >= 1 << 31 for m in range(M))
    rho = [i / n_rho for i in range(n_rho)]          # (every total is a whole number of units at both scales)
    want = O.profile_build(curves, knots, b_min, b_max, L, rho)
    phi = torch.full((n_rho, NH), float("nan"), device="cuda")
    ws = lukv.alloc_workspace(lukv.lukv_profile_workspace_bytes(M, NH, Gp))
    ws.fill_(255)
    lukv.lukv_profile_build(M, NH, Gp, dev(curves.reshape(M * NH, Gp)), dev(knots.reshape(M * NH, Gp) * SCALE),
                            dev(b_min * SCALE), dev(b_max * SCALE), L * SCALE, rho, phi, ws)
    assert np.array_equal(phi.cpu().numpy(), want)
