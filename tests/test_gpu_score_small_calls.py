"""Score kernels in calls that leave the chip idle: chunks cut finer, rows of a chunk shared out over
workgroups.  The scores are bit for bit those of the same layer inside a call that fills the chip."""
import pytest
import torch

from paper_2602_08585_amd import lukv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,d,group,w,lens,layers", [
    (torch.bfloat16, 128, 4, 32, [513], 160),          # two chunks, the second with one key
    (torch.bfloat16, 128, 4, 32, [4001], 160),
    (torch.bfloat16, 128, 7, 16, [700, 97, 2048], 120),     # 112 rows: the last block half full
    (torch.bfloat16, 64, 7, 64, [1500], 160),          # 448 rows: 14 blocks, four wave groups, the last part half empty
    (torch.bfloat16, 128, 5, 32, [129], 200),          # 160 rows: five blocks, two wave groups
    (torch.float32, 64, 2, 16, [1024], 160),
    (torch.float32, 128, 3, 32, [640], 160),
    (torch.bfloat16, 128, 1, 8, [300], 200),
    (torch.bfloat16, 128, 1, 32, [4001], 160),         # one block of rows: one workgroup a chunk
    (torch.bfloat16, 64, 2, 16, [530, 1100], 160)])    # a short last chunk, its later pieces without a key
def test_small_calls_give_the_same_scores(dt, d, group, w, lens, layers):
    print("case", dt, d, group, w, lens, flush=True)
    hkv, T = 2, sum(lens)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q = torch.randn(layers, group * hkv, len(lens) * w, d, generator=gen, device="cuda").to(dt)
    k = torch.randn(layers, hkv, T, d, generator=gen, device="cuda").to(dt)
    cu = [sum(lens[:i]) for i in range(len(lens) + 1)]

    def score(n):
        cfg = lukv.Config.for_tensors(q[:n], k[:n], w, cu, 7, 4)
        out = torch.full((n, hkv, T), float("nan"), device="cuda")
        lukv.lukv_score(cfg, q[:n], k[:n], out, lukv.alloc_workspace(lukv.lukv_workspace_bytes(cfg, 0)))
        torch.cuda.synchronize()
        return out

    whole = score(layers)
    assert not whole.isnan().any()
    for n in (1, 3):
        assert torch.equal(score(n).view(torch.int32), whole[:n].view(torch.int32)), n


@pytest.mark.parametrize("dt,d,group,w,lens", [
    (torch.bfloat16, 128, 4, 32, [513]), (torch.bfloat16, 128, 4, 32, [2500]), (torch.bfloat16, 64, 1, 16, [530, 1100]),
    (torch.bfloat16, 64, 7, 64, [1500]), (torch.float32, 128, 3, 32, [640]), (torch.float32, 64, 2, 16, [3000])])
@pytest.mark.parametrize("with_lse", [False, True])
def test_small_calls_select_by_their_scores(dt, d, group, w, lens, with_lse):
    """The value range that the accumulation kernel leaves for the selection, cut into pieces or not: the
    fused call keeps what the selection keeps on the scores it returns."""
    print("case", dt, d, group, w, lens, with_lse, flush=True)
    hkv, T, ns = 2, sum(lens), len(lens)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    q = torch.randn(1, group * hkv, ns * w, d, generator=gen, device="cuda").to(dt)
    k, v = (torch.randn(1, hkv, T, d, generator=gen, device="cuda").to(dt) for _ in range(2))
    lse = torch.rand(1, group * hkv, ns * w, generator=gen, device="cuda") * 4 + 6 if with_lse else None
    cfg = lukv.Config.for_tensors(q, k, w, [sum(lens[:i]) for i in range(ns + 1)], 7, 4)
    budgets = torch.tensor([max(w + 5, n // 5) for n in lens for _ in range(hkv)], dtype=torch.int32, device="cuda")
    offsets = torch.cat([torch.zeros(1, device="cuda", dtype=torch.int64), budgets.cumsum(0)])
    rows = int(offsets[-1])
    ws = lukv.alloc_workspace(lukv.lukv_workspace_bytes(cfg, 0))
    ws.fill_(255)

    def outputs():
        return (torch.full((rows,), -1, dtype=torch.int32, device="cuda"), torch.zeros(rows, d, dtype=dt, device="cuda"),
                torch.zeros(rows, d, dtype=dt, device="cuda"), torch.full((1,), -1, dtype=torch.int32, device="cuda"))

    pooled = torch.full((1, hkv, T), float("nan"), device="cuda")
    a, b = outputs(), outputs()
    lukv.lukv_evict_budgets(cfg, q, k, v, lse, budgets, offsets, rows, a[0], a[1], a[2], pooled, a[3], ws)
    scores = torch.full((1, hkv, T), float("nan"), device="cuda")
    if with_lse:
        lukv.lukv_score_lse(cfg, q, k, lse, scores, ws)
    else:
        lukv.lukv_score(cfg, q, k, scores, ws)
    assert torch.equal(pooled.view(torch.int32), scores.view(torch.int32))
    lukv.lukv_select_compact(cfg, scores, budgets, offsets, k, v, rows, b[0], b[1], b[2], b[3], ws)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    # and it is the highest scores that are kept (the lowest position of equal ones)
    for hi in range(ns * hkv):
        s, h = divmod(hi, hkv)
        row = scores[0, h, sum(lens[:s]):sum(lens[:s + 1])]
        best = torch.sort(row, descending=True, stable=True).indices[:int(budgets[hi])].sort().values
        assert torch.equal(a[0][offsets[hi]:offsets[hi + 1]].long(), best), hi
