"""Decode attention where the cut of the packed rows into equal shares can go wrong: heads without
rows, of one row and around the tile and block sizes, more heads than one probe round finds, groups
around the query heads held in registers, rows that do not start at the cache's beginning; shares of many
blocks and several heads, with a maximum that moves along the rows; caches large enough to be streamed;
offsets that fall."""
import math

import numpy as np
import pytest
import torch

from paper_2602_08585_amd import lukv

pytestmark = pytest.mark.gpu

ROWS = [0, 1, 15, 16, 17, 31, 33, 63, 64, 65, 0, 0, 127, 128, 129, 255, 257, 1000]
FORMS = [("bf16", 128, 1), ("bf16", 128, 4), ("bf16", 128, 5), ("bf16", 64, 4), ("bf16", 64, 16), ("f32", 128, 3),
         ("f32", 128, 8), ("f32", 64, 4), ("f32", 64, 9)]
SHAPES = [(1, 1, 1, 0), (1, 9, 2, 37), (7, 3, 3, 5), (8, 8, 1, 0), (5, 13, 1, 63)]
MANY = (41, 5, 20, 1)
# one of every compiled form: storage type, head dimension, up to four or up to eight queries at a time
ALL_FORMS = [("bf16", 128, 2), ("bf16", 128, 5), ("bf16", 64, 4), ("bf16", 64, 7), ("f32", 128, 3), ("f32", 128, 8),
             ("f32", 64, 4), ("f32", 64, 6)]


def _decode(dtype, d, group, layers, hkv, seqs, off, L, ramp=0.0):
    """The call on random rows (logits of standard deviation 1.5, plus a ramp along every head's rows of
    up to `ramp`), every head compared with the same in 64 bits."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(off) + d + group)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    total, hq = int(max(off)) + 1, hkv * group
    k = torch.randn(total, d, generator=gen, device="cuda") / math.sqrt(d)
    q = torch.randn(layers, hq, seqs, d, generator=gen, device="cuda") * 1.5 * math.sqrt(d)
    if ramp:
        q[..., 0] = math.sqrt(d)
        for a, b in zip(off[:-1], off[1:]):
            if b > a:
                k[a:b, 0] = torch.linspace(0.0, ramp, int(b - a), device="cuda")
    k, q = k.to(dt), q.to(dt)
    v = torch.randn(total, d, generator=gen, device="cuda").to(dt)
    cfg = lukv.Config(layers, hq, hkv, d, 8, 7, 0, lukv.LUKV_BF16 if dtype == "bf16" else lukv.LUKV_F32,
                      [L * i for i in range(seqs + 1)], hkv * L * seqs * d, L * seqs * d, d, hq * seqs * 8 * d,
                      seqs * 8 * d, d)
    out = torch.full((layers, hq, seqs, d), float("nan"), device="cuda")
    ws = lukv.alloc_workspace(lukv.lukv_decode_workspace_bytes(cfg))
    ws.fill_(255)                       # (not initialised, as far as the call may know)
    lukv.lukv_decode_attention(cfg, q, k, v, torch.from_numpy(np.asarray(off, dtype=np.int64)).cuda(), out, ws)
    # A logit is a 32-bit sum: off by a few units in the last place of the largest, which moves a
    # probability by as much in absolute terms; the weighted sum adds its own units.
    eps = 2.0 ** -24
    dev = torch.device("cuda" if total > 20000 else "cpu")
    got, qd = out.double().to(dev), q.double().to(dev)
    kd, vd = (k.to(dev), v.to(dev)) if total > 20000 else (k.double().cpu(), v.double().cpu())
    for i in range(len(off) - 1):
        h, l, s = i % hkv, i // hkv % layers, i // (hkv * layers)
        a, b = int(off[i]), int(off[i + 1])
        g = got[l, h * group:(h + 1) * group, s]
        if b <= a:
            assert (g == 0).all(), i
            continue
        vv = vd[a:b].double()
        x = qd[l, h * group:(h + 1) * group, s] @ kd[a:b].double().t().contiguous() / math.sqrt(d)
        want = torch.softmax(x, dim=1) @ vv
        bound = 16 * eps * (float(x.abs().max()) * 1.4427 + 8) * float(vv.abs().max())
        assert float((g - want).abs().max()) <= bound, (i, b - a)


@pytest.mark.parametrize("dtype,d,group,layers,hkv,seqs,start",
                         [f + s for s in SHAPES for f in FORMS] + [f + MANY for f in FORMS if f[2] in (4, 5)])
def test_decode_shares(dtype, d, group, layers, hkv, seqs, start):
    n = layers * hkv * seqs
    print("case", dtype, d, group, layers, hkv, seqs, start, flush=True)
    rng = np.random.RandomState(n + d + group)
    rows = np.array([ROWS[i % len(ROWS)] for i in range(n)]) if n < 1000 else rng.randint(0, 40, n)
    if n == 1:
        rows[0] = 130
    _decode(dtype, d, group, layers, hkv, seqs, start + np.concatenate([[0], np.cumsum(rows)]), 1100)


@pytest.mark.parametrize("dtype,d,group", ALL_FORMS)
@pytest.mark.parametrize("hkv,L,rows", [
    (1, 9, [9]), (3, 70, [70, 1, 65]),            # fewer blocks than workgroups a full chip takes
    # shares of several blocks, of one head and across heads; more partial results of a head than one pass
    # of the merge takes; ends off every tile
    (5, 190000, [190000 - 1, 0, 17, 100003, 45]), (3, 400000, [13, 399999, 131]),
    (70, 7000, [(137 * i * i) % 7000 for i in range(70)])])
@pytest.mark.parametrize("ramp", [0.0, 24.0])
def test_decode_long_shares(dtype, d, group, hkv, L, rows, ramp):
    print("case", dtype, d, group, hkv, L, ramp, flush=True)
    _decode(dtype, d, group, 1, hkv, 1, 3 + np.concatenate([[0], np.cumsum(rows)]), L, ramp)


@pytest.mark.parametrize("dtype,d,group", ALL_FORMS)
def test_decode_streamed(dtype, d, group):
    """256 MiB of K and V and more are read with non-temporal loads (groups of up to eight)."""
    print("case", dtype, d, group, flush=True)
    need = (256 << 20) // (2 * d * (4 if dtype == "f32" else 2))
    share = np.array([0.31, 0.0, 0.0007, 0.22, 0.12, 0.3493])
    rows = (share * need).astype(np.int64) + np.array([1, 0, 3, 77, 5, 64])
    _decode(dtype, d, group, 2, 3, 1, np.concatenate([[0], np.cumsum(rows)]), int(rows.max()), 12.0)


@pytest.mark.parametrize("dtype,d,group", ALL_FORMS)
@pytest.mark.parametrize("hkv,off", [(5, [200, 333, 20, 21, 700, 0]), (3, [5000, 4000, 4130, 9]),
                                     (91, [(1000 - 7 * i if i % 3 else 900 + i) for i in range(92)])])
def test_decode_offsets_that_fall(dtype, d, group, hkv, off):
    """Offsets are a prefix sum; where they fall nonetheless, a head without rows is zero and the call keeps
    to its buffers (what a head with rows gets is not said)."""
    print("case", dtype, d, group, hkv, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + group)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    k, v = (torch.randn(max(off), d, generator=gen, device="cuda").to(dt) for _ in range(2))
    q = torch.randn(1, hkv * group, 1, d, generator=gen, device="cuda").to(dt)
    cfg = lukv.Config(1, hkv * group, hkv, d, 8, 7, 0, lukv.LUKV_BF16 if dtype == "bf16" else lukv.LUKV_F32, [0, 1100],
                      hkv * 1100 * d, 1100 * d, d, hkv * group * 8 * d, 8 * d, d)
    need = lukv.lukv_decode_workspace_bytes(cfg)
    ws = torch.full((need + 8192,), 0x5A, dtype=torch.uint8, device="cuda")
    out = torch.full((hkv * group + 2, d), 7.0, device="cuda")
    lukv.lukv_decode_attention(cfg, q, k, v, torch.tensor(off, dtype=torch.int64, device="cuda"), out[1:-1], ws[4096:4096 + need])
    assert (ws[:4096] == 0x5A).all() and (ws[4096 + need:] == 0x5A).all()
    assert (out[0] == 7.0).all() and (out[-1] == 7.0).all()
    for hi in range(hkv):
        if off[hi + 1] <= off[hi]:
            assert (out[1 + hi * group:1 + (hi + 1) * group] == 0).all(), hi
