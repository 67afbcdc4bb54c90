"""Rows of more than 65536 ids on the GPU: candidate lists where the top-k fits them, whole passes
over the row otherwise.  The two must agree to the bit in every decision."""
import numpy as np
import pytest
import torch

from oracle import logits as lg
from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(Bn, L, n, seed, kind="normal"):
    g = torch.Generator(device=DEV).manual_seed(seed)
    base = 2.0 * torch.randn(Bn, L, n, device=DEV, generator=g)
    z = base + 0.7 * torch.randn(Bn, L, n, device=DEV, generator=g)
    if kind == "ties":                       # thousands of equal logits at the threshold: the lists overflow
        base, z = (torch.round(v) for v in (base, z))
    x = base.argmax(2).to(torch.int32)
    fresh = (torch.arange(L, device=DEV) % 4 == 3).to(torch.uint8).repeat(Bn, 1)
    return z.contiguous(), base.contiguous(), x, fresh


def _draft(sc, args, pos, it, static):
    Bn, L = args[2].shape
    y = torch.full((Bn, L), -5, dtype=torch.int32, device=DEV)
    k = torch.full((Bn, L), 9, dtype=torch.uint8, device=DEV)
    (sc.couple_draft_static if static else sc.couple_draft)(*args, pos, it, y, k)
    torch.cuda.synchronize()
    return y.cpu().numpy(), k.cpu().numpy()


@pytest.mark.parametrize("n,top_k,kind", [
    (65537, 2000, "normal"),      # odd rows, the shortest that take this path
    (131072, 300, "normal"),
    (70001, 1500, "ties"),        # not certified: whole passes
    (65540, 3072, "normal"),      # the largest top-k that the lists serve
])
def test_draft_with_lists_equals_draft_without(n, top_k, kind):
    # 168 rows: more than the static array holds lists for, so that entry point reads whole rows
    Bn, L = 7, 24
    sc = B.Scd(B.make_config(B=Bn, L=L, N=400, V=n, top_k=top_k, seed=n), DEV)
    args = _rows(Bn, L, n, n + top_k, kind)
    pos = torch.tensor([0, 5, 50, 100, 200, 300, 390], dtype=torch.int32, device=DEV)   # the last one clipped
    (y0, k0), (y1, k1) = (_draft(sc, args, pos, 3, static) for static in (False, True))
    assert np.array_equal(k0, k1) and np.array_equal(y0, y1)
    assert (k0 == 0).any() and (y0[-1, 10:] == -1).all() and (k0[-1, 10:] == 1).all()


@pytest.mark.parametrize("n,top_k", [(65540, 1000), (80004, 5000), (65544, 0)])
def test_select_on_rows_that_are_not_16_byte_aligned(n, top_k):
    rows = 3
    g = torch.Generator(device=DEV).manual_seed(n)
    buf = 3.0 * torch.randn(rows * n + 1, device=DEV, generator=g)
    sc = B.Scd(B.make_config(B=1, L=rows, N=64, V=n, top_k=top_k), DEV)
    got = []
    for z in (buf[1:], buf[1:].clone()):
        thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
        nk = torch.empty(rows, dtype=torch.int32, device=DEV)
        sc.select(z, rows, thr, lse, nk)
        got.append([t.cpu().numpy() for t in (thr, lse, nk)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    z = buf[1:].view(rows, n).cpu().numpy()
    for r in range(rows):
        _, thr, lse = lg.distribution(z[r], top_k)
        assert got[0][0][r] == thr and got[0][2][r] == int((z[r] >= thr).sum())
        assert abs(float(got[0][1][r]) - lse) <= 1e-6 * max(1.0, abs(lse))   # fp32 sum, as in the stage tests
