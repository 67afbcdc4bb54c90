"""Rows with a few logits far from the others: the range that the selection's bins are laid over is then wide
against the spread of the row, and most logits share a few bins."""
import pytest
import torch

from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LIST_CAP, MAX_TILES, SLACK = 6144, 256, 8     # kRowListCap, kRowMaxTiles, kTileSlack of the library


@pytest.mark.parametrize("rows,n,top_k", [
    (40, 8192, 2000),      # whole row in registers
    (40, 16383, 100),
    (300, 3001, 1000),     # more rows than compute units
    (40, 65536, 2000),     # slices and candidate lists
    (10, 70001, 3000),
])
def test_threshold_of_rows_with_far_logits(rows, n, top_k):
    g = torch.Generator(device=DEV).manual_seed(n)
    z = 2.0 * torch.randn(rows, n, device=DEV, generator=g)
    # from a handful to all of the row in the bin of the threshold
    far = torch.logspace(0.5, 6, rows, device=DEV)
    z[:, 5], z[:, 9] = -far, far
    z[::3, 9] = 0.0                                 # one-sided as well
    sc = B.Scd(B.make_config(B=1, L=256, N=2000, V=n, top_k=top_k), DEV)
    thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
    nk = torch.empty(rows, dtype=torch.int32, device=DEV)
    sc.select(z, rows, thr, lse, nk)
    want = torch.topk(z, top_k, dim=1).values[:, -1]
    assert torch.equal(thr, want)
    assert torch.equal(nk.long(), (z >= want[:, None]).sum(1))
    zd = z.double()
    ref = torch.logsumexp(torch.where(zd >= want[:, None], zd, -torch.inf), 1)
    assert bool(((lse - ref).abs() <= 1e-6 * ref.abs().clamp(min=1.0)).all())     # 32-bit sum, as in the stage tests


def _counts(sc, rows, tiles):
    """Pairs emitted per (window row, tile): behind six per-row arrays and the pairs in the workspace."""
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    off = 6 * up(4 * rows) + rows * LIST_CAP * 8
    return sc.workspace[off:off + 4 * rows * tiles].view(torch.int32).view(rows, tiles)


@pytest.mark.parametrize("n,d,top_k,cols,far", [
    (65536, 128, 2000, 256, [100.0]),            # one far logit per tile, above or below the others
    (65500, 64, 2000, 256, [1e4, 30.0]),         # two, at different distances; a ragged last tile
    (32768, 128, 2000, 128, [1e30]),
    (17000, 200, 500, 128, [3e3, -3e3]),
])
def test_lists_are_full_on_rows_with_far_logits(n, d, top_k, cols, far):
    L, lam = 32, 3.0
    g = torch.Generator(device=DEV).manual_seed(n)
    W = 0.05 * torch.randn(n, d, device=DEV, generator=g)
    for i, f in enumerate(far):
        W[17 + 40 * i::cols] *= f
    W = W.to(torch.bfloat16)
    h = torch.randn(1, 2, L, d, device=DEV, generator=g).to(torch.bfloat16)
    sc = B.Scd(B.make_config(B=1, L=L, N=300, V=n, d=d, top_k=top_k, cfg_lambda=lam, seed=3), DEV)
    tiles = (n + cols - 1) // cols
    assert f", {cols}, " in sc.lm_head_kernel_name() and tiles <= MAX_TILES
    cap = LIST_CAP // tiles
    assert 2 * top_k <= tiles * (cap - SLACK)
    st = sc.alloc_state()
    sc.reset(st)
    sc.step(h, W, st)
    cnt = _counts(sc, L, tiles)
    have = torch.full((tiles,), cols, device=DEV)
    have[-1] = n - (tiles - 1) * cols
    assert bool((cnt <= cap).all()) and bool((cnt >= torch.clamp(have, max=cap - SLACK)).all()), (int(cnt.min()), int(cnt.max()))
    f = lambda field, *shape: sc.state_field(st, field).view(*shape)  # noqa: E731
    z = f(B.F_Z, 2, L, n)[0]
    thr = torch.topk(z, top_k, dim=1).values[:, -1]
    assert torch.equal(f(B.F_THR, 2, L)[0], thr)
    assert torch.equal(f(B.F_NKEPT, 2, L)[0].long(), (z >= thr[:, None]).sum(1))
