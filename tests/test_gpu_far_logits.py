"""Rows with a few logits far from the others: the range that the selection's bins are laid over is then wide
against the spread of the row, and most logits share a few bins."""
import pytest
import torch

from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


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
