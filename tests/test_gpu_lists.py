"""Candidate lists of supplied logits: every decision on rows of all kinds must equal the one on the row read whole (the
entry point without lists takes that path for them), bit for bit; and the selection must equal the oracle's."""
import numpy as np
import pytest
import torch

from oracle import logits as lg
from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KINDS = ("normal", "flat", "far", "masked", "mask_1e10", "lopsided", "sorted", "tied", "constant")


def _rows(kind, rows, n, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    z = 2.0 * torch.randn(rows, n, device=DEV, generator=g)
    if kind == "flat":
        z = 300000.0 + z                       # a few thousand values in all
    elif kind == "far":
        z[:, n // 3] = 1.0e6
        z[:, n // 2] = -1.0e20
    elif kind in ("masked", "mask_1e10"):      # most ids, and the whole of the last piece
        mask = torch.rand(rows, n, device=DEV, generator=g) < 0.7
        mask[:, -1500:] = True
        z[mask] = float("-inf") if kind == "masked" else -1.0e10
    elif kind == "lopsided":
        z = -torch.exp(z)
    elif kind == "sorted":
        z = torch.sort(z, dim=1).values
    elif kind == "tied":
        z = torch.round(z)
    elif kind == "constant":
        z[:] = 1.25
    return z.contiguous()


@pytest.mark.parametrize("n,top_k", [
    (16385, 1500),       # the last piece holds one id
    (16385, 3072),
    (17411, 20),         # three ids of a last group
    (65536, 2000),
    (65535, 3072),       # pieces of 2048
    (131071, 2000),      # pieces of 2048, rows of more than 65536 ids
    (131072, 300),
])
def test_selection_on_rows_of_all_kinds(n, top_k):
    rows = len(KINDS)
    z = torch.cat([_rows(kind, 1, n, n + i) for i, kind in enumerate(KINDS)])
    sc = B.Scd(B.make_config(B=1, L=rows, N=400, V=n, top_k=top_k, seed=3), DEV)
    thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
    nk = torch.empty(rows, dtype=torch.int32, device=DEV)
    sc.workspace.fill_(0xEE)                   # slots that nobody writes must not be read as pairs
    sc.select(z, rows, thr, lse, nk)
    for i, kind in enumerate(KINDS):
        row = z[i].cpu().numpy()
        _, want, want_lse = lg.distribution(row, top_k)
        assert thr[i].item() == want, kind
        assert nk[i].item() == int((row >= want).sum()), kind
        assert abs(lse[i].item() - want_lse) <= 1e-6 * max(1.0, abs(want_lse)), kind   # fp32 sum, as in the stage tests


@pytest.mark.parametrize("n,top_k,kind", [(65536, 2000, "normal"), (30001, 1500, "lopsided"), (131071, 2000, "masked"),
                                          (65537, 2500, "far"), (20483, 100, "mask_1e10")])
def test_lists_do_not_depend_on_the_alignment_and_are_repeatable(n, top_k, kind):
    rows = 5
    buf = torch.empty(rows * n + 1, device=DEV)
    buf[1:] = _rows(kind, rows, n, 11).view(-1)
    sc = B.Scd(B.make_config(B=1, L=rows, N=400, V=n, top_k=top_k, seed=3), DEV)
    got = []
    for z in (buf[1:], buf[1:].clone(), buf[1:]):
        x, fresh = torch.zeros(1, rows, dtype=torch.int32, device=DEV), torch.ones(1, rows, dtype=torch.uint8, device=DEV)
        y, k = torch.empty(1, rows, dtype=torch.int32, device=DEV), torch.empty(1, rows, dtype=torch.uint8, device=DEV)
        thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
        nk = torch.empty(rows, dtype=torch.int32, device=DEV)
        sc.select(z, rows, thr, lse, nk)
        sc.couple_draft(z, z, x, fresh, torch.zeros(1, dtype=torch.int32, device=DEV), 4, y, k)
        got.append([t.cpu().numpy() for t in (thr, lse, nk, y, k)])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)


def _certified(sc, rows, n, top_k, thr):
    """Whether each row's lists were enough: none overflowed, and its threshold is not below their largest cut."""
    for per in (1024, 2048):                   # ids per list, as the launcher picks them
        lists = -(-n // per)
        if lists <= 256 and top_k / lists + 5 * (top_k / lists) ** 0.5 + 4 <= 0.75 * (6144 // lists):
            break
    behind = 6 * ((4 * rows + 255) // 256 * 256) + rows * 6144 * 8
    block = (rows * 256 * 4 + 255) // 256 * 256
    words = lambda at: sc.workspace[at:at + 4 * rows * lists].view(torch.int32).view(rows, lists).cpu().numpy()  # noqa: E731
    counts, cuts = words(behind), words(behind + block).view(np.uint32)
    bits = thr.cpu().numpy().view(np.uint32)
    key = np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31))
    return (counts <= 6144 // lists).all(1) & (counts.sum(1) >= top_k) & (key >= cuts.max(1))


@pytest.mark.parametrize("n,top_k", [(65536, 2000), (81146, 2000), (30001, 1500), (16385, 1000), (131071, 1000)])
def test_neighbours_that_are_likely_together_do_not_overflow_a_list(n, top_k):
    """Ids whose logits rise and fall together in runs, fall with the id, or are masked over a range: the lists still hold
    every row's top-k, so that no row is read whole."""
    g = torch.Generator(device=DEV).manual_seed(n)
    z = 2.0 * torch.randn(6, n, device=DEV, generator=g)
    ids = torch.arange(n, device=DEV)
    for row, width in ((0, 1024), (1, 200)):
        z[row] += 0.75 * torch.randn(-(-n // width), device=DEV, generator=g).repeat_interleave(width)[:n]
    z[2] -= 0.5 * torch.log1p(ids.float())
    z[3, n // 3:] = float("-inf")
    z[4, :n // 2] = -1.0e10
    rows = len(z)
    sc = B.Scd(B.make_config(B=1, L=rows, N=400, V=n, top_k=top_k, seed=3), DEV)
    thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
    nk = torch.empty(rows, dtype=torch.int32, device=DEV)
    sc.select(z, rows, thr, lse, nk)
    assert torch.equal(thr, torch.topk(z, top_k, dim=1).values[:, -1])
    assert _certified(sc, rows, n, top_k, thr).all()
