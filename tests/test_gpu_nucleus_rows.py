"""Rows of more than 16384 ids under a nucleus filter alone, which stay in registers: against the same rows under a
top-k that drops one weightless id, which take the general path, and against the oracle."""
import numpy as np
import pytest
import torch

from oracle import logits as lg
from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# the shortest row; whole groups of 4096 ids and one id more; the edges of 32 and 64 logits per thread; odd lengths;
# the longest.  Spread 3: hundreds to thousands of ids kept; 0.3: more than are parked in LDS; with shared-noise
# redrafts, independent ones and the statistics
@pytest.mark.parametrize("n,spread,top_p,extra", [
    (16385, 3.0, 0.8, {}),
    (20480, 3.0, 0.9, dict(diagnostics=1)),
    (20481, 0.3, 0.97, dict(coupling=B.COUPLING_GS)),
    (32768, 3.0, 0.8, dict(sjd_mix=0.5)),
    (32769, 3.0, 0.8, dict(coupling=B.COUPLING_GS)),
    (45003, 0.3, 0.6, dict(diagnostics=1)),
    (45003, 20.0, 0.9, {}),
    (65535, 3.0, 0.95, {}),
    (65536, 0.3, 0.9, {}),
])
def test_rows_in_registers_decide_like_the_general_path(n, spread, top_p, extra):
    L, steps = 16, 3
    g = torch.Generator(device=DEV).manual_seed(n)
    base = spread * torch.randn(1, 1, n, device=DEV, generator=g)
    xs = [base + 0.3 * spread * torch.randn(1, L, n, device=DEV, generator=g) for _ in range(steps)]
    for x in xs:
        x[..., 7] = x[..., 11] = x.amax(2)                   # equal logits at the top
        x[..., n - 2] = -1.0e4                               # no mass: exp underflows
    got = []
    for top_k in (0, n - 1):
        sc = B.Scd(B.make_config(B=1, L=L, N=200, V=n, top_k=top_k, top_p=top_p, seed=5, **extra), DEV)
        st = sc.alloc_state()
        sc.reset(st)
        f = lambda field, *shape: sc.state_field(st, field).view(*shape).clone()  # noqa: E731
        run = []
        for it, x in enumerate(xs):
            sc.step_logits(x, st)
            thr, lse, nkept = (f(i, 2, L)[it & 1] for i in (B.F_THR, B.F_LSE, B.F_NKEPT))
            run.append(dict(thr=thr, lse=lse, nkept=nkept, y=f(B.F_Y, L), k=f(B.F_K, L),
                            px=f(B.F_PX, L), x=f(B.F_X, L), pos=f(B.F_POS, 1)))
            if extra.get("diagnostics"):
                run[-1]["stats"] = f(B.F_DIAG, L, 4)
        got.append(run)
        z = f(B.F_Z, 2, L, n)
        assert torch.equal(z[(steps - 1) & 1].sort(0).values, xs[-1][0].sort(0).values)   # the ring's copy, by slot
    rows = agree = 0
    for a, b in zip(*got):
        assert torch.equal(a["thr"], b["thr"]) and torch.equal(a["nkept"], b["nkept"])
        # 32-bit sums of up to 65536 terms in another order, in the logarithm: a few units of the last place
        assert bool(((a["lse"] - b["lse"]).abs() <= 1e-6 * b["lse"].abs().clamp(min=1.0)).all())
        rows += L
        agree += int(((a["y"] == b["y"]) & (a["k"] == b["k"])).sum())
        if not all(torch.equal(a[i], b[i]) for i in ("y", "k", "x", "pos")):
            break                                            # a near-tie: what follows starts from other drafts
        assert bool(((a["px"] - b["px"]).abs() <= 4e-6 * (b["px"].abs() + 1e-30) * b["lse"].abs().max().clamp(min=1.0)).all())
        if "stats" in a:
            assert bool(((a["stats"] - b["stats"]).abs() <= 1e-4 * b["stats"].abs()).all())
    # a score or an accept test moves by 1e-6 of itself: of 48 decisions over thousands of ids hardly one is that close
    assert agree >= rows - 1


def _select(z, top_k, top_p):
    rows, n = z.shape
    sc = B.Scd(B.make_config(B=1, L=1, N=1, V=n, top_k=top_k, top_p=top_p), DEV)
    thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
    nkept = torch.empty(rows, dtype=torch.int32, device=DEV)
    sc.select(torch.from_numpy(z).to(DEV), rows, thr, lse, nkept)
    return thr.cpu().numpy(), lse.cpu().numpy(), nkept.cpu().numpy()


# rows that span a few hundred to a few thousand units in the last place: a bin of the search holds one value, or none
@pytest.mark.parametrize("n,offset,spread,top_p", [
    (16385, 3e5, 3.0, 0.8),
    (20480, 3e5, 3.0, 0.8),
    (20481, -3e5, 3.0, 0.8),
    (32768, 1e5, 3.0, 0.5),
    (32769, 3e5, 3.0, 0.8),
    (20000, 100.0, 0.001, 0.02),
    (64000, 5e5, 3.0, 0.8),
    (65536, 3e6, 3.0, 0.9),
])
def test_rows_in_registers_against_the_oracle_where_bins_are_narrow(n, offset, spread, top_p):
    rng = np.random.default_rng(n)
    z = (offset + spread * rng.standard_normal((64, n))).astype(np.float32)
    thr, lse, nkept = _select(z, 0, top_p)
    adopted = 0
    for r in range(len(z)):
        want = lg.nucleus_threshold(z[r], slice(None), top_p)
        if thr[r] != want:          # a comparison of sums: within 2e-6 of the target mass either side is right
            inner, outer = (lg.nucleus_threshold(z[r], slice(None), top_p + d) for d in (-2e-6, 2e-6))
            assert outer <= thr[r] <= inner and (z[r] == thr[r]).any(), (r, thr[r], want)
            adopted += 1
        _, ref = lg.softmax_kept(z[r], thr[r])
        m = float(z[r].max())
        assert nkept[r] == (z[r] >= thr[r]).sum()
        # the sum's logarithm as in the stage tests, and the rounding of its addition to the maximum
        assert abs(lse[r] - ref) <= 1e-6 * max(1.0, abs(ref - m)) + 2.0 ** -23 * abs(ref), (r, lse[r], ref)
    assert adopted <= 2


# Masked ids weigh nothing, whatever finite or infinite value masks them.  Rows 0 and 1: two ids, the second one's mass w
# in units of 2^-40 100 above and below what top_p = 1 - 2^-20 asks for (2^40 * 2^24 < (2^24 - 16) (2^40 + w), that is
# w >= 1048578; w comes out within 2 units), so that a mass of one unit per masked id decides; then half of the ids
# masked, a stretch of them, all but one.
@pytest.mark.parametrize("low", [-float("inf"), float(np.finfo(np.float32).min), -1e10, -2e10, -1e30, -1e38])
@pytest.mark.parametrize("n,top_k", [
    (1000, 0),            # rows in registers: of short rows ...
    (12000, 5000),
    (16385, 0),           # ... and of long ones
    (20000, 0),
    (65536, 0),
    (65536, 2000),        # lists that are not certified: more ids tie at the mask than fit
    (40000, 5000),        # no lists
])
def test_masked_ids_weigh_nothing(n, top_k, low):
    rng = np.random.default_rng(n)
    z = (3.0 * rng.standard_normal((5, n))).astype(np.float32)
    z[:2], z[:2, 3] = low, 0.0
    z[0, n - 5], z[1, n - 5] = np.log(np.array([1048578.0 + 100, 1048578.0 - 100]) / 2.0 ** 40)
    z[2, rng.permutation(n)[:n // 2]] = low
    z[3, n // 4:n - n // 4] = low
    z[4, :n - 1] = low
    thr, lse, nkept = _select(z, top_k, 1.0 - 2.0 ** -20)
    assert thr[0] == z[0, n - 5] and nkept[0] == 2
    assert thr[1] == 0.0 and nkept[1] == 1 and lse[1] == 0.0
    assert thr[4] == z[4, n - 1] and nkept[4] == 1
    thr, lse, nkept = _select(z, top_k, 0.8)
    for r in range(5):
        p, want, ref = lg.distribution(z[r], top_k, 0.8)
        assert thr[r] == want and nkept[r] == (z[r] >= want).sum(), (r, thr[r], want)
        assert abs(lse[r] - ref) <= 1e-6 * max(1.0, abs(ref))
