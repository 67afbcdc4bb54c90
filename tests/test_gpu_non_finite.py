"""Rows with NaN, infinities and masks of the type's lowest value, on every path that a row can take: a NaN or an
unusable normaliser is reported, -inf and masked ids are ordinary, and no other row notices."""
import pytest
import torch

from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
INF = float("inf")
NAN, NEG_NAN = 0x7FC00000, -0x400000                 # bit patterns: quiet NaN of either sign
ROWS = [
    # Bn, L, n, top_k, top_p
    (1, 6, 5000, 0, 0.0),          # whole row in registers
    (1, 6, 8191, 2000, 0.0),
    (2, 3, 16384, 1000, 0.9),
    (9, 32, 3001, 100, 0.0),       # more rows than compute units
    (1, 6, 30001, 1500, 0.0),      # slices and lists
    (1, 6, 65536, 2000, 0.8),
    (1, 6, 30001, 0, 0.0),         # in place
    (1, 6, 30004, 0, 0.8),         # in registers until the threshold is known
    (1, 6, 40000, 4000, 0.0),      # in place: too many for the lists
    (1, 6, 70001, 1500, 0.0),      # longer rows: lists, whole passes
    (1, 6, 70002, 0, 0.0),
    (1, 6, 66000, 5000, 0.0),
]


def _step(sc, z):
    st = sc.alloc_state()
    sc.reset(st)
    sc.step_logits(z, st)
    rc, flags = sc.status(st)
    L, Bn = sc.cfg.L, sc.cfg.B
    return rc, flags[0], [sc.state_field(st, f)[:Bn * L].clone() for f in (B.F_THR, B.F_LSE, B.F_NKEPT, B.F_Y, B.F_K)]


@pytest.mark.parametrize("Bn,L,n,top_k,top_p", ROWS)
def test_rows_with_values_that_are_not_finite(Bn, L, n, top_k, top_p):
    rows = Bn * L
    g = torch.Generator(device=DEV).manual_seed(n + top_k)
    z = 2.0 * torch.randn(rows, n, device=DEV, generator=g)
    sc = B.Scd(B.make_config(B=Bn, L=L, N=1000, V=n, top_k=top_k, top_p=top_p, seed=5), DEV)
    rc, fault, clean = _step(sc, z)
    assert rc == B.SCD_OK and fault == 0
    bad = rows - 2
    others = [r for r in range(rows) if r != bad]
    nan_at = [(0, NAN), (n // 2, NEG_NAN), (n - 1, NAN)]
    for what, ids, value in ([("nan", [i], bits) for i, bits in nan_at] +
                             [("inf", [n // 3], INF), ("both", [1, n - 2], None), ("all", slice(None), -INF)]):
        zb = z.clone()
        if what == "nan":
            zb.view(torch.int32)[bad, ids] = value
        elif what == "both":
            zb[bad, 1], zb[bad, n - 2] = INF, -INF
        else:
            zb[bad, ids] = value
        rc, fault, got = _step(sc, zb)
        assert rc == B.SCD_ENUMERIC and fault == 1, (what, ids)
        for a, b in zip(got, clean):
            assert torch.equal(a[others], b[others]), (what, ids)


@pytest.mark.parametrize("low", [-INF, torch.finfo(torch.float32).min])
@pytest.mark.parametrize("Bn,L,n,top_k,top_p", [r for r in ROWS if r[4] == 0.0])
def test_masked_ids(Bn, L, n, top_k, top_p, low):
    rows = Bn * L
    g = torch.Generator(device=DEV).manual_seed(n)
    z = 2.0 * torch.randn(rows, n, device=DEV, generator=g)
    z[0, torch.randperm(n, device=DEV, generator=g)[:n // 2]] = low     # scattered
    z[1, :n - max(n // 3, 1)] = low                                     # whole slices
    z[2, 1:] = low                                                      # a single id left: the threshold may be the mask
    sc = B.Scd(B.make_config(B=Bn, L=L, N=1000, V=n, top_k=top_k, seed=5), DEV)
    rc, fault, (thr, lse, nkept, _, _) = _step(sc, z)
    assert rc == B.SCD_OK and fault == 0
    want = torch.topk(z, top_k, dim=1).values[:, -1] if top_k else torch.full((rows,), -INF, device=DEV)
    assert torch.equal(thr, want)
    assert torch.equal(nkept.long(), (z >= want[:, None]).sum(1))
    zd = z.double()
    ref = torch.logsumexp(torch.where(zd >= want[:, None], zd, -INF), 1)
    assert bool(((lse - ref).abs() <= 1e-6 * ref.abs().clamp(min=1.0)).all())     # 32-bit sum, as in the stage tests


@pytest.mark.parametrize("L,n,d,lam,top_k,kernel", [
    (40, 50000, 128, 3.0, 1500, "tile_kernel<2, 128, 256, 3, false>"),
    (32, 17000, 128, 3.0, 500, "tile_kernel<2, 64, 128, 6, false>"),
    (20, 50001, 256, 0.0, 900, "kernel<1, 1, 8, false>"),
    (33, 65536, 128, 0.0, 2000, "tile_kernel<1, 64, 256, 4, false>"),
])
def test_lists_of_the_lm_head(L, n, d, lam, top_k, kernel):
    C = 2 if lam else 1
    g = torch.Generator(device=DEV).manual_seed(n)
    W = (0.05 * torch.randn(n, d, device=DEV, generator=g)).to(torch.bfloat16)
    h = torch.randn(1, C, L, d, device=DEV, generator=g).to(torch.bfloat16)
    h[..., 0] = 1.0
    sc = B.Scd(B.make_config(B=1, L=L, N=1000, V=n, d=d, top_k=top_k, cfg_lambda=lam, seed=5), DEV)
    assert sc.lm_head_kernel_name() == "lm_head_" + kernel

    def step(h, W):
        st = sc.alloc_state()
        sc.reset(st)
        sc.step(h, W, st)
        rc, flags = sc.status(st)
        f = [sc.state_field(st, f)[:L].clone() for f in (B.F_THR, B.F_LSE, B.F_NKEPT, B.F_Y, B.F_K)]
        return rc, flags[0], f, sc.state_field(st, B.F_Z).view(2, L, n)[0].clone()

    rc, fault, clean, _ = step(h, W)
    assert rc == B.SCD_OK and fault == 0
    others = [r for r in range(L) if r != 5]
    for value in (float("nan"), INF):                # one hidden row: its logits are NaN, or infinite of both signs
        hb = h.clone()
        hb[0, 0, 5, 3] = value
        rc, fault, got, _ = step(hb, W)
        assert rc == B.SCD_ENUMERIC and fault == 1, value
        for a, b in zip(got, clean):
            assert torch.equal(a[others], b[others]), value
    for j in (0, n // 2, n - 1):                     # one weight row: a NaN in every row of one tile
        Wb = W.clone()
        Wb[j, 7] = float("nan")
        rc, fault, _, _ = step(h, Wb)
        assert rc == B.SCD_ENUMERIC and fault == 1, j
    if C == 1:                                       # -inf in every row (guidance would make it a NaN)
        Wb = W.clone()
        Wb[n // 2] = 0.0
        Wb[n // 2, 0] = -INF
        rc, fault, (thr, lse, nkept, _, _), z = step(h, Wb)
        assert rc == B.SCD_OK and fault == 0 and bool((z[:, n // 2] == -INF).all())
        want = torch.topk(z, top_k, dim=1).values[:, -1]
        assert torch.equal(thr, want) and torch.equal(nkept.long(), (z >= want[:, None]).sum(1))


@pytest.mark.parametrize("Bn,L,n,top_k,top_p", [(2, 3, 3, 0, 0.0), (1, 6, 700, 100, 0.0), (1, 6, 3000, 0, 0.9), (9, 32, 6001, 0, 0.0)] +
                         ROWS)
def test_the_previous_logits_of_a_new_position_decide_nothing(Bn, L, n, top_k, top_p):
    g = torch.Generator(device=DEV).manual_seed(n)
    z, z_prev = (2.0 * torch.randn(Bn, L, n, device=DEV, generator=g) for _ in range(2))
    fresh = (torch.arange(L, device=DEV) % 2).to(torch.uint8).repeat(Bn, 1)
    x = (torch.arange(Bn * L, device=DEV).to(torch.int32) * 7 % n).view(Bn, L)
    pos = torch.zeros(Bn, dtype=torch.int32, device=DEV)
    sc = B.Scd(B.make_config(B=Bn, L=L, N=1000, V=n, top_k=top_k, top_p=top_p, seed=5), DEV)
    got = []
    for value in (None, float("nan"), INF, -INF):
        if value is not None:
            z_prev[fresh.bool()] = value
        y, k = torch.empty(Bn, L, dtype=torch.int32, device=DEV), torch.empty(Bn, L, dtype=torch.uint8, device=DEV)
        sc.couple_draft(z, z_prev, x, fresh, pos, 3, y, k)
        got.append((y, k))
    for y, k in got[1:]:
        assert torch.equal(y, got[0][0]) and torch.equal(k, got[0][1])
