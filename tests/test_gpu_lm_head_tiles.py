"""LM-head kernels over the shapes where their choice, their tiles or their tails change: logits against
64 bits, and the candidate lists of the epilogue against a selection over the stored logits."""
import numpy as np
import pytest
import torch

from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(Bn, C, L, n, d, v_lo, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    W = (0.05 * torch.randn(v_lo + n + 3, d, device=DEV, generator=g)).to(torch.bfloat16)
    h = torch.randn(Bn, C, L, d, device=DEV, generator=g).to(torch.bfloat16)
    return W, h


def _want(W, h, n, v_lo, lam, tau):
    w = W[v_lo:v_lo + n].double()
    a = torch.stack([h[:, c].double().reshape(-1, h.shape[3]) @ w.t() for c in range(h.shape[1])])
    z = a[0] if len(a) == 1 else (1 + lam) * a[0] - lam * a[1]
    # every raw logit is a sum of d products: the worst order of 32-bit additions errs by less than
    # d * 2^-24 * sum |h w|, a realistic one by sqrt(d) of that; sum |h w| <= |h| |w|
    size = torch.stack([h[:, c].double().norm(dim=2).reshape(-1) for c in range(h.shape[1])]).max(0).values
    bound = 4 * np.sqrt(h.shape[3]) * 2.0 ** -24 * size[:, None] * w.norm(dim=1)[None] * (1 + 2 * lam) / tau
    return (z / tau).reshape(h.shape[0], h.shape[2], n), bound.reshape(h.shape[0], h.shape[2], n)


# every kernel and tile, at its edges in rows, ids and k
SHAPES = [
    # Bn, L, n, d, lam, kernel
    (1, 1, 1, 64, 0.0, "tile_kernel<1, 64, 128, 6, false>"),          # one row, one id, one k-tile
    (2, 40, 300, 56, 0.0, "kernel<1, 1, 4, false>"),                  # no whole k-tile
    (1, 5, 70, 8, 3.0, "kernel<1, 2, 4, false>"),
    (3, 7, 129, 72, 3.0, "tile_kernel<2, 64, 128, 6, false>"),        # a ragged k-tile of one chunk, rows of three sequences packed
    (2, 16, 1000, 120, 0.0, "tile_kernel<1, 64, 128, 6, false>"),     # one whole k-tile and 7 chunks
    (2, 17, 8300, 200, 3.0, "tile_kernel<2, 64, 128, 6, false>"),     # 34 rows: two blocks, three whole k-tiles
    (1, 32, 8193, 512, 3.0, "tile_kernel<2, 64, 128, 6, false>"),     # one workgroup more than the split kernel takes
    (300, 1, 3000, 640, 0.0, "tile_kernel<1, 64, 128, 6, false>"),    # many sequences of one position
    (5, 6, 16384, 520, 0.0, "splitk_kernel<1, 1, 8>"),                # packed rows
    (1, 33, 8192, 576, 0.0, "splitk_kernel<2, 1, 4>"),
    (1, 20, 32769, 328, 3.0, "tile_kernel<2, 64, 256, 4, false>"),    # last tile a single column
    (3, 20, 51210, 136, 0.0, "tile_kernel<1, 64, 256, 4, false>"),
    (2, 33, 33000, 4104, 3.0, "tile_kernel<2, 64, 256, 4, true>"),    # W past the caches, rows over two sequences
    (1, 31, 33000, 256, 0.0, "kernel<1, 1, 8, false>"),
    (1, 20, 65000, 1608, 0.0, "kernel<1, 1, 8, true>"),
    (2, 17, 32700, 392, 3.0, "tile_kernel<2, 128, 128, 5, false>"),   # six whole k-tiles and one chunk
    (1, 100, 24000, 392, 0.0, "tile_kernel<1, 128, 128, 5, false>"),
    (1, 128, 25001, 4168, 0.0, "tile_kernel<1, 128, 128, 5, true>"),
    (7, 21, 20001, 328, 3.0, "tile_kernel<2, 128, 256, 3, false>"),   # rows ragged in blocks and tiles, odd ids
    (1, 100, 44000, 264, 0.0, "tile_kernel<1, 128, 256, 3, false>"),
    (9, 29, 65535, 64, 0.0, "tile_kernel<1, 128, 256, 3, false>"),    # one k-tile
    (1, 64, 50001, 2200, 3.0, "tile_kernel<2, 128, 256, 3, true>"),
    (3, 40, 20003, 200, 3.0, "tile_kernel<2, 256, 128, 3, false>"),
    (2, 100, 20001, 328, 0.0, "tile_kernel<1, 256, 128, 3, false>"),
    (2, 128, 25000, 4160, 0.0, "tile_kernel<1, 256, 128, 3, true>"),
    (2, 33, 44000, 264, 3.0, "tile_kernel<2, 256, 256, 3, false>"),
    (3, 40, 60001, 136, 3.0, "tile_kernel<2, 256, 256, 3, false>"),   # two whole k-tiles and one chunk
    (5, 50, 65535, 72, 0.0, "tile_kernel<1, 256, 256, 3, false>"),    # one whole k-tile and one chunk
    (2, 64, 56000, 1800, 3.0, "tile_kernel<2, 256, 256, 3, true>"),
]


@pytest.mark.parametrize("Bn,L,n,d,lam,kernel", SHAPES)
def test_logits_against_64_bits(Bn, L, n, d, lam, kernel):
    C, v_lo, tau = (2 if lam else 1), 5, 0.8
    W, h = _inputs(Bn, C, L, n, d, v_lo, Bn * n + d)
    sc = B.Scd(B.make_config(B=Bn, L=L, N=300, V=W.shape[0], d=d, v_lo=v_lo, v_hi=v_lo + n, temperature=tau,
                             cfg_lambda=lam), DEV)
    assert sc.lm_head_kernel_name() == "lm_head_" + kernel
    buf = torch.full((Bn * L * n + 64,), float("nan"), device=DEV)
    sc.lm_head(h, W, buf[:Bn * L * n])
    z = buf[:Bn * L * n].view(Bn, L, n)
    want, bound = _want(W, h, n, v_lo, lam, tau)
    assert bool(((z.double() - want).abs() <= bound).all()), float(((z.double() - want).abs() / bound).max())
    assert bool(buf[Bn * L * n:].isnan().all())                        # nothing past the last row


@pytest.mark.parametrize("Bn,L,n,d,lam,top_k,kernel,lists", [
    (1, 32, 17000, 256, 3.0, 500, "tile_kernel<2, 64, 128, 6, false>", 133),
    (2, 17, 32768, 128, 3.0, 2000, "tile_kernel<2, 128, 128, 5, false>", 256),    # as many lists as a row has room for
    (3, 40, 20003, 192, 3.0, 1500, "tile_kernel<2, 256, 128, 3, false>", 157),    # rows packed over sequences, ragged ids
    (1, 32, 65536, 128, 3.0, 2000, "tile_kernel<2, 64, 256, 4, false>", 256),
    (1, 20, 50001, 200, 0.0, 900, "kernel<1, 1, 8, false>", 196),
    (1, 64, 65500, 128, 3.0, 2000, "tile_kernel<2, 128, 256, 3, false>", 256),
    (4, 33, 32768, 136, 3.0, 1000, "tile_kernel<2, 256, 256, 3, false>", 128),    # a second row tile with 4 of 128 rows
    (5, 50, 65536, 64, 0.0, 2000, "tile_kernel<1, 256, 256, 3, false>", 256),     # 250 rows in two passes
    (1, 8, 40000, 64, 3.0, 2433, "tile_kernel<2, 64, 256, 4, false>", 157),       # the largest top-k for these lists
    (1, 8, 40000, 64, 3.0, 2434, "tile_kernel<2, 64, 256, 4, false>", 40),        # one more: a list per 1024 ids
    (1, 8, 50001, 64, 3.0, 3000, "tile_kernel<2, 64, 256, 4, false>", 25),        # a list per 2048 ids
    (2, 7, 100003, 64, 3.0, 2000, "tile_kernel<2, 64, 256, 4, false>", 49),       # more tiles than a row has room for lists
])
def test_step_selects_what_a_selection_over_its_logits_does(Bn, L, n, d, lam, top_k, kernel, lists):
    C = 2 if lam else 1
    W, h = _inputs(Bn, C, L, n, d, 0, n + top_k)
    rows = Bn * L
    W[:40] = W[0].clone()                      # ids that tie in every row
    cfg = dict(B=Bn, L=L, N=L + 20, V=W.shape[0], d=d, v_lo=0, v_hi=n, top_k=top_k, cfg_lambda=lam, seed=9)
    sc = B.Scd(B.make_config(**cfg), DEV)
    assert sc.lm_head_kernel_name() == "lm_head_" + kernel
    st = sc.alloc_state()
    sc.reset(st)
    f = lambda field, *shape: sc.state_field(st, field).view(*shape)  # noqa: E731
    # the lists' lengths, behind six per-row arrays and 6144 pairs per row
    lengths = sc.workspace[6 * ((4 * rows + 255) // 256 * 256) + rows * 6144 * 8:][:4 * 256 * rows].view(torch.int32)
    lengths.fill_(-1)
    pos = torch.zeros(Bn, dtype=torch.int64)
    for it in range(3):                        # the windows of later iterations wrap around the ring and end
        live = [[b, (int(pos[b]) + s) % L] for b in range(Bn) for s in range(min(L, L + 20 - int(pos[b])))]
        sc.step(h, W, st)
        assert it > 0 or int((lengths >= 0).sum()) == rows * lists
        sel = torch.tensor(live, device=DEV)
        z = f(B.F_Z, 2, Bn, L, n)[it & 1, sel[:, 0], sel[:, 1]].contiguous()
        thr, lse = torch.empty(rows, device=DEV), torch.empty(rows, device=DEV)
        nk = torch.empty(rows, dtype=torch.int32, device=DEV)
        sc.select(z, len(live), thr, lse, nk)
        got = [f(field, 2, Bn, L)[it & 1, sel[:, 0], sel[:, 1]] for field in (B.F_THR, B.F_LSE, B.F_NKEPT)]
        assert torch.equal(got[0], thr[:len(live)]) and torch.equal(got[2], nk[:len(live)])
        assert bool(((got[1] - lse[:len(live)]).abs() <= 1e-6 * lse[:len(live)].abs().clamp(min=1.0)).all())
        pos = f(B.F_POS, Bn).cpu().long()
    assert bool((pos > 0).all())


@pytest.mark.parametrize("Bn,L,n,d,lam,parts,kernel", [
    (1, 8, 32768, 4096, 0.0, 8, "tile_kernel<1, 64, 128, 6, true>"),
    (1, 32, 8193, 3072, 3.0, 8, "tile_kernel<2, 64, 128, 6, false>"),     # 48 k-tiles, the fewest for 8 parts
    (1, 32, 49024, 4096, 0.0, 8, "tile_kernel<1, 64, 256, 4, true>"),     # the longest rows that are split
    (3, 20, 2000, 1032, 3.0, 4, "tile_kernel<2, 64, 128, 6, false>"),     # 16 k-tiles and a ragged one
    (1, 64, 40000, 1280, 0.0, 4, "tile_kernel<1, 64, 256, 4, false>"),
    (2, 32, 30001, 2048, 3.0, 4, "tile_kernel<2, 128, 128, 5, false>"),
    (3, 32, 45000, 1280, 0.0, 4, "tile_kernel<1, 128, 256, 3, false>"),
    (3, 32, 49024, 2048, 3.0, 4, "tile_kernel<2, 256, 128, 3, false>"),
])
def test_small_calls_add_up_in_parts(Bn, L, n, d, lam, parts, kernel):
    W, h = _inputs(Bn, 2 if lam else 1, L, n, d, 0, n + d)
    sc = B.Scd(B.make_config(B=Bn, L=L, N=300, V=W.shape[0], d=d, v_hi=n, cfg_lambda=lam), DEV)
    assert sc.lm_head_kernel_name() == "lm_head_" + kernel
    z = torch.empty(Bn, L, n, device=DEV)
    sc.lm_head(h, W, z)
    want, _ = _want(W, h, n, 0, lam, 1.0)
    err = float((z.double() - want).norm() / want.norm())
    # T = d / 16 accumulations per logit, each rounding a sum that has grown like a random walk: over `parts`
    # chains of T / parts and the chain that adds them up the error is u sqrt(T / (2 parts) + (parts + 1) / 2) of
    # the result, u the rms of a rounding error in units of the value, at most 2^-24 / sqrt(3) * 1.2 (one chain
    # would be u sqrt(T / 2), 1.4 times this bound and more)
    assert err <= 0.7 * 2.0 ** -24 * np.sqrt(d / 32 / parts + (parts + 1) / 2), err


@pytest.mark.parametrize("Bn,L,n,d,lam,top_k", [
    (1, 32, 32769, 128, 3.0, 2000),      # the last tile of a row is one column
    (1, 30, 20503, 128, 3.0, 1500),      # 23 columns of 128, fewer than a list holds; rows of a wavefront that do not exist
    (3, 43, 60003, 64, 3.0, 2000),       # 99 columns of 256, odd rows; a second row tile with one live row
    (5, 45, 50179, 72, 0.0, 900),        # three columns; 225 rows in two passes
    (1, 20, 50020, 200, 0.0, 900),       # the kernel with a shared h tile
])
def test_logits_stored_beside_lists_are_those_stored_without(Bn, L, n, d, lam, top_k):
    W, h = _inputs(Bn, 2 if lam else 1, L, n, d, 0, n)
    sc = B.Scd(B.make_config(B=Bn, L=L, N=L + 20, V=W.shape[0], d=d, v_hi=n, top_k=top_k, cfg_lambda=lam, seed=9), DEV)
    st = sc.alloc_state()
    sc.reset(st)
    ring = sc.state_field(st, B.F_Z).view(2, Bn, L, n)
    ring.fill_(float("nan"))
    sc.step(h, W, st)
    z = torch.empty(Bn, L, n, device=DEV)
    sc.lm_head(h, W, z)
    assert torch.equal(ring[0], z) and bool(ring[1].isnan().all())     # the same sums, and nothing past a row's end
    want = torch.topk(z.view(Bn * L, n), top_k, dim=1).values[:, -1].view(Bn, L)
    assert torch.equal(sc.state_field(st, B.F_THR).view(2, Bn, L)[0], want)
    assert torch.equal(sc.state_field(st, B.F_NKEPT).view(2, Bn, L)[0].long(), (z >= want[..., None]).sum(2))
