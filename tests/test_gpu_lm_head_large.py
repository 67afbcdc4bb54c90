"""LM head on operands of more than 4 GiB: the last rows of W and of h lie beyond what a 32-bit byte offset reaches."""
import pytest
import torch

from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Bn,C,L,n,d,kernel", [
    (1, 1, 8, 262144 + 301, 8192, "lm_head_kernel<1, 1, 8, true>"),       # W: few rows, a long stream
    (1, 1, 1, 38347922 + 300, 56, "lm_head_kernel<1, 1, 4, true>"),       # W: no whole k-tile
    (1, 2, 8, 262144 + 301, 8192, "lm_head_tile_kernel<2, 64, 256, 4, true>"),
    (513, 2, 256, 40, 8192, "lm_head_tile_kernel<2, 256, 128, 3, false>"),   # h: the last sequence
])
def test_logits_beyond_4_gib(Bn, C, L, n, d, kernel):
    g = torch.Generator(device=DEV).manual_seed(n)
    W = torch.empty(n, d, dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.05, generator=g)
    h = torch.empty(Bn, C, L, d, dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    assert 2 * max(W.numel(), h.numel()) > 1 << 32
    lam = 2.0 if C == 2 else 0.0
    sc = B.Scd(B.make_config(B=Bn, L=L, N=300, V=n, d=d, cfg_lambda=lam), DEV)
    assert sc.lm_head_kernel_name() == kernel
    z = torch.full((Bn, L, n), float("nan"), device=DEV)
    sc.lm_head(h, W, z)
    for b in sorted({0, Bn // 2, Bn - 1}):
        for lo, hi in ((0, min(n, 300)), (max(0, n - 300), n)):
            w = W[lo:hi].double()
            a = [h[b, c].double() @ w.t() for c in range(C)]
            want = a[0] if C == 1 else (1 + lam) * a[0] - lam * a[1]
            # as in the tests of the tiles: four times what sqrt(d) of d additions in 32 bits err by
            size = torch.stack([h[b, c].double().norm(dim=1) for c in range(C)]).max(0).values
            bound = 4 * d ** 0.5 * 2.0 ** -24 * size[:, None] * w.norm(dim=1)[None] * (1 + 2 * lam)
            assert bool(((z[b, :, lo:hi].double() - want).abs() <= bound).all()), (b, lo)
    assert not bool(z.isnan().any())
