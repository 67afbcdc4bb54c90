"""step_logits keeps the supplied logits for the next iteration: the ring slots of the window hold exactly
them afterwards, whichever kernel made the copy, and nothing else of the ring changes."""
import pytest
import torch

from paper_2510_24211_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Bn,L,N,n,top_k,top_p,offset", [
    (2, 5, 40, 1, 0, 0.0, 0),            # one id
    (2, 5, 40, 1027, 100, 0.0, 1),       # row kernel, 8 logits per thread; odd rows at an odd address
    (9, 32, 400, 1023, 50, 0.0, 0),      # more rows than compute units
    (1, 7, 40, 16383, 0, 0.0, 3),        # 16 logits per thread
    (2, 5, 12, 16385, 300, 0.0, 0),      # list kernel; the window is clipped at the end
    (1, 6, 40, 65536, 2000, 0.0, 1),
    (1, 6, 40, 30003, 0, 0.8, 0),        # whole row, in registers until the threshold is known
    (1, 6, 40, 30003, 4000, 0.0, 2),
    (1, 4, 40, 65537, 500, 0.0, 0),      # longer rows: with lists and without
    (1, 4, 40, 70002, 0, 0.0, 1),
    (2, 3, 40, 98305, 2000, 0.0, 0),     # pieces of 2048 ids
    (1, 4, 40, 131071, 2000, 0.0, 1),
    (1, 4, 40, 65535, 3072, 0.0, 3),     # slice kernel
])
def test_ring_holds_the_supplied_logits(Bn, L, N, n, top_k, top_p, offset):
    sc = B.Scd(B.make_config(B=Bn, L=L, N=N, V=n, top_k=top_k, top_p=top_p, seed=n), DEV)
    st = sc.alloc_state()
    sc.reset(st)
    ring = sc.state_field(st, B.F_Z).view(2, Bn, L, n)
    ring.fill_(-7.0)
    pos_v = sc.state_field(st, B.F_POS)
    g = torch.Generator(device=DEV).manual_seed(n + L)
    want = ring.clone()
    for it in range(4):
        buf = torch.randn(Bn * L * n + offset, device=DEV, generator=g)
        z = buf[offset:].view(Bn, L, n)
        pos = pos_v.tolist()
        sc.step_logits(z, st)
        for b in range(Bn):
            for s in range(min(L, N - pos[b])):
                want[it & 1, b, (pos[b] + s) % L] = z[b, s]
        assert torch.equal(ring, want), it
