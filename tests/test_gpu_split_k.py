"""Steps whose LM head deals k over workgroups (up to 8 parts per 64 x 128 tile), against the oracle: the row kernel adds the
parts up, processes the logits and leaves them in the ring.  Ragged ids, rows and k; every number of parts; every option."""
import numpy as np
import pytest
import torch

from lockstep import LockStep
from paper_2510_24211_amd import binding as B
from paper_2510_24211_amd import workload as wl
from test_gpu_lm_head_tiles import _inputs, _want

pytestmark = pytest.mark.gpu


def _fields_end(sc, state):
    views = [sc.state_field(state, f) for f in range(B.F_COUNT)]
    end = max(v.data_ptr() + v.numel() * v.element_size() for v in views) - state.data_ptr()
    return (end + 255) // 256 * 256


@pytest.mark.parametrize("parts,kw,opts", [
    (2, dict(B=2, L=32, V=3000, d=1280, v_lo=3, v_hi=2900), dict()),              # five k-tiles of ten in flight, odd rows
    (2, dict(B=5, L=26, V=1285, d=1288, cfg_lambda=0.0), dict()),                 # ragged k-tile, 130 rows, no guidance
    (4, dict(B=2, L=32, V=1031, d=1280), dict(coupling="gs", diagnostics=True)),
    (4, dict(B=1, L=40, V=2047, d=1304, top_p=0.9), dict()),
    (4, dict(B=1, L=64, V=4090, d=1280, cfg_lambda=0.0), dict()),                 # 8 logits per thread, four arrays
    (8, dict(B=3, L=16, V=260, d=2048, temperature=0.8), dict(sjd_mix=0.5)),      # short rows, windows below 32
    (8, dict(B=1, L=64, V=1024, d=2056, cfg_lambda=0.0), dict(diagnostics=True)),
    (8, dict(B=1, L=32, V=1900, d=4096, top_p=0.95), dict(coupling="gs")),        # up to 32 rows
    (4, dict(B=1, L=30, V=4000, d=4096), dict()),
])
def test_lockstep_with_k_in_parts(parts, kw, opts):
    kw = dict(dict(N=3 * kw["L"] + 5, age_cap=8, top_k=kw["V"] // 5), **kw)
    w = wl.scaled(wl.WORKLOADS["C2"], name="parts", **dict(dict(v_lo=0, v_hi=kw["V"]), **kw))
    ls = LockStep(w, "cuda:0", **opts)
    # the arrays of the parts, [parts, 1 + CFG, rows, n], behind the fields of the state; the workspace is left alone
    words = ls.state[_fields_end(ls.gpu, ls.state):].view(torch.int32)
    words.fill_(-1)
    ls.gpu.workspace.fill_(0xA5)
    ls.step()
    used = parts * w.C * w.B * w.L * w.n_allowed
    assert (words[:used] != -1).all() and (words[used:] == -1).all() and words.numel() - used < 64
    assert (ls.gpu.workspace == 0xA5).all()
    st = ls.run()
    assert ls.oracle.done()
    # the lock-step tests' bounds on adopted decisions; a logit itself has to lie within the measured-discrepancy cap
    assert st["adopt_accept"] + st["adopt_resid"] <= max(3, 1e-3 * st["draws"])
    assert st["adopt_topk"] <= max(3, 1e-2 * st["draws"])


def test_parts_are_run_to_run_identical():
    s = B.Scd(B.make_config(B=2, L=32, N=400, V=2048, d=2048, top_k=500, cfg_lambda=3.0, seed=5))
    g = torch.Generator(device="cuda").manual_seed(1)
    W = torch.randn(2048, 2048, device="cuda", generator=g).to(torch.bfloat16) * 0.02
    hs = [torch.randn(2, 2, 32, 2048, device="cuda", generator=g).to(torch.bfloat16) for _ in range(4)]
    got = []
    for _ in range(2):
        st = s.alloc_state().fill_(0x7f)
        s.reset(st)
        for h in hs:
            s.step(h, W, st)
        got.append([s.state_field(st, f).clone() for f in (B.F_OUT, B.F_Z, B.F_LSE, B.F_PX)])
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("parts,chains,Bn,L,n,d,lam", [
    (2, 4, 2, 32, 2897, 1280, 3.0),       # two sums per part; odd rows
    (2, 2, 5, 26, 1285, 1288, 0.0),       # a ragged k-tile
    (4, 4, 2, 32, 1031, 1280, 3.0),
    (4, 4, 1, 64, 4090, 1288, 0.0),
    (4, 8, 1, 30, 3999, 4104, 3.0),
    (8, 8, 3, 16, 260, 2048, 3.0),
    (8, 8, 1, 32, 1901, 4096, 3.0),
])
def test_logits_of_a_step_against_64_bits(parts, chains, Bn, L, n, d, lam):
    """The ring after a step with k in parts, as the tests of the LM head bound its kernels. (scd_lm_head adds up in another
    order on these shapes: the two agree to rounding only.)"""
    v_lo, tau = 5, 0.8
    W, h = _inputs(Bn, 2 if lam else 1, L, n, d, v_lo, n + d)
    sc = B.Scd(B.make_config(B=Bn, L=L, N=400, V=W.shape[0], d=d, v_lo=v_lo, v_hi=v_lo + n, temperature=tau, cfg_lambda=lam,
                             top_k=n // 5), "cuda:0")
    st = sc.alloc_state()
    sc.reset(st)
    assert (st.numel() - _fields_end(sc, st)) // (4 * Bn * L * n * (2 if lam else 1)) == parts
    ring = sc.state_field(st, B.F_Z).view(2, Bn, L, n)
    ring.fill_(float("nan"))
    sc.step(h, W, st)
    want, bound = _want(W, h, n, v_lo, lam, tau)
    diff = ring[0].double() - want
    assert bool((diff.abs() <= bound).all()) and bool(ring[1].isnan().all())
    # the tiles' bound on the rounding of a logit added up in `chains` chains
    err = float(diff.norm() / want.norm())
    assert err <= 0.7 * 2.0 ** -24 * np.sqrt(d / 32 / chains + (chains + 1) / 2), err
    alone = torch.empty(Bn, L, n, device="cuda:0")
    sc.lm_head(h, W, alone)
    assert bool(((alone.double() - ring[0].double()).abs() <= 2 * bound).all())
