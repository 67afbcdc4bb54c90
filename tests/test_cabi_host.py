"""Host-only checks of the C ABI (no GPU, no kernel launches): the library
loads, exports every symbol the headers declare, and validates arguments."""
import ctypes
import os
import re

import pytest

from paper_2510_24211_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    names = set()
    for hdr in ("scd.h", "scd_workload.h"):
        src = open(os.path.join(ROOT, "include", hdr)).read()
        src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
        names |= set(re.findall(r"\b(scdw?_[a-z_]+)\s*\(", src))
    return names


def test_library_exports_every_declared_symbol():
    lib = B.load()
    decl = _declared_symbols()
    assert {"scd_step", "scd_verify", "scd_couple_draft", "scd_lm_head"} <= decl
    for name in decl:
        assert hasattr(lib, name), name


def test_config_struct_matches_header_layout(tmp_path):
    """sizeof / offsetof as the C compiler sees the header against the ctypes mirror."""
    import os
    import subprocess
    fields = [name for name, _ in B.ScdConfig._fields_]
    src = tmp_path / "layout.c"
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "scd.h"\nint main(void) {\n'
                   '  printf("%zu", sizeof(scd_config));\n' +
                   "".join(f'  printf(" %zu", offsetof(scd_config, {f}));\n' for f in fields) +
                   "  return 0;\n}\n")
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-I", inc, str(src), "-o", str(exe)], check=True)
    got = [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]
    assert got[0] == ctypes.sizeof(B.ScdConfig) == 64
    assert got[1:] == [getattr(B.ScdConfig, f).offset for f in fields]


def test_size_queries_validate_config():
    ok = B.make_config(B=2, L=32, N=100, V=1000, d=64, top_k=10)
    assert B.workspace_bytes(ok) > 0
    # state holds two copies of the [B, L, n] fp32 logits plus small arrays
    assert B.state_bytes(ok) >= 2 * 2 * 32 * 1000 * 4
    bad = [dict(B=0), dict(L=0), dict(L=257), dict(N=0), dict(V=0), dict(d=12), dict(d=-8),
           dict(v_lo=-1), dict(v_lo=10, v_hi=10), dict(v_hi=1001), dict(top_k=-1),
           dict(temperature=0.0), dict(temperature=float("nan")), dict(cfg_lambda=float("inf"))]
    for kw in bad:
        args = dict(B=2, L=32, N=100, V=1000, d=64, top_k=10)
        args.update(kw)
        cfg = B.make_config(**args)
        assert B.workspace_bytes(cfg) == 0, kw
        assert B.state_bytes(cfg) == 0, kw


@pytest.mark.parametrize("kw", [
    dict(B=2, L=32, V=2048, d=2048, cfg_lambda=3.0, top_k=500),      # k in 4 parts
    dict(B=1, L=64, V=4090, d=1280),                                  # in 4, without guidance
    dict(B=5, L=26, V=1285, d=1288),                                  # in 2
    dict(B=1, L=32, V=16384, d=1280, top_k=1000),                     # not split
])
def test_a_step_on_short_rows_has_its_scratch_in_the_state(kw):
    """The workspace of such a context may serve another stream meanwhile: it holds what the stages and the lists need
    (six words per row; 6144 pairs, 256 counts and 256 cuts per row), whether or not there is an LM head."""
    cfg, bare = B.make_config(N=400, **kw), B.make_config(N=400, **dict(kw, d=0))
    rows = kw["B"] * kw["L"]
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    assert B.workspace_bytes(cfg) == 6 * up(4 * rows) + up(rows * 6144 * 8 + 2 * up(rows * 256 * 4))
    assert B.workspace_bytes(cfg) == B.workspace_bytes(bare)
    extra = B.state_bytes(cfg) - B.state_bytes(bare)
    assert extra <= 4 << 20 and (extra > 0) == (kw["V"] < 16384)


def test_k_is_dealt_in_parts_that_the_row_kernels_add_up():
    """Eight logits per thread in up to 4 parts (rows of up to 4096 ids), four (2048) in up to 8; longer rows in one."""
    seen = set()
    for n in (255, 256, 1000, 1024, 1025, 2048, 2049, 3000, 4095, 4096, 4097, 5000, 8192, 8193, 16384):
        for rows in (1, 8, 32, 33, 60, 64, 65, 96, 97, 128, 129, 256, 500, 1024):
            for d in (64, 1024, 1280, 2048, 4096, 16384):
                for lam in (0.0, 3.0):
                    kw = dict(B=-(-rows // 64), L=min(rows, 64), N=400, V=n, cfg_lambda=lam)
                    extra = B.state_bytes(B.make_config(d=d, **kw)) - B.state_bytes(B.make_config(**kw))
                    one = 4 * kw["B"] * kw["L"] * n * (2 if lam else 1)
                    parts = extra // one                 # (each array's share of the last 255 bytes is less than one)
                    assert extra - parts * one < 256 and parts in ((0, 2, 4, 8) if n <= 2048 else (0, 2, 4) if n <= 4096 else (0,))
                    seen.add((n <= 2048, parts))
    assert {(True, 2), (True, 4), (True, 8), (False, 2), (False, 4)} <= seen


def test_create_rejects_bad_arguments_without_touching_the_device():
    lib = B.load()
    cfg = B.make_config(B=1, L=8, N=64, V=1024)
    need = B.workspace_bytes(cfg)
    ctx = ctypes.c_void_p()
    fake = ctypes.c_void_p(0x10000)          # never dereferenced by scd_create
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(cfg), None, need, None) == B.SCD_EWORKSPACE
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(cfg), ctypes.c_void_p(0x10010), need, None) \
        == B.SCD_EWORKSPACE                                   # misaligned
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(cfg), fake, need - 1, None) == B.SCD_EWORKSPACE
    assert lib.scd_create(None, ctypes.byref(cfg), fake, need, None) == B.SCD_EINVAL
    bad = B.make_config(B=1, L=8, N=64, V=1024, coupling=2)           # no such coupling
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(bad), fake, need, None) == B.SCD_EUNSUPPORTED
    neg = B.make_config(B=1, L=8, N=64, V=1024, sjd_mix=1.5)           # probability outside [0, 1]
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(neg), fake, need, None) == B.SCD_EINVAL
    big = B.make_config(B=1, L=8, N=64, V=70000, coupling=B.COUPLING_GS)   # GS: rows <= 65536 ids
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(big), fake, 1 << 40, None) == B.SCD_EUNSUPPORTED
    wide = B.make_config(B=1, L=8, N=64, V=70000, top_p=0.8)          # nucleus: rows <= 65536 ids
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(wide), fake, 1 << 40, None) == B.SCD_EUNSUPPORTED
    dg = B.make_config(B=1, L=8, N=64, V=70000, diagnostics=1)        # statistics: rows <= 65536 ids
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(dg), fake, 1 << 40, None) == B.SCD_EUNSUPPORTED
    off = B.make_config(B=1, L=8, N=64, V=1024, top_p=1.25)            # mass outside [0, 1]
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(off), fake, need, None) == B.SCD_EINVAL
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(cfg), fake, need, None) == B.SCD_OK
    # null pointers are refused before any launch
    assert lib.scd_lm_head(ctx, None, None, None) == B.SCD_EINVAL
    assert lib.scd_step(ctx, None, None, None) == B.SCD_EINVAL
    assert lib.scd_step_logits(ctx, None, None) == B.SCD_EINVAL
    assert lib.scd_couple_draft(ctx, None, None, None, None, None, 0, None, None) == B.SCD_EINVAL
    assert lib.scd_verify(ctx, None, None, None, None, None) == B.SCD_EINVAL
    assert lib.scd_reset(ctx, None) == B.SCD_EINVAL
    # d == 0: the LM-head entry points are refused
    assert lib.scd_lm_head(ctx, fake, fake, fake) == B.SCD_EINVAL
    # state layout is host arithmetic: fields are disjoint, aligned, inside the buffer
    total = B.state_bytes(cfg)
    base = 0x100000
    spans = []
    for f in range(B.F_COUNT):
        p, nb = ctypes.c_void_p(), ctypes.c_size_t()
        assert lib.scd_state_field(ctx, ctypes.c_void_p(base), f, ctypes.byref(p), ctypes.byref(nb)) == 0
        assert p.value % 256 == 0 and nb.value > 0
        spans.append((p.value - base, p.value - base + nb.value))
    spans.sort()
    assert spans[-1][1] <= total
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
    assert lib.scd_state_field(ctx, ctypes.c_void_p(base), B.F_COUNT, ctypes.byref(p), ctypes.byref(nb)) == B.SCD_EINVAL
    assert lib.scd_destroy(ctx) == B.SCD_OK
    assert lib.scd_destroy(None) == B.SCD_EINVAL
    assert B.strerror(B.SCD_EWORKSPACE).startswith("workspace")


@pytest.mark.parametrize("kw,step,alone", [
    (dict(L=32, V=1900, d=4096, cfg_lambda=3.0), "lm_head_tile_kernel<2, 64, 128, 6, false>", "lm_head_splitk_kernel<1, 2, 8>"),
    (dict(B=4, L=64, V=4096, d=4096), "lm_head_tile_kernel<1, 64, 128, 6, false>", "lm_head_tile_kernel<1, 64, 128, 6, false>"),
    (dict(L=32, V=8192, d=4096, cfg_lambda=3.0), "lm_head_splitk_kernel<1, 2, 8>", "lm_head_splitk_kernel<1, 2, 8>"),
])
def test_kernel_names_of_a_step_and_of_the_head_alone(kw, step, alone):
    lib = B.load()
    cfg = B.make_config(N=400, **dict(dict(B=1), **kw))
    ctx = ctypes.c_void_p()
    assert lib.scd_create(ctypes.byref(ctx), ctypes.byref(cfg), ctypes.c_void_p(0x10000), 1 << 40, None) == B.SCD_OK
    want = step if step == alone else step + " / " + alone
    buf = ctypes.create_string_buffer(96)
    assert lib.scd_lm_head_kernel_name(ctx, buf, 96) == B.SCD_OK and buf.value.decode() == want
    assert lib.scd_lm_head_kernel_name(ctx, buf, len(want) + 1) == B.SCD_OK and buf.value.decode() == want
    assert lib.scd_lm_head_kernel_name(ctx, buf, len(want)) == (B.SCD_EINVAL if step == alone else B.SCD_OK)
    assert step == alone or buf.value.decode() == step
    assert lib.scd_lm_head_kernel_name(ctx, buf, len(step)) == B.SCD_EINVAL
    assert lib.scd_destroy(ctx) == B.SCD_OK


def test_gather_rejects_bad_arguments():
    lib = B.load()
    fake = ctypes.c_void_p(0x10000)
    assert lib.scdw_gather_hidden(None, None, 1, 1, 8, 64, 64, 4, fake, fake, fake) == -1
    assert lib.scdw_gather_hidden(None, fake, 1, 1, 8, 64, 60, 4, fake, fake, fake) == -1
