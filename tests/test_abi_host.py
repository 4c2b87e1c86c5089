"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol include/moe.h declares,
and rejects bad arguments before anything is launched."""
import copy
import ctypes
import os
import re

import pytest

import paper_2605_05049_amd as moe
from paper_2605_05049_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    return moe.load_library()


def test_exports_every_declared_symbol(lib):
    header = open(os.path.join(ROOT, "include", "moe.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(moe_[a-z_0-9]+)\s*\(", header))
    assert declared == set(moe.EXPORTED_SYMBOLS)
    for name in declared:
        assert hasattr(lib, name), name
    assert moe.abi_version() == 1


def test_status_strings(lib):
    assert moe.status_str(0) == "ok"
    for code in (-1, -2, -3, -4, -5):
        assert moe.status_str(code) not in ("ok", "unknown status")
    assert moe.status_str(-99) == "unknown status"


def test_workspace_bytes_follows_the_shape(lib):
    s = moe.Shape(256, 512, 1024, 8, 2)
    n = moe.workspace_bytes(s)
    # three [N,f] bf16 intermediates (H, dG, dU) plus the fixed 80 MiB of partial tiles of split contractions
    assert 3 * s.N * s.d_ffn * 2 + (80 << 20) <= n <= 3 * s.N * s.d_ffn * 2 + (82 << 20) and n % 256 == 0
    assert moe.workspace_bytes(moe.Shape(512, 512, 1024, 8, 2)) > n
    assert moe.workspace_bytes(moe.Shape(256, 500, 1024, 8, 2)) == 0       # d not a multiple of 64
    assert moe.workspace_bytes(moe.Shape(256, 512, 1024, 8, 9)) == 0       # k > E
    assert moe.workspace_bytes(moe.Shape(256, 512, 1024, 2000, 2)) == 0    # E over the limit
    assert moe.workspace_bytes(moe.Shape(2 ** 30, 512, 1024, 8, 2)) == 0   # T*K' >= 2^31
    assert moe.workspace_bytes(moe.Shape(1, 2 ** 22, 64, 8, 2)) > 0        # the widest rows the GEMM loads can address
    assert moe.workspace_bytes(moe.Shape(1, 2 ** 22 + 64, 64, 8, 2)) == 0  # beyond: the 32-bit row offsets would wrap
    assert moe.workspace_bytes(moe.Shape(1, 64, 2 ** 22 + 64, 8, 2)) == 0


def test_shape_fields_stay_consistent():
    s = moe.Shape(256, 512, 1024, 8, 2, 1)
    s.T = 100
    assert (s.N, s.K_slots, s.E_total) == (300, 3, 9) and s._c.T == 100
    s.E_shared = 0
    assert (s.N, s.K_slots, s.E_total) == (200, 2, 8)
    assert moe.workspace_bytes(s) == moe.workspace_bytes(moe.Shape(100, 512, 1024, 8, 2))
    for derived in ("N", "K_slots", "E_total"):
        with pytest.raises(AttributeError):
            setattr(s, derived, 1)
    t = copy.copy(s)
    t.T = 7
    assert (s.N, t.N, s._c.T, t._c.T) == (200, 14, 100, 7)


def _shape(**kw):
    base = dict(T=256, d_model=512, d_ffn=1024, E=8, k=2, E_shared=0, renorm=1)
    base.update(kw)
    return moe.Shape(**base)


FAKE = ctypes.c_void_p(0x10000)        # aligned, never dereferenced: every call below fails its host checks first
ODD = ctypes.c_void_p(0x10004)


def test_argument_checks_run_before_any_launch(lib):
    s = _shape()
    sp = ctypes.byref(s._c)
    bad = ctypes.byref(_shape(k=0)._c)
    assert lib.moe_route_topk(sp, None, FAKE, FAKE, None, None) == -1
    assert lib.moe_route_topk(bad, FAKE, FAKE, FAKE, None, None) == -2
    assert lib.moe_route_topk(sp, ODD, FAKE, FAKE, None, None) == -3
    assert lib.moe_route_topk(None, FAKE, FAKE, FAKE, None, None) == -1
    assert lib.moe_route_topk_bwd(sp, FAKE, FAKE, FAKE, None, None, None) == -1
    nr = ctypes.byref(_shape(renorm=0)._c)
    assert lib.moe_route_topk_bwd(nr, FAKE, FAKE, FAKE, None, FAKE, None) == -1    # probs needed without renorm
    assert lib.moe_permute(sp, FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 40, None) == -1
    assert lib.moe_permute(sp, FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 40, None) == -1   # x without x_perm
    assert lib.moe_permute(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 16, None) == -4
    assert lib.moe_permute(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, ctypes.c_void_p(0x10010), 1 << 40, None) == -3
    assert lib.moe_permute_bwd(sp, FAKE, None, FAKE, None) == -1
    assert lib.moe_grouped_ffn_fwd(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 16, None) == -4
    assert lib.moe_grouped_ffn_fwd(sp, FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 40, None) == -1
    assert lib.moe_grouped_ffn_fwd(bad, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 40, None) == -2
    wide = ctypes.byref(_shape(d_model=2 ** 22 + 64)._c)
    assert lib.moe_grouped_ffn_fwd(wide, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 40, None) == -2
    assert lib.moe_grouped_ffn_bwd(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, 0,
                                   FAKE, 1 << 40, None) == -1
    assert lib.moe_grouped_ffn_bwd(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 0,
                                   FAKE, 16, None) == -4
    assert lib.moe_grouped_ffn_fwd(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, FAKE, FAKE, 1 << 40, None) == -1   # G without U
    assert lib.moe_grouped_ffn_bwd_recompute(sp, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 0, FAKE, 16, None) == -4
    assert lib.moe_grouped_ffn_bwd_recompute(sp, FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 0, FAKE, 1 << 40, None) == -1
    assert lib.moe_grouped_ffn_bwd_recompute(sp, None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 0, FAKE, 1 << 40, None) == -1
    assert lib.moe_unpermute_combine(sp, FAKE, FAKE, None, FAKE, None) == -1
    assert lib.moe_unpermute_combine(sp, FAKE, FAKE, ODD, FAKE, None) == -3
    assert lib.moe_unpermute_combine_bwd(sp, FAKE, FAKE, FAKE, FAKE, FAKE, None, None) == -1
    assert lib.moe_permute_bwd_add(sp, FAKE, FAKE, None, FAKE, None) == -1
    assert lib.moe_permute_bwd_add(sp, FAKE, FAKE, ODD, FAKE, None) == -3
    assert lib.moe_router_fwd(sp, FAKE, None, FAKE, FAKE, 1 << 40, None) == -1
    assert lib.moe_router_fwd(sp, FAKE, FAKE, FAKE, FAKE, 16, None) == -4
    assert lib.moe_router_fwd(bad, FAKE, FAKE, FAKE, FAKE, 1 << 40, None) == -2
    ffn = [FAKE] * 12
    assert lib.moe_grouped_ffn_router_bwd(sp, *ffn, FAKE, FAKE, FAKE, FAKE, None, 0, FAKE, 1 << 40, None) == -1
    assert lib.moe_grouped_ffn_router_bwd(sp, *ffn, FAKE, FAKE, ODD, FAKE, FAKE, 0, FAKE, 1 << 40, None) == -3
    assert lib.moe_grouped_ffn_router_bwd(sp, *ffn[:11], None, FAKE, FAKE, FAKE, FAKE, FAKE, 0, FAKE, 1 << 40, None) == -1
    assert lib.moe_grouped_ffn_router_bwd(sp, *ffn, FAKE, FAKE, FAKE, FAKE, FAKE, 0, FAKE, 256, None) == -4
    assert lib.moe_router_bwd(sp, FAKE, FAKE, FAKE, FAKE, None, 0, FAKE, 1 << 40, None) == -1
    assert lib.moe_router_bwd(sp, FAKE, FAKE, ODD, FAKE, FAKE, 0, FAKE, 1 << 40, None) == -3
    assert lib.moe_router_bwd(sp, FAKE, FAKE, FAKE, FAKE, FAKE, 0, None, 0, None) == -1


def test_binding_rejects_host_tensors(lib):
    import torch
    s = _shape(T=4)
    with pytest.raises(ValueError):
        moe.moe_route_topk(s, torch.zeros(4, 8), torch.zeros(4, 2, dtype=torch.int32), torch.zeros(4, 2))


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_LIB_NAME", "libmoe_does_not_exist.so")
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        B.load_library()


# (T, d, f, E, k) -> the GEMMs on 64-row tiles, and not on those of 128 columns, which are asked first.  Each goes by its own output width and
# contraction: a layer that is small in d_ffn is not small in its down projection and dX (and the other way round).
@pytest.mark.parametrize("T,d,f,E,k,expected", [
    (256, 512, 1024, 8, 2, ("down", "dh", "dx")),
    (8192, 7168, 512, 4, 1, ()),
    (512, 7168, 512, 1, 1, ("gate_up", "dh")),
    (1024, 7168, 512, 1, 1, ("gate_up", "dh")),    # 128 tiles of gate | up and dH, 1792 of down and dX
    (8192, 7168, 512, 8, 1, ()),                   # 17000 tiles of down and dX, twice the time on them
    (64, 7168, 1024, 8, 1, ("gate_up",)),          # 112 k-steps of dH, which the 256-row kernel cuts along k
    (32, 512, 2048, 4, 1, ("down", "dh", "dx")),   # 64 k-steps of dX: 0.79 of the 256-row kernel's time
    (32, 512, 14336, 4, 1, ()),                    # 32 tiles of down and dX, but 224 and 448 k-steps
    (8, 4096, 14336, 1, 1, ("gate_up",)),
    (4096, 1024, 2048, 1, 1, ()),                  # 1024 64-row tiles of down and dX, 2048 of the others
    (2048, 1024, 2048, 32, 1, ()),                 # 768 and more
    (4096, 4096, 14336, 8, 2, ()),
    (0, 512, 1024, 8, 2, ("gate_up", "down", "dh", "dx")),
])
def test_which_gemms_run_on_small_tiles(lib, T, d, f, E, k, expected):
    assert moe.grouped_ffn_small_tiles(moe.Shape(T, d, f, E, k)) == expected


# Both sides of the limits of few rows per expert and long contractions: 200 tiles and 128 k-steps of down, 256 tiles and 200 of dX, which are one
# limit from 48 k-steps on
@pytest.mark.parametrize("T,d,f,E,k,down,dx", [
    (200, 512, 6144, 25, 1, True, True),       # 200 tiles of 96 and 192 steps
    (200, 512, 6144, 26, 1, False, True),      # 208
    (200, 512, 6144, 33, 1, False, False),     # 264
    (200, 512, 6400, 25, 1, True, False),      # 100 and 200 steps
    (200, 512, 8192, 25, 1, False, False),     # 128 and 256
    (600, 512, 3584, 20, 1, True, True),       # 30 rows per expert: 160 tiles of dX, 112 steps
    (990, 512, 3584, 33, 1, True, False),      # 264, and of down, 56 steps
    (80, 512, 1984, 10, 1, True, True),        # 8 rows per expert: 80 tiles of dX of 62 steps,
    (80, 512, 2048, 10, 1, True, True),        # 64,
    (80, 512, 3008, 10, 1, True, True),        # 94
    (80, 512, 3072, 10, 1, True, True),        # and 96
    (1032, 128, 2560, 129, 1, True, False),    # 258 tiles of 80 steps (more than 128 experts: none of 128 columns)
    (1032, 64, 2560, 129, 1, True, True),      # 129
])
def test_small_tiles_of_few_rows_and_long_contractions(lib, T, d, f, E, k, down, dx):
    small = moe.grouped_ffn_small_tiles(moe.Shape(T, d, f, E, k))
    assert ("down" in small, "dx" in small) == (down, dx)


# (T, d, f, E, k) -> the GEMMs on the tiles of 128 columns: both sides of the least and the most tiles, by rows per expert and k-steps
@pytest.mark.parametrize("T,d,f,E,k,expected", [
    (256, 512, 1024, 8, 2, ("gate_up",)),                  # 128 tiles of gate | up, 64 of the others
    (1003, 1088, 1984, 14, 4, ("gate_up", "down", "dh", "dx")),
    (4096, 4096, 14336, 8, 2, ()),                         # 8000 tiles, contractions of 64 steps and more
    (8192, 2048, 1408, 66, 8, ()),                         # 32 steps of dH, 6000 tiles
    (2048, 2048, 1408, 66, 8, ("dh", "dx")),               # ... and 1400
    (7871, 832, 2624, 24, 6, ("dh",)),                     # 13 steps of dH: any number of tiles
    (16, 2048, 1408, 66, 8, ("gate_up", "down", "dx")),    # 726 tiles of dH, 32 steps, two rows per expert
    (512, 4096, 14336, 8, 1, ("down", "dx")),              # 1792 tiles of gate | up, 256 of down and dX
    # even counts that fill rounds of 256-row tiles: 32 row tiles of 248 .. 264 rows, 256 tiles of down and 192 of dH
    (7872, 2048, 1408, 8, 1, ("down", "dh", "dx")),        # 246 rows
    (7936, 2048, 1408, 8, 1, ("dx",)),
    (8448, 2048, 1408, 8, 1, ("dx",)),
    (8640, 2048, 1408, 8, 1, ("down", "dx")),              # 270
    (4096, 2048, 1408, 4, 1, ("dh", "dx")),                # 176 and 128 tiles of gate | up and down; dH else on 64-row tiles
    (4096, 4096, 1024, 8, 1, ("dh", "dx")),                # 128 and 256
    (2048, 7168, 2048, 8, 1, ("dh", "dx")),                # 224 tiles of down, 64 of dH
    (4012, 1088, 1984, 14, 1, ("gate_up", "down", "dh", "dx")),   # 287 rows
    (2048, 4096, 14336, 8, 1, ()),                         # 640 tiles of dX, 448 steps; even counts are 128 tiles, half a round
    (2240, 4096, 14336, 8, 1, ("dx",)),                    # 280 rows
    (2048, 4096, 9536, 8, 1, ("dx",)),                     # 298 steps,
    (2048, 4096, 9600, 8, 1, ()),                          # 300
    (2400, 4352, 14336, 8, 1, ("dx",)),                    # 748 tiles,
    (2400, 4416, 14336, 8, 1, ()),                         # 770
    (3600, 576, 11136, 12, 1, ("gate_up", "down", "dh", "dx")),   # 170 tiles, 348 steps; 2.25 column tiles of 256
    (4800, 512, 11136, 16, 1, ("gate_up", "down", "dh")),   # 180; 2
    (512, 4096, 14336, 4, 1, ("down", "dh")),              # 192 tiles of dX, 128 rows
    (768, 4096, 14336, 4, 1, ("down", "dx")),              # 256
    (256, 4096, 14336, 4, 1, ("gate_up", "dh")),           # 128, 64 rows
    (320, 4096, 14336, 5, 1, ("gate_up", "down", "dh", "dx")),   # 160
    (576, 4096, 14336, 9, 1, ("down", "dx")),              # 288,
    (640, 4096, 14336, 10, 1, ("down",)),                  # 320
    (2048, 3200, 14336, 8, 1, ("dx",)),                    # 500 tiles,
    (2048, 3328, 14336, 8, 1, ()),                         # 520
    (300, 512, 1024, 129, 1, ()),                          # more experts than a block finds its tile among
    (0, 512, 1024, 8, 2, ()),
])
def test_which_gemms_run_on_mid_tiles(lib, T, d, f, E, k, expected):
    assert moe.grouped_ffn_mid_tiles(moe.Shape(T, d, f, E, k)) == expected


def test_small_tiles_of_an_invalid_shape(lib):
    assert moe.grouped_ffn_mid_tiles(moe.Shape(8, 500, 64, 4, 1)) == ()
    assert moe.grouped_ffn_small_tiles(moe.Shape(8, 500, 64, 4, 1)) == ()
