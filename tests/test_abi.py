"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol include/fq.h declares, and rejects bad arguments before touching
the device."""
import ctypes as C
import os
import re

import pytest

import paper_2503_08040_amd as fq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "fq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fq_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = fq.lib()
    names = _declared_symbols()
    assert set(names) == set(fq.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_qtensor_bytes_and_bind():
    assert fq.fq_qtensor_bytes(0, 0, 0) > 0
    nb = 2 * 4
    small = fq.fq_qtensor_bytes(256, 512, 0)
    big = fq.fq_qtensor_bytes(256, 512, nb)
    assert big - small >= nb * fq.FQ_BLOCK_BYTES - 512
    assert fq.fq_qtensor_bytes(256, 512, nb, True) - big >= 2 * nb * fq.FQ_BLOCK_BYTES - 512
    assert fq.fq_qtensor_bytes(256, 512, nb + 1) == 0          # capacity beyond nbr*nbc
    assert fq.fq_qtensor_bytes(-1, 5, 0) == 0
    assert fq.fq_qtensor_bytes(256, 512, 1, block=64) == 0
    t = fq.fq_qtensor()
    base = 0x10000
    assert fq.lib().fq_qtensor_bind(C.c_void_p(base), 130, 200, 128, 3, 1, C.byref(t)) == fq.FQ_OK
    assert (t.rows, t.cols, t.block, t.capacity) == (130, 200, 128, 3)
    ptrs = [t.codes, t.codes_t, t.scales, t.mask, t.fb_counters, t.fb_list, t.fb_slot, t.res_codes,
            t.res_codes_t, t.res_scales]
    assert all(p and p % 256 == 0 for p in ptrs) and len(set(ptrs)) == len(ptrs)
    assert t.fb_count == t.fb_counters and t.epoch == 0
    assert max(ptrs) < base + fq.fq_qtensor_bytes(130, 200, 3, True)
    assert fq.lib().fq_qtensor_bind(C.c_void_p(base + 8), 130, 200, 128, 3, 1, C.byref(t)) == fq.FQ_ERR_SHAPE
    assert fq.lib().fq_qtensor_bind(None, 130, 200, 128, 3, 1, C.byref(t)) == fq.FQ_ERR_NULL
    assert fq.lib().fq_qtensor_bind(C.c_void_p(base), 130, 200, 64, 3, 1, C.byref(t)) == fq.FQ_ERR_BLOCK


def _fake(rows, cols, cap=1, want_t=True, crit=fq.FQ_CRIT_NONE):
    """A struct with non-NULL fake pointers: valid for host-side validation only."""
    t = fq.fq_qtensor()
    assert fq.lib().fq_qtensor_bind(C.c_void_p(0x100000), rows, cols, 128, cap, int(want_t),
                                    C.byref(t)) == fq.FQ_OK
    t.criterion = crit
    return t


def test_quantize_rejects_bad_arguments_on_the_host():
    L = fq.lib()
    t = _fake(256, 256)
    x = C.c_void_p(0x2000)
    q = lambda *a: L.fq_quantize(*a)
    assert q(x, 256, 256, 256, 128, 0, 0.0, None, None) == fq.FQ_ERR_NULL
    assert q(None, 256, 256, 256, 128, 0, 0.0, C.byref(t), None) == fq.FQ_ERR_NULL
    assert q(x, 256, 256, 256, 64, 0, 0.0, C.byref(t), None) == fq.FQ_ERR_BLOCK
    assert q(x, 256, 256, 255, 128, 0, 0.0, C.byref(t), None) == fq.FQ_ERR_SHAPE     # ld < cols
    assert q(x, -1, 256, 256, 128, 0, 0.0, C.byref(t), None) == fq.FQ_ERR_SHAPE
    assert q(x, 128, 256, 256, 128, 0, 0.0, C.byref(t), None) == fq.FQ_ERR_SHAPE     # shape != out
    assert q(x, 256, 256, 256, 128, 7, 0.0, C.byref(t), None) == fq.FQ_ERR_ENUM
    t0 = _fake(256, 256, cap=0)
    assert q(x, 256, 256, 256, 128, 1, 0.0, C.byref(t0), None) == fq.FQ_ERR_CAPACITY
    t.codes = None
    assert q(x, 256, 256, 256, 128, 0, 0.0, C.byref(t), None) == fq.FQ_ERR_NULL


def test_gemm_rejects_bad_arguments_on_the_host():
    L = fq.lib()
    out = C.c_void_p(0x3000)
    A, Bm = _fake(256, 512, crit=fq.FQ_CRIT_ABSMAX_GT), _fake(384, 512)
    g = lambda *a: L.fq_gemm(*a)
    assert g(0, None, C.byref(Bm), out, 0, 384, None) == fq.FQ_ERR_NULL
    assert g(0, C.byref(A), C.byref(Bm), None, 0, 384, None) == fq.FQ_ERR_NULL
    assert g(5, C.byref(A), C.byref(Bm), out, 0, 384, None) == fq.FQ_ERR_ENUM
    assert g(0, C.byref(A), C.byref(Bm), out, 9, 384, None) == fq.FQ_ERR_ENUM
    assert g(0, C.byref(A), C.byref(Bm), out, 0, 383, None) == fq.FQ_ERR_SHAPE        # ldc < N
    assert g(0, C.byref(A), C.byref(_fake(384, 640)), out, 0, 384, None) == fq.FQ_ERR_SHAPE
    # NN needs A.cols == B.rows, TN needs A.rows == B.rows
    assert g(1, C.byref(A), C.byref(Bm), out, 0, 512, None) == fq.FQ_ERR_SHAPE
    assert g(2, C.byref(A), C.byref(Bm), out, 0, 512, None) == fq.FQ_ERR_SHAPE
    # the B operand must be plain block INT8 (Alg. 1 defines fallback for A only)
    Bf = _fake(384, 512, crit=fq.FQ_CRIT_ABSMAX_GT)
    assert g(0, C.byref(A), C.byref(Bf), out, 0, 384, None) == fq.FQ_ERR_ENUM
    # backward forms need the transposed copies
    Bnt = _fake(512, 384, want_t=False)
    assert g(1, C.byref(A), C.byref(Bnt), out, 0, 384, None) == fq.FQ_ERR_NULL
    Ant = _fake(256, 512, want_t=False, crit=fq.FQ_CRIT_ABSMAX_GT)
    assert g(2, C.byref(Ant), C.byref(_fake(256, 384)), out, 0, 384, None) == fq.FQ_ERR_NULL
    A.block = 64
    assert g(0, C.byref(A), C.byref(Bm), out, 0, 384, None) == fq.FQ_ERR_BLOCK
    A.block = 128
    p = lambda *a: L.fq_gemm_debug_partials(*a)
    assert p(0, C.byref(A), C.byref(Bm), 4, 0, out, None) == fq.FQ_ERR_SHAPE          # nkb = 4
    assert p(0, C.byref(A), C.byref(Bm), -1, 0, out, None) == fq.FQ_ERR_SHAPE
    assert p(0, C.byref(A), C.byref(Bm), 0, 0, None, None) == fq.FQ_ERR_NULL


def test_status_strings():
    for s in range(0, -8, -1):
        assert fq.status_string(s) and "unknown" not in fq.status_string(s)
    assert "unknown" in fq.status_string(-99)


def test_untile_rejects_bad_arguments():
    L = fq.lib()
    assert L.fq_codes_to_rowmajor(None, 4, 4, C.c_void_p(0x10), None) == fq.FQ_ERR_NULL
    assert L.fq_codes_to_rowmajor(C.c_void_p(0x10), -4, 4, C.c_void_p(0x10), None) == fq.FQ_ERR_SHAPE
    assert L.fq_codes_to_rowmajor(None, 0, 4, None, None) == fq.FQ_OK


def test_tile_plan_covers_the_output_and_never_costs_more():
    """fq_gemm_tile_plan (host-only): 256x256 tiles over the first block columns, 128x384 tiles
    over the rest; every block column is covered exactly once, and the plan is only split when
    that shortens the last round (costs in units of one 256x256 tile per compute unit)."""
    import itertools
    import random
    rng = random.Random(0)
    cases = [(4096, 11008, 256), (8192, 8192, 256), (4096, 4096, 256), (11008, 4096, 256), (1, 1, 256)]
    cases += [(rng.randint(1, 6000), rng.randint(1, 14000), rng.choice([1, 3, 8, 64, 256, 304]))
              for _ in range(300)]
    split = 0
    for rows, cols, cus in cases:
        n_main, main_tj, tail_tj = fq.fq_gemm_tile_plan(rows, cols, cus)
        nib, njb = -(-rows // 128), -(-cols // 128)
        tiles_i, tiles_j = -(-nib // 2), -(-njb // 2)
        assert n_main == tiles_i * main_tj and 0 <= main_tj <= tiles_j and tail_tj >= 0
        if tail_tj == 0:
            assert main_tj == tiles_j
            continue
        split += 1
        tail_cols = njb - 2 * main_tj
        assert tail_cols > 0 and 3 * (tail_tj - 1) < tail_cols <= 3 * tail_tj
        rounds = lambda n: -(-n // cus)
        assert rounds(n_main) + 0.75 * rounds(nib * tail_tj) < rounds(tiles_i * tiles_j)
    assert split > 10
    assert fq.fq_gemm_tile_plan(4096, 11008, 256) == (512, 32, 8)
    assert fq.fq_gemm_tile_plan(8192, 8192, 256) == (1024, 32, 0)
    p = (C.c_int32 * 3)()
    assert fq.lib().fq_gemm_tile_plan(-1, 5, 4, p) == fq.FQ_ERR_SHAPE
    assert fq.lib().fq_gemm_tile_plan(5, 5, 4, None) == fq.FQ_ERR_NULL


def test_gemm_path_says_what_covers_the_output():
    """fq_gemm_path (host-only): the tiles it names are as many as cover the output, 128x384 tiles appear
    over columns or over rows and only with 256x256 tiles, and the kinds of the documented shapes."""
    import random
    rng = random.Random(1)
    seen = set()
    for _ in range(600):
        rows, cols = (int(round(2 ** rng.uniform(0, 13.5))) for _ in range(2))
        cus, biased = rng.choice([1, 2, 3, 8, 64, 256, 304]), rng.random() < 0.5
        kind, n, over_cols, over_rows = fq.fq_gemm_path(rows, cols, cus, biased)
        ceil = lambda a, b: -(-a // b)
        if kind != fq.FQ_TILES_256x256:
            r, c = {fq.FQ_TILES_32x32: (32, 32), fq.FQ_TILES_128x64: (128, 64), fq.FQ_TILES_128x128: (128, 128)}[kind]
            assert (n, over_cols, over_rows) == (ceil(rows, r) * ceil(cols, c), 0, 0)
            seen.add(kind)
            continue
        nib, njb = ceil(rows, 128), ceil(cols, 128)
        ti, tj = ceil(nib, 2), ceil(njb, 2)
        assert n > 0 and not (over_cols and over_rows)
        seen.add((kind, over_cols > 0, over_rows > 0))
        if over_rows:
            assert n % tj == 0 and over_rows == (nib - 2 * (n // tj)) * ceil(njb, 3)
        elif over_cols:
            assert n % ti == 0 and over_cols == nib * ceil(njb - 2 * (n // ti), 3)
            assert fq.fq_gemm_tile_plan(rows, cols, cus) == (n, n // ti, over_cols // nib)
        else:
            assert n == ti * tj
    assert len(seen) == 6
    large = fq.FQ_TILES_256x256
    assert fq.fq_gemm_path(4096, 11008, 256) == (large, 512, 256, 0)
    assert fq.fq_gemm_path(11008, 4096, 256) == (large, 512, 0, 242)
    assert fq.fq_gemm_path(33, 11008, 256) == (fq.FQ_TILES_32x32, 688, 0, 0)
    assert fq.fq_gemm_path(512, 4096, 256) == (fq.FQ_TILES_128x64, 256, 0, 0)
    assert fq.fq_gemm_path(2048, 11008, 256) == (fq.FQ_TILES_128x128, 1376, 0, 0)
    assert fq.fq_gemm_path(2048, 11008, 256, biased=True) == (large, 256, 128, 0)
    assert fq.fq_gemm_path(0, 5, 256) == fq.fq_gemm_path(5, 0, 256) == (0, 0, 0, 0)
    p = (C.c_int32 * 4)()
    assert fq.lib().fq_gemm_path(-1, 5, 4, 0, p) == fq.FQ_ERR_SHAPE
    assert fq.lib().fq_gemm_path(5, 5, 4, 0, None) == fq.FQ_ERR_NULL


def test_gemm_form_says_which_kernel_runs():
    """fq_gemm_form (host-only): the kernels of the documented shapes, as many workgroups as cover the output, and for a
    long contraction and an A that can fall back the tiles that fq_gemm_path names."""
    import random
    ceil = lambda a, b: -(-a // b)
    edges = {fq.FQ_FORM_32x32: (32, 32, fq.FQ_TILES_32x32), fq.FQ_FORM_128x64: (128, 64, fq.FQ_TILES_128x64),
             fq.FQ_FORM_128x128: (128, 128, fq.FQ_TILES_128x128), fq.FQ_FORM_LOADERS_128x64: (128, 64, fq.FQ_TILES_128x64),
             fq.FQ_FORM_LOADERS_128x128: (128, 128, fq.FQ_TILES_128x128),
             fq.FQ_FORM_LOADERS_128x256: (128, 256, fq.FQ_TILES_128x128)}
    rng = random.Random(2)
    seen = set()
    for _ in range(800):
        rows, cols = (int(round(2 ** rng.uniform(0, 13.5))) for _ in range(2))
        cus, biased = rng.choice([1, 2, 3, 8, 64, 256, 304]), rng.random() < 0.3
        for falls_back in (True, False):
            form, n = fq.fq_gemm_form(rows, cols, 2 ** 24, cus, biased, falls_back)
            seen.add((form, falls_back))
            if form != fq.FQ_FORM_256x256:
                r, c, _ = edges[form]
                assert n == ceil(rows, r) * ceil(cols, c)
                # the kernels with wavefronts that only load run one round of workgroups, or two of the smallest
                assert form < fq.FQ_FORM_LOADERS_128x64 or n <= cus * (2 if form == fq.FQ_FORM_LOADERS_128x64 else 1)
            if falls_back:
                path = fq.fq_gemm_path(rows, cols, cus, biased)
                assert path[0] == (edges[form][2] if form else fq.FQ_TILES_256x256)
                if form == fq.FQ_FORM_256x256:
                    assert n == path[1] + path[2] + path[3]
    assert seen == {(f, b) for f in range(7) for b in (True, False)}
    for rows, cols, form, n in [(33, 11008, fq.FQ_FORM_32x32, 688), (777, 2200, fq.FQ_FORM_LOADERS_128x64, 245),
                                (512, 4096, fq.FQ_FORM_LOADERS_128x64, 256), (2048, 2048, fq.FQ_FORM_LOADERS_128x128, 256),
                                (2048, 4096, fq.FQ_FORM_LOADERS_128x256, 256), (1536, 4096, fq.FQ_FORM_128x64, 768),
                                (3072, 3072, fq.FQ_FORM_128x64, 1152), (2048, 9984, fq.FQ_FORM_128x128, 1248),
                                (4096, 11008, fq.FQ_FORM_256x256, 768)]:
        for falls_back in (True, False):
            assert fq.fq_gemm_form(rows, cols, 4096, 256, falls_back=falls_back) == (form, n)
    assert fq.fq_gemm_form(0, 5, 128, 256) == fq.fq_gemm_form(5, 0, 128, 256) == (0, 0)
    assert fq.fq_gemm_form(5, 5, 0, 256) == (fq.FQ_FORM_32x32, 1)
    p = (C.c_int32 * 2)()
    assert fq.lib().fq_gemm_form(-1, 5, 128, 4, 0, 0, p) == fq.FQ_ERR_SHAPE
    assert fq.lib().fq_gemm_form(5, 5, -1, 4, 0, 0, p) == fq.FQ_ERR_SHAPE
    assert fq.lib().fq_gemm_form(5, 5, 128, 4, 0, 0, None) == fq.FQ_ERR_NULL


def test_short_contractions_take_tiles_without_loaders():
    """The tiles with wavefronts that only load start later than the others, which a short contraction does not make up
    for: with them 2048 x 2048 outputs of two k-blocks took 9 to 15 % longer."""
    loaders = (fq.FQ_FORM_LOADERS_128x64, fq.FQ_FORM_LOADERS_128x128, fq.FQ_FORM_LOADERS_128x256)
    form = lambda rows, cols, nkb, falls_back: fq.fq_gemm_form(rows, cols, 128 * nkb, 256, falls_back=falls_back)[0]
    for rows, cols, without in [(512, 4096, fq.FQ_FORM_128x64), (777, 2200, fq.FQ_FORM_128x64),
                                (2048, 2048, fq.FQ_FORM_128x64), (3496, 640, fq.FQ_FORM_32x32),
                                (1838, 1280, fq.FQ_FORM_32x32), (2048, 4096, fq.FQ_FORM_128x128),
                                (1600, 4000, fq.FQ_FORM_128x64), (128, 10368, fq.FQ_FORM_32x32)]:
        for falls_back in (True, False):
            forms = [form(rows, cols, nkb, falls_back) for nkb in range(40)]
            first = next(k for k, f in enumerate(forms) if f in loaders)
            assert forms[:first] == [without] * first and len(set(forms[first:])) == 1
            wide = forms[-1] == fq.FQ_FORM_LOADERS_128x256
            assert first == (8 if not falls_back else 16 if wide or (rows, cols) == (128, 10368) else 12)
    # up to five 32 x 32 tiles per compute unit: as long as A fits an XCD's L2
    assert form(1024, 1280, 31, True) == form(1024, 1280, 31, False) == fq.FQ_FORM_32x32
    assert form(1024, 1280, 32, True) == form(1024, 1280, 32, False) == fq.FQ_FORM_LOADERS_128x64


def test_outputs_that_take_large_tiles_only_if_a_cannot_fall_back():
    """The line of the large tiles: 2050 ns per k-block without residual slots, 2340 with them, against 128 x 64 tiles of
    390 each and pairs of 128 x 128 of 1360, on 256 compute units."""
    kinds = lambda rows, cols: [fq.fq_gemm_form(rows, cols, 4096, 256, falls_back=f)[0] for f in (True, False)]
    for rows, cols, tiles in [(1280, 9700, fq.FQ_FORM_128x128), (4096, 5760, fq.FQ_FORM_128x128),
                              (1400, 8001, fq.FQ_FORM_128x64), (2048, 11008, fq.FQ_FORM_128x128)]:
        assert kinds(rows, cols) == [tiles, fq.FQ_FORM_256x256]
    assert kinds(3584, 3584) == kinds(1280, 9856) == [fq.FQ_FORM_256x256] * 2      # 6.1 and 6.02 128 x 64 tiles per unit
    assert kinds(1280, 8576) == kinds(2560, 4096) == [fq.FQ_FORM_128x64] * 2       # 5.2 and 5
