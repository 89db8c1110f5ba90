"""GPU parity: fq_gemm / fq_gemm_debug_partials against the CPU oracle.

INT32 block products must match bit for bit.  FP32 outputs must be within
1e-3 (max |diff| / max |ref|); because the kernel keeps Alg. 1's accumulation
order they are in fact expected to be identical, which is asserted too.
bf16 outputs may differ by one bf16 ulp only where the fp32 values differ."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from oracle import fqo
from paper_2503_08040_amd import synth
from tests import gpu_util as gu

F32 = np.float32
TOL = 1e-3


def _quant_pair(a_bits, b_bits, crit, theta):
    ga = fq.fq_quantize(gu.to_device_bf16(a_bits), crit, theta, want_transposed=True)
    gb = fq.fq_quantize(gu.to_device_bf16(b_bits), fq.FQ_CRIT_NONE, 0.0, want_transposed=True)
    oa = fqo.quantize(a_bits, 128, crit, theta)
    ob = fqo.quantize(b_bits, 128, fqo.CRIT_NONE, 0.0)
    return ga, gb, oa, ob


def _check_gemm(op, ga, gb, oa, ob, label, partials=True, exact_ref=None):
    Mo, No = fqo.out_shape(op, oa, ob)
    nkb = -(-(oa.rows if op == fqo.OP_TN else oa.cols) // 128)
    if partials:
        for kb in range(nkb):
            for res in (False, True):
                gu.announce(f"{label}: partials op={op} kb={kb} res={res}")
                gp = fq.fq_gemm_debug_partials(op, ga, gb, kb, res).cpu().numpy()
                op_ = fqo.gemm_partials(op, oa, ob, kb, res)
                assert np.array_equal(gp, op_), f"{label}: INT32 partials kb={kb} res={res}"
    gu.announce(f"{label}: gemm op={op} fp32")
    ref, refb = fqo.gemm(op, oa, ob, want_bf16=True)
    c = fq.fq_gemm(op, ga, gb).cpu().numpy()
    assert c.shape == (Mo, No)
    err = gu.rel_err(c, ref)
    assert err <= TOL, f"{label}: rel err {err}"
    assert np.array_equal(c, ref), f"{label}: fp32 output not bit-identical (rel err {err})"
    gu.announce(f"{label}: gemm op={op} bf16")
    cb = fq.fq_gemm(op, ga, gb, out_dtype=torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(cb, refb), f"{label}: bf16 output differs"
    if exact_ref is not None:
        e64 = gu.rel_err(c, exact_ref)
        print(f"{label}: error vs exact fp64 GEMM {e64:.3e}", flush=True)
        assert e64 < 0.1     # accuracy of the method itself (INT8 blocks), informational
    return c


def test_config1_forward():
    wl = synth.config1()
    ga, gb, oa, ob = _quant_pair(wl.X, wl.W, fq.FQ_CRIT_ABSMAX_GT, wl.theta)
    exact = synth.bf16_bits_to_f32(wl.X).astype(np.float64) @ synth.bf16_bits_to_f32(wl.W).astype(np.float64).T
    c = _check_gemm(fq.FQ_OP_NT, ga, gb, oa, ob, "cfg1", exact_ref=exact)
    # fallback visibly helps: the plain block-INT8 product is farther from the exact one
    gn = fq.fq_quantize(gu.to_device_bf16(wl.X), fq.FQ_CRIT_NONE, 0.0)
    cn = fq.fq_gemm(fq.FQ_OP_NT, gn, gb).cpu().numpy()
    on = fqo.quantize(wl.X, 128, fqo.CRIT_NONE, 0.0)
    assert np.array_equal(cn, fqo.gemm(fqo.OP_NT, on, ob))
    rows = slice(128, 256)
    assert np.abs(cn[rows] - exact[rows]).mean() > 3 * np.abs(c[rows] - exact[rows]).mean()


def test_config1_full_fallback_and_none():
    wl = synth.config1()
    for crit in (fq.FQ_CRIT_ALL, fq.FQ_CRIT_NONE):
        ga, gb, oa, ob = _quant_pair(wl.X, wl.W, crit, 0.0)
        _check_gemm(fq.FQ_OP_NT, ga, gb, oa, ob, f"cfg1 crit={crit}", partials=False)


def test_config4_backward():
    wl = synth.config4()
    dy, w, x = wl.dY, wl.W, wl.X
    f64 = lambda b: synth.bf16_bits_to_f32(b).astype(np.float64)
    ga, gb, oa, ob = _quant_pair(dy, w, fq.FQ_CRIT_ABSMAX_GT, wl.theta)
    assert int(oa.fb_count[0]) == 2
    _check_gemm(fq.FQ_OP_NN, ga, gb, oa, ob, "cfg4 dX", exact_ref=f64(dy) @ f64(w))
    ga, gx, oa, ox = _quant_pair(dy, x, fq.FQ_CRIT_ABSMAX_GT, wl.theta)
    _check_gemm(fq.FQ_OP_TN, ga, gx, oa, ox, "cfg4 dW", exact_ref=f64(dy).T @ f64(x))


@pytest.mark.parametrize("op,sa,sb", [
    (fq.FQ_OP_NT, (130, 200), (77, 200)),
    (fq.FQ_OP_NT, (300, 513), (260, 513)),
    (fq.FQ_OP_NT, (1, 1), (1, 1)),
    (fq.FQ_OP_NN, (130, 200), (200, 77)),
    (fq.FQ_OP_NN, (257, 384), (384, 300)),
    (fq.FQ_OP_TN, (200, 130), (200, 77)),
    (fq.FQ_OP_TN, (384, 257), (384, 300)),
    (fq.FQ_OP_NT, (640, 384), (768, 384)),
])
def test_ragged_and_multi_tile_shapes(op, sa, sb):
    rng = np.random.default_rng(sa[0] + 7 * sb[1] + op)
    a = rng.standard_normal(sa).astype(F32)
    for _ in range(4):
        a[rng.integers(sa[0]), rng.integers(sa[1])] *= 120.0
    b = rng.standard_normal(sb).astype(F32) * F32(0.02)
    ga, gb, oa, ob = _quant_pair(synth.to_bf16_bits(a), synth.to_bf16_bits(b),
                                 fq.FQ_CRIT_ABSMAX_GT, 8.0)
    _check_gemm(op, ga, gb, oa, ob, f"ragged op={op} {sa}x{sb}", partials=(sa[0] <= 300))


LARGE, T128x64, T128x128 = fq.FQ_TILES_256x256, fq.FQ_TILES_128x64, fq.FQ_TILES_128x128


@pytest.mark.parametrize("op,sa,sb,cus,kind", [
    (fq.FQ_OP_NT, (250, 300), (1661, 300), 2, LARGE),      # 128x384 tiles with one valid block column
    (fq.FQ_OP_NT, (250, 300), (1833, 300), 3, LARGE),      # three valid block columns
    (fq.FQ_OP_NT, (129, 260), (1589, 260), 4, LARGE),      # two columns of 128x384 tiles, the last ragged
    (fq.FQ_OP_NN, (250, 200), (200, 1661), 4, LARGE),
    (fq.FQ_OP_TN, (200, 450), (200, 1225), 4, LARGE),
    (fq.FQ_OP_NT, (129, 128), (1600, 128), 2, LARGE),      # one k-block, ragged rows and columns
    # the same kinds of edges where smaller tiles are the faster ones
    (fq.FQ_OP_NT, (700, 300), (1100, 300), 6, T128x128),
    (fq.FQ_OP_NT, (700, 300), (1100, 300), 10, T128x128),
    (fq.FQ_OP_NT, (300, 260), (1300, 260), 7, T128x64),
    (fq.FQ_OP_NN, (300, 200), (200, 1300), 7, T128x64),
    (fq.FQ_OP_TN, (200, 700), (200, 1100), 10, T128x128),
    (fq.FQ_OP_NT, (129, 128), (1281, 128), 5, T128x64),
])
def test_mixed_tile_geometries(op, sa, sb, cus, kind, monkeypatch):
    """The large tiles' second geometry (128 x 384 tiles for the last block columns), and the smaller
    tiles that take its place, forced on small problems by telling the planner the GPU has only a few
    compute units."""
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    rng = np.random.default_rng(sa[0] + 3 * sb[1] + op + cus)
    a = rng.standard_normal(sa).astype(F32)
    for _ in range(12):
        a[rng.integers(sa[0]), rng.integers(sa[1])] *= 120.0
    b = rng.standard_normal(sb).astype(F32) * F32(0.02)
    ga, gb, oa, ob = _quant_pair(synth.to_bf16_bits(a), synth.to_bf16_bits(b),
                                 fq.FQ_CRIT_ABSMAX_GT, 8.0)
    Mo, No = fqo.out_shape(op, oa, ob)
    path = fq.fq_gemm_path(Mo, No)
    assert path[0] == kind, f"path {path}"
    assert kind != LARGE or (path[1] > 0 and path[2] > 0), f"path {path} does not use both geometries"
    assert fq.fq_gemm_form(Mo, No, sa[0] if op == fq.FQ_OP_TN else sa[1])[0] == kind, "another kernel's tiles of that size"
    assert int(oa.fb_count[0]) > 0
    c = _check_gemm(op, ga, gb, oa, ob, f"mixed op={op} {sa}x{sb} cus={cus} path={path}", partials=False)
    # the tiles do not change a single bit of the result
    monkeypatch.setenv("FQ_GEMM_CUS", "1000000")
    assert fq.fq_gemm_path(Mo, No)[0] == fq.FQ_TILES_32x32
    assert np.array_equal(fq.fq_gemm(op, ga, gb).cpu().numpy(), c)


@pytest.mark.parametrize("cols,cus,kind", [(384, 256, fq.FQ_TILES_32x32), (512, 1, LARGE), (384, 3, T128x128)])
def test_scale_products_in_the_subnormal_range(cols, cus, kind, monkeypatch):
    """A and B blocks so small that a^A * a^B is subnormal or underflows to zero: the product of
    the scales, the FMA with it and the accumulator must behave as IEEE binary32 without
    flush-to-zero on both sides."""
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    assert fq.fq_gemm_path(256, cols)[0] == fq.fq_gemm_form(256, cols, 512)[0] == kind
    rng = np.random.default_rng(44)
    a = rng.standard_normal((256, 512))
    for bk, k in enumerate((-126, -118, -110, -104)):
        a[:, bk * 128:(bk + 1) * 128] *= 2.0 ** k
    a[5, 3] = 50.0 * 2.0 ** -126                      # an outlier among tiny values
    b = rng.standard_normal((cols, 512)) * 2.0 ** -24
    b[:128] *= 2.0 ** -20
    with np.errstate(under="ignore"):
        ab, bb = synth.to_bf16_bits(a.astype(F32)), synth.to_bf16_bits(b.astype(F32))
    ga, gb, oa, ob = _quant_pair(ab, bb, fq.FQ_CRIT_ALL, 0.0)
    c = _check_gemm(fq.FQ_OP_NT, ga, gb, oa, ob, "tiny scales", partials=False)
    assert np.isfinite(c).all()
    sub = (c != 0) & (np.abs(c) < 2.0 ** -126)
    assert sub.mean() > 0.1                            # subnormal outputs were produced and kept


def test_strided_output_and_reuse():
    wl = synth.config1()
    ga, gb, oa, ob = _quant_pair(wl.X, wl.W, fq.FQ_CRIT_ABSMAX_GT, wl.theta)
    ref = fqo.gemm(fqo.OP_NT, oa, ob)
    big = torch.full((256, 600), 7.0, device="cuda")
    gu.announce("gemm into a strided output view")
    fq.fq_gemm(fq.FQ_OP_NT, ga, gb, out=big[:, 40:552])
    out = big.cpu().numpy()
    assert np.array_equal(out[:, 40:552], ref)
    assert np.all(out[:, :40] == 7.0) and np.all(out[:, 552:] == 7.0)
    gu.announce("gemm twice: deterministic")
    c1 = fq.fq_gemm(fq.FQ_OP_NT, ga, gb)
    c2 = fq.fq_gemm(fq.FQ_OP_NT, ga, gb)
    assert torch.equal(c1, c2)


@pytest.mark.parametrize("cus,kind", [(256, fq.FQ_TILES_32x32), (3, T128x64), (2, T128x128), (1, LARGE)])
def test_empty_contraction_and_empty_output(cus, kind, monkeypatch):
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    assert fq.fq_gemm_path(256, 256)[0] == fq.fq_gemm_form(256, 256, 0, falls_back=False)[0] == kind
    a = fq.fq_quantize(torch.empty((256, 0), dtype=torch.bfloat16, device="cuda"),
                       fq.FQ_CRIT_NONE, 0.0, capacity=0)
    b = fq.fq_quantize(torch.empty((256, 0), dtype=torch.bfloat16, device="cuda"),
                       fq.FQ_CRIT_NONE, 0.0, capacity=0)
    gu.announce("gemm with K = 0")
    c = fq.fq_gemm(fq.FQ_OP_NT, a, b, out=torch.full((256, 256), 3.0, device="cuda"))
    assert torch.count_nonzero(c).item() == 0
    a0 = fq.fq_quantize(torch.empty((0, 256), dtype=torch.bfloat16, device="cuda"),
                        fq.FQ_CRIT_NONE, 0.0, capacity=0)
    b0 = fq.fq_quantize(torch.zeros((128, 256), dtype=torch.bfloat16, device="cuda"),
                        fq.FQ_CRIT_NONE, 0.0, capacity=0)
    gu.announce("gemm with M = 0")
    assert fq.fq_gemm(fq.FQ_OP_NT, a0, b0).shape == (0, 128)


def test_capacity_overflow_poisons_output():
    wl = synth.config1()
    x = gu.to_device_bf16(wl.X)
    gb = fq.fq_quantize(gu.to_device_bf16(wl.W), fq.FQ_CRIT_NONE, 0.0)
    ga = fq.fq_quantize(x, fq.FQ_CRIT_ALL, 0.0, capacity=3)
    gu.announce("gemm on a tensor whose residual slots overflowed")
    c = fq.fq_gemm(fq.FQ_OP_NT, ga, gb)
    assert torch.isnan(c).any().item()      # never a silently wrong product


@pytest.mark.parametrize("shape_a,shape_b,cus,kind,tail", [
    ((500, 384), (1281, 384), 4, LARGE, False),         # 256x256 tiles only
    ((450, 300), (1225, 300), 4, LARGE, True),          # 128x384 tiles beside them
    ((600, 384), (300, 384), 0, fq.FQ_TILES_32x32, False),
    ((700, 300), (1100, 300), 6, T128x128, False),
])
def test_capacity_overflow_poisons_exactly_the_affected_block_rows(shape_a, shape_b, cus, kind, tail, monkeypatch):
    """Every block is flagged but only some get a residual slot: the rows of an i-block that has
    a flagged block without a slot are NaN, all other rows are the complete result."""
    if cus:
        monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    rng = np.random.default_rng(shape_a[0])
    a_bits = synth.to_bf16_bits(rng.standard_normal(shape_a).astype(F32))
    b_bits = synth.to_bf16_bits(rng.standard_normal(shape_b).astype(F32) * F32(0.02))
    nbr, nbc = -(-shape_a[0] // 128), -(-shape_a[1] // 128)
    ga = fq.fq_quantize(gu.to_device_bf16(a_bits), fq.FQ_CRIT_ALL, 0.0, capacity=(nbr * nbc) // 2)
    gb = fq.fq_quantize(gu.to_device_bf16(b_bits), fq.FQ_CRIT_NONE, 0.0)
    with pytest.raises(fq.FqError):
        fq.fq_qtensor_check(ga)
    slot = ga.view("fb_slot").cpu().numpy()
    assert (slot == -2).sum() == nbr * nbc - (nbr * nbc) // 2
    bad = (slot == -2).any(axis=1)
    assert bad.any()
    path = fq.fq_gemm_path(shape_a[0], shape_b[0])
    assert path[0] == fq.fq_gemm_form(shape_a[0], shape_b[0], shape_a[1])[0] == kind and (path[2] > 0) == tail
    gu.announce(f"gemm with overflowed residual slots, path {path}")
    c = fq.fq_gemm(fq.FQ_OP_NT, ga, gb).cpu().numpy()
    ref = fqo.gemm(fqo.OP_NT, fqo.quantize(a_bits, 128, fqo.CRIT_ALL, 0.0),
                   fqo.quantize(b_bits, 128, fqo.CRIT_NONE, 0.0))
    for bi in range(nbr):
        rows = slice(bi * 128, min((bi + 1) * 128, shape_a[0]))
        if bad[bi]:
            assert np.isnan(c[rows]).all(), f"block row {bi} should be poisoned"
        else:
            assert np.array_equal(c[rows], ref[rows]), f"block row {bi} should be complete"


def _sampled_windows(rng, Mo, No, flagged_rows, n=24, h=4, w=8):
    wins = []
    rows = list(flagged_rows[:n // 2]) + list(rng.integers(0, Mo - h, size=n - len(flagged_rows[:n // 2])))
    for r in rows:
        r = int(min(max(r, 0), Mo - h))
        c = int(rng.integers(0, No - w))
        wins.append((r, r + h, c, c + w))
    wins.append((Mo - h, Mo, No - w, No))
    wins.append((0, h, 0, w))
    return wins


def _tile_windows(rng, Mo, No, flagged_block_rows, n=64):
    """At least n whole 128 x 128 output tiles: one in every block-row that holds a flagged A
    block (random tile column), the four corner tiles, and random ones up to n."""
    nbi, nbj = -(-Mo // 128), -(-No // 128)
    tiles = {(int(bi), int(rng.integers(0, nbj))) for bi in flagged_block_rows}
    tiles |= {(0, 0), (0, nbj - 1), (nbi - 1, 0), (nbi - 1, nbj - 1)}
    while len(tiles) < min(n, nbi * nbj):
        tiles.add((int(rng.integers(0, nbi)), int(rng.integers(0, nbj))))
    return [(bi * 128, min(bi * 128 + 128, Mo), bj * 128, min(bj * 128 + 128, No))
            for bi, bj in sorted(tiles)]


@pytest.mark.parametrize("cfg", ["cfg2", "cfg3", "cfg5_random", "cfg5_sequential"])
def test_full_size(cfg, monkeypatch):
    """Workload configs 2, 3 and 5 at full size, in the launch configuration the benchmark
    times: quantizer outputs bit-exact in full; GEMM outputs against the oracle on the whole
    output for config 2 and, for configs 3 and 5, on at least 64 whole 128 x 128 tiles that
    include one in every block-row holding a flagged block, the corner tiles and random ones."""
    wl = {"cfg2": lambda: synth.config2(), "cfg3": lambda: synth.config3(),
          "cfg5_random": lambda: synth.config5(frac=0.05, placement="random"),
          "cfg5_sequential": lambda: synth.config5(frac=0.05, placement="sequential")}[cfg]()
    gu.announce(f"{cfg}: quantize X {wl.X.shape} / W {wl.W.shape}")
    ga = fq.fq_quantize(gu.to_device_bf16(wl.X), fq.FQ_CRIT_ABSMAX_GT, wl.theta)
    gb = fq.fq_quantize(gu.to_device_bf16(wl.W), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    oa = fqo.quantize(wl.X, 128, fqo.CRIT_ABSMAX_GT, wl.theta)
    ob = fqo.quantize(wl.W, 128, fqo.CRIT_NONE, 0.0)
    assert np.array_equal(oa.fb_list[:oa.fb_count[0]], wl.flagged_blocks)
    gu.compare_quantized(ga, oa, f"{cfg} X")
    gu.compare_quantized(gb, ob, f"{cfg} W")
    gu.announce(f"{cfg}: gemm")
    c = fq.fq_gemm(fq.FQ_OP_NT, ga, gb, out_dtype=torch.bfloat16)
    c32 = fq.fq_gemm(fq.FQ_OP_NT, ga, gb)
    torch.cuda.synchronize()
    rng = np.random.default_rng(0)
    if cfg == "cfg2":
        windows = [(0, wl.M, 0, wl.N)]
    else:
        windows = _tile_windows(rng, wl.M, wl.N, sorted({int(b) // oa.nbc for b in wl.flagged_blocks}))
        assert len(windows) >= 64
    gu.announce(f"{cfg}: oracle on {len(windows)} window(s)")
    worst = 0.0
    for (i0, i1, j0, j1) in windows:
        ref, refb = fqo.gemm_window(fqo.OP_NT, oa, ob, (i0, i1, j0, j1), want_bf16=True)
        got = c32[i0:i1, j0:j1].cpu().numpy()
        worst = max(worst, gu.rel_err(got, ref[:, j0:j1]))
        assert np.array_equal(got, ref[:, j0:j1]), f"{cfg}: window {(i0, i1, j0, j1)}"
        gotb = c[i0:i1, j0:j1].contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
        assert np.array_equal(gotb, refb[:, j0:j1])
        del ref, refb
    assert worst <= TOL
    # properties that hold at any size: finite everywhere, bf16 output is the rounding of fp32,
    # and the result does not depend on the tiles (config 2 on 256 compute units uses both
    # large tile geometries; 256 x 256 tiles alone and 32 x 32 tiles must give the same bits)
    assert torch.isfinite(c32).all().item()
    assert torch.equal(c, c32.to(torch.bfloat16))
    path = fq.fq_gemm_path(wl.M, wl.N)
    print(f"{cfg}: tiles {path}", flush=True)
    assert path[0] == LARGE and (path[2] > 0) == (cfg == "cfg2")
    single = -(-wl.M // 256) * -(-wl.N // 256)
    for cus, want in ((single, (LARGE, single, 0, 0)),
                      (1000000, (fq.FQ_TILES_32x32, -(-wl.M // 32) * -(-wl.N // 32), 0, 0))):
        monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
        assert fq.fq_gemm_path(wl.M, wl.N) == want
        gu.announce(f"{cfg}: gemm with a single tile geometry {want}")
        assert torch.equal(fq.fq_gemm(fq.FQ_OP_NT, ga, gb), c32)


@pytest.mark.parametrize("variant", ["stochastic", "fallback"])
def test_full_size_backward_sampled(variant):
    """Config 2's backward at full size, as the benchmark's backward mode launches it:
    dX = dY W (NN) and dW = dY^T X (TN) through the transposed copies the quantizer emits.
    "stochastic": the paper's recipe (Sec. 5.1, 5.3), Q_s(dY) and the Q_s(X) context without
    fallback; "fallback": config 4's recipe at this size, dY quantized to nearest with about
    5 % of its blocks flagged, so that both products take residual blocks from the
    transposed and the plain residual storage.  Quantizer outputs are compared in full, GEMM
    outputs on sampled windows the oracle computes element by element."""
    wl = synth.config2()
    M, K, N = wl.M, wl.K, wl.N
    rng = np.random.default_rng(21)
    dy = (rng.standard_t(3.0, size=(M, N)) * 1e-3).astype(F32)
    dy_bits = synth.to_bf16_bits(dy)
    gu.announce(f"backward/{variant}: quantize dY {dy.shape}, W, X")
    if variant == "stochastic":
        gdy = fq.fq_quantize_sr(gu.to_device_bf16(dy_bits), 7, want_transposed=True)
        ody = fqo.quantize_sr(dy_bits, 128, 7)
        gx = fq.fq_quantize_sr(gu.to_device_bf16(wl.X), 5, want_transposed=True)
        ox = fqo.quantize_sr(wl.X, 128, 5)
        flagged = np.zeros(0, np.int64)
    else:
        amax = np.abs(synth.bf16_bits_to_f32(dy_bits)).reshape(M // 128, 128, N // 128, 128).max(axis=(1, 3))
        srt = np.sort(amax.ravel())
        cut = int(0.95 * srt.size)
        theta = float(0.5 * (srt[cut - 1] + srt[cut]))
        gdy = fq.fq_quantize(gu.to_device_bf16(dy_bits), fq.FQ_CRIT_ABSMAX_GT, theta, want_transposed=True)
        ody = fqo.quantize(dy_bits, 128, fqo.CRIT_ABSMAX_GT, theta)
        gx = fq.fq_quantize(gu.to_device_bf16(wl.X), fq.FQ_CRIT_NONE, 0.0, want_transposed=True)
        ox = fqo.quantize(wl.X, 128, fqo.CRIT_NONE, 0.0)
        flagged = ody.fb_list[:ody.fb_count[0]].astype(np.int64)
        assert 0.03 * amax.size < flagged.size < 0.07 * amax.size
    gw = fq.fq_quantize(gu.to_device_bf16(wl.W), fq.FQ_CRIT_NONE, 0.0, want_transposed=True)
    ow = fqo.quantize(wl.W, 128, fqo.CRIT_NONE, 0.0)
    gu.compare_quantized(gdy, ody, f"backward/{variant} dY")
    gu.compare_quantized(gx, ox, f"backward/{variant} X")
    nbc = ody.nbc
    for op, gb, ob, name in ((fq.FQ_OP_NN, gw, ow, "dX"), (fq.FQ_OP_TN, gx, ox, "dW")):
        Mo, No = fqo.out_shape(op, ody, ob)
        assert (Mo, No) == ((M, K) if op == fq.FQ_OP_NN else (N, K))
        gu.announce(f"backward/{variant}: gemm {name} {Mo}x{No}")
        c32 = fq.fq_gemm(op, gdy, gb)
        cb = fq.fq_gemm(op, gdy, gb, out_dtype=torch.bfloat16)
        torch.cuda.synchronize()
        # output rows that meet a flagged dY block: its rows for dX, its columns for dW
        frows = sorted({((int(b) // nbc) if op == fq.FQ_OP_NN else (int(b) % nbc)) * 128
                        + int(rng.integers(0, 124)) for b in flagged})
        rng.shuffle(frows)
        for (i0, i1, j0, j1) in _sampled_windows(rng, Mo, No, frows):
            ref, refb = fqo.gemm(op, ody, ob, window=(i0, i1, j0, j1), want_bf16=True)
            got = c32[i0:i1, j0:j1].cpu().numpy()
            assert gu.rel_err(got, ref[i0:i1, j0:j1]) <= TOL
            assert np.array_equal(got, ref[i0:i1, j0:j1]), f"{name}: window {(i0, i1, j0, j1)}"
            gotb = cb[i0:i1, j0:j1].contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
            assert np.array_equal(gotb, refb[i0:i1, j0:j1]), f"{name}: bf16 window {(i0, i1, j0, j1)}"
        assert torch.isfinite(c32).all().item()
        assert torch.equal(cb, c32.to(torch.bfloat16))
        del c32, cb
