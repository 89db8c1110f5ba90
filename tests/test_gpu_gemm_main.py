"""GPU parity of the large tiles for an A operand without fallback (the kernel that has no residual items) against the
CPU oracle, bit for bit, in both geometries, and against the kernel with residual items on the same codes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from oracle import fqo
from tests import gpu_util as gu
from tests.test_gpu_gemm_tile import NN, NT, TN, _operands

# (rows, columns, compute units assumed): one 256 x 256 tile, ragged; 128 x 384 tiles over the last block columns,
# and over the last block rows
TILES = {"one": (250, 256, 1), "column tail": (129, 1589, 4), "row tail": (1275, 253, 2)}


# contraction lengths: one and two k-blocks (the prologue alone), odd, and around the 64 whose scales are held at a time
@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("op,K", [(NT, 100), (NN, 256), (TN, 384), (NT, 8192), (NN, 8300), (TN, 16500)])
def test_large_tiles_without_fallback(tile, op, K, monkeypatch):
    Mo, No, cus = TILES[tile]
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    path = fq.fq_gemm_path(Mo, No)
    assert path[0] == fq.FQ_TILES_256x256 and (path[2] > 0, path[3] > 0) == ("column" in tile, "row" in tile), path
    a, b = _operands(op, Mo, No, K, K + Mo + op, 4)
    at, bt = op == TN, op in (NN, TN)
    ga = fq.fq_quantize(gu.to_device_bf16(a), fq.FQ_CRIT_NONE, 0.0, capacity=0, want_transposed=at)
    gb = fq.fq_quantize(gu.to_device_bf16(b), fq.FQ_CRIT_NONE, 0.0, capacity=0, want_transposed=bt)
    gu.announce(f"large tiles without fallback, {tile} op={op} {Mo}x{No} K={K}")
    ref, refb = fqo.gemm(op, fqo.quantize(a, 128, fqo.CRIT_NONE, 0.0), fqo.quantize(b, 128, fqo.CRIT_NONE, 0.0),
                         want_bf16=True)
    c = fq.fq_gemm(op, ga, gb)
    assert np.array_equal(c.cpu().numpy(), ref)
    got = fq.fq_gemm(op, ga, gb, out_dtype=torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, refb)
    # the same codes with residual slots that nobody uses: the other kernel
    gf = fq.fq_quantize(gu.to_device_bf16(a), fq.FQ_CRIT_ABSMAX_GT, float("inf"), want_transposed=at)
    assert torch.equal(fq.fq_gemm(op, gf, gb), c)


# which of the tile's two block rows are flagged at each of nine k-blocks (1, 2, 3: upper, lower, both)
PATTERNS = {"first": "300000000", "last": "000000003", "last upper": "000000001", "halves in turn": "121212121",
            "same half in a row": "111022200", "all": "333333333", "mixed": "013231203"}


@pytest.mark.parametrize("pattern", list(PATTERNS))
def test_patterns_of_flagged_blocks(pattern, monkeypatch):
    """Residual products of a 256 x 256 tile: the turns of its two halves, the blocks they share in LDS."""
    monkeypatch.setenv("FQ_GEMM_CUS", "1")
    assert fq.fq_gemm_path(250, 256) == (fq.FQ_TILES_256x256, 1, 0, 0) == fq.fq_gemm_path(250, 256, biased=True)
    bits = PATTERNS[pattern]
    K = 128 * len(bits)
    a, b = _operands(NT, 250, 256, K, 17, 0)
    for k, p in enumerate(bits):
        for half in range(2):
            if int(p) >> half & 1:
                a[128 * half + 7 * k, 128 * k + 5] = 0x4300 + k           # 128 and more
    ga = fq.fq_quantize(gu.to_device_bf16(a), fq.FQ_CRIT_ABSMAX_GT, 12.0)
    gb = fq.fq_quantize(gu.to_device_bf16(b), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    oa, ob = fqo.quantize(a, 128, fqo.CRIT_ABSMAX_GT, 12.0), fqo.quantize(b, 128, fqo.CRIT_NONE, 0.0)
    assert int(oa.fb_count[0]) == sum(bin(int(p)).count("1") for p in bits)
    gu.announce(f"flagged blocks: {pattern}")
    ref = fqo.gemm(NT, oa, ob)
    for _ in range(3):
        assert np.array_equal(fq.fq_gemm(NT, ga, gb).cpu().numpy(), ref)
    assert np.abs(fq.fq_gemm_biased(NT, ga, gb).cpu().numpy() - ref).max() <= 1e-3 * np.abs(ref).max()


# outputs on which only an A without residual slots takes 256 x 256 tiles, in one round and with 128 x 384 tails
@pytest.mark.parametrize("M,N", [(1280, 9700), (4096, 5760), (1400, 8001)])
def test_planner_line_depends_on_slots(M, N):
    assert fq.fq_gemm_form(M, N, 300)[0] != fq.FQ_FORM_256x256
    assert fq.fq_gemm_form(M, N, 300, falls_back=False)[0] == fq.FQ_FORM_256x256
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    x = torch.randn(M, 300, device="cuda", generator=g).bfloat16()
    b = fq.fq_quantize(torch.randn(N, 300, device="cuda", generator=g).bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    slots = fq.fq_quantize(x, fq.FQ_CRIT_ABSMAX_GT, float("inf"))
    none = fq.fq_quantize(x, fq.FQ_CRIT_NONE, 0.0, capacity=0)
    gu.announce(f"planner line {M}x{N}")
    for dt in (torch.float32, torch.bfloat16):
        assert torch.equal(fq.fq_gemm(NT, slots, b, out_dtype=dt), fq.fq_gemm(NT, none, b, out_dtype=dt))
