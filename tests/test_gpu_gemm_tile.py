"""GPU parity of fq_gemm's smaller tiles (32 x 32, 128 x 64, 128 x 128, without loading wavefronts) against the CPU
oracle, bit for bit: they keep Alg. 1's order of the terms, so no tolerance is needed.  FQ_GEMM_CUS, the number of
compute units the planner assumes, steers a small problem to the tile that a larger one would get; fq_gemm_form says
that it did, as tiles of the same size with loading wavefronts would give the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from oracle import fqo
from paper_2503_08040_amd import synth
from tests import gpu_util as gu
from tests.test_gpu_gemm import _quant_pair

F32 = np.float32
NT, NN, TN = fq.FQ_OP_NT, fq.FQ_OP_NN, fq.FQ_OP_TN
# (rows, columns of the output, compute units assumed) and the tile they lead to
TILES = {"32x32": (65, 33, 256), "32x32 one row": (1, 300, 256), "128x64": (300, 260, 6),
         "128x64 odd": (253, 301, 4), "128x128": (300, 370, 5), "128x128 odd": (200, 371, 3),
         "256x256 and 128x384": (700, 1400, 7)}
FORM = {"32x32": fq.FQ_FORM_32x32, "128x64": fq.FQ_FORM_128x64, "128x128": fq.FQ_FORM_128x128,
        "256x256": fq.FQ_FORM_256x256}


def _assert_form(tile, K):
    Mo, No = TILES[tile][:2]
    assert fq.fq_gemm_form(Mo, No, K)[0] == FORM[tile.split()[0]]
    path = fq.fq_gemm_path(Mo, No)
    assert (path[2] + path[3] > 0) == ("128x384" in tile), path


def _operands(op, Mo, No, K, seed, spikes):
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((K, Mo) if op == TN else (Mo, K)).astype(F32)
    for _ in range(spikes):
        a[rng.integers(a.shape[0]), rng.integers(a.shape[1])] *= 120.0
    b = rng.standard_normal((No, K) if op == NT else (K, No)).astype(F32) * F32(0.02)
    return synth.to_bf16_bits(a), synth.to_bf16_bits(b)


# contraction lengths: one k-block, a part of one, an odd and an even number of them, and more than
# the 64 whose scales a wavefront holds at a time
@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("op,K,spikes", [(NT, 128, 0), (NT, 77, 2), (NN, 384, 5), (TN, 640, 6), (NT, 520, 400),
                                         (NT, 8400, 30)])
def test_tiles_match_the_oracle(tile, op, K, spikes, monkeypatch):
    Mo, No, cus = TILES[tile]
    if K > 1000 and Mo * No > 200 * 400:
        K = 1300                    # the oracle's time; eleven k-blocks are enough where the others have had 66
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    _assert_form(tile, K)
    a, b = _operands(op, Mo, No, K, K + Mo + op, spikes)
    ga, gb, oa, ob = _quant_pair(a, b, fq.FQ_CRIT_ABSMAX_GT, 12.0)
    gu.announce(f"tile {tile} op={op} {Mo}x{No} K={K} flagged {int(oa.fb_count[0])}")
    ref, refb = fqo.gemm(op, oa, ob, want_bf16=True)
    assert np.array_equal(fq.fq_gemm(op, ga, gb).cpu().numpy(), ref)
    got = fq.fq_gemm(op, ga, gb, out_dtype=torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, refb)
    # a padded row pitch: 16-byte stores, and nothing written beside the output
    wide = torch.full((Mo, (No + 7) // 8 * 8 + 8), 5.0, device="cuda")
    fq.fq_gemm(op, ga, gb, out=wide[:, :No])
    assert np.array_equal(wide[:, :No].cpu().numpy(), ref)
    assert (wide[:, No:] == 5.0).all().item()


# contractions of four k-blocks, and of 66 with the block in the second 64 of them
@pytest.mark.parametrize("tile,K", [("32x32", 512), ("128x64", 512), ("128x128", 512), ("128x64 odd", 8448),
                                    ("128x128 odd", 8448)])
def test_blocks_without_a_slot_poison_their_rows(tile, K, monkeypatch):
    Mo, No, cus = TILES[tile]
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    _assert_form(tile, K)
    a, b = _operands(NT, Mo, No, K, 3, 0)
    nbr = -(-Mo // 128)
    crit, theta, capacity = fq.FQ_CRIT_ALL, 0.0, nbr * 4 - 1
    if K > 512:
        crit, theta, capacity = fq.FQ_CRIT_ABSMAX_GT, 12.0, nbr - 1
        a[::128, 65 * 128 + 3] = 0x4300                     # one flagged block per block row, one slot too few
    ga = fq.fq_quantize(gu.to_device_bf16(a), crit, theta, capacity=capacity)
    gb = fq.fq_quantize(gu.to_device_bf16(b), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    bad = (ga.view("fb_slot").cpu().numpy() == -2).any(axis=1)
    assert bad.sum() == 1
    gu.announce(f"tile {tile}: one block without a residual slot")
    c = fq.fq_gemm(NT, ga, gb).cpu().numpy()
    ref = fqo.gemm(fqo.OP_NT, fqo.quantize(a, 128, crit, theta), fqo.quantize(b, 128, fqo.CRIT_NONE, 0.0))
    for bi in range(nbr):
        rows = slice(bi * 128, min(bi * 128 + 128, Mo))
        assert np.isnan(c[rows]).all() if bad[bi] else np.array_equal(c[rows], ref[rows])
