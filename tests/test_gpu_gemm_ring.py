"""GPU parity of fq_gemm's tiles with loading wavefronts (one round of 128 x 64, 128 x 128 or 128 x 256 tiles) against
the CPU oracle, bit for bit.  FQ_GEMM_CUS, the number of compute units the planner assumes, steers a small problem to
them: they are chosen where the output is at most two, one and one of these tiles per compute unit and the contraction is
not short; fq_gemm_form says that they were."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from oracle import fqo
from tests import gpu_util as gu
from tests.test_gpu_gemm import _quant_pair
from tests.test_gpu_gemm_tile import NN, NT, TN, _operands

# (rows, columns of the output, compute units assumed): ragged rows and columns, an odd number of block
# columns under 128 x 256 tiles, fewer rows than a tile has
TILES = {"128x64": (129, 301, 5), "128x64 few rows": (97, 301, 5), "128x128": (300, 370, 9), "128x256": (250, 500, 4),
         "128x256 odd": (129, 600, 6)}


FORM = {"128x64": fq.FQ_FORM_LOADERS_128x64, "128x128": fq.FQ_FORM_LOADERS_128x128, "128x256": fq.FQ_FORM_LOADERS_128x256}


def _tiles(tile, K, falls_back, monkeypatch):
    Mo, No, cus = TILES[tile]
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    size = tile.split()[0]
    assert fq.fq_gemm_form(Mo, No, K, falls_back=falls_back) == \
        (FORM[size], -(-Mo // 128) * -(-No // int(size.split("x")[1])))
    return Mo, No


# contraction lengths: 16 to 22 k-blocks (all residues of the ring's three stages, with few, many and no residual items),
# around the 64 k-blocks whose flags are looked at together and the 128 whose scales and slots are in LDS; spikes flag
# few or nearly all blocks
@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("op,K,spikes", [(NT, 2040, 0), (NT, 2048, 3), (NN, 2100, 5), (TN, 2304, 0), (NT, 2500, 1600),
                                         (TN, 2700, 6), (NT, 8192, 30), (NN, 8300, 900), (NT, 16500, 60),
                                         (TN, 25500, 700)])
def test_ring_tiles_match_the_oracle(tile, op, K, spikes, monkeypatch):
    Mo, No = _tiles(tile, K, True, monkeypatch)
    a, b = _operands(op, Mo, No, K, K + Mo + op, spikes)
    ga, gb, oa, ob = _quant_pair(a, b, fq.FQ_CRIT_ABSMAX_GT, 12.0)
    gu.announce(f"ring {tile} op={op} {Mo}x{No} K={K} flagged {int(oa.fb_count[0])}")
    ref, refb = fqo.gemm(op, oa, ob, want_bf16=True)
    wide = torch.full((Mo, (No + 7) // 8 * 8 + 8), 5.0, device="cuda")
    fq.fq_gemm(op, ga, gb, out=wide[:, :No])
    assert np.array_equal(wide[:, :No].cpu().numpy(), ref)
    assert (wide[:, No:] == 5.0).all().item()
    got = fq.fq_gemm(op, ga, gb, out_dtype=torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, refb)


# an A that cannot fall back: from 8 k-blocks on
@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("op,K", [(NT, 1000), (NT, 1152), (NN, 1200), (TN, 1281), (NT, 8320), (TN, 16500)])
def test_ring_tiles_without_residual_slots(tile, op, K, monkeypatch):
    Mo, No = _tiles(tile, K, False, monkeypatch)
    a, b = _operands(op, Mo, No, K, K + Mo + op, 5)
    ga = fq.fq_quantize(gu.to_device_bf16(a), fq.FQ_CRIT_NONE, 0.0, capacity=0, want_transposed=True)
    gb = fq.fq_quantize(gu.to_device_bf16(b), fq.FQ_CRIT_NONE, 0.0, capacity=0, want_transposed=True)
    gu.announce(f"ring {tile} op={op} {Mo}x{No} K={K} without residual slots")
    ref = fqo.gemm(op, fqo.quantize(a, 128, fqo.CRIT_NONE, 0.0), fqo.quantize(b, 128, fqo.CRIT_NONE, 0.0))
    assert np.array_equal(fq.fq_gemm(op, ga, gb).cpu().numpy(), ref)


@pytest.mark.parametrize("tile", [t for t in TILES if TILES[t][0] > 128])
@pytest.mark.parametrize("k_block", [0, 3, 70, 130])
def test_ring_blocks_without_a_slot_poison_their_rows(tile, k_block, monkeypatch):
    K = 128 * max(k_block + 2, 16)
    Mo, No = _tiles(tile, K, True, monkeypatch)
    nbr = -(-Mo // 128)
    a, b = _operands(NT, Mo, No, K, 3, 0)
    for bi in range(nbr):
        a[bi * 128, k_block * 128 + 3] = 0x4300           # one flagged block per block row, one slot too few
    ga = fq.fq_quantize(gu.to_device_bf16(a), fq.FQ_CRIT_ABSMAX_GT, 12.0, capacity=nbr - 1)
    gb = fq.fq_quantize(gu.to_device_bf16(b), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    bad = (ga.view("fb_slot").cpu().numpy() == -2).any(axis=1)
    assert bad.sum() == 1
    gu.announce(f"ring {tile}: a block without a residual slot at k-block {k_block}")
    c = fq.fq_gemm(NT, ga, gb).cpu().numpy()
    ref = fqo.gemm(fqo.OP_NT, fqo.quantize(a, 128, fqo.CRIT_ABSMAX_GT, 12.0), fqo.quantize(b, 128, fqo.CRIT_NONE, 0.0))
    for bi in range(nbr):
        rows = slice(bi * 128, min(bi * 128 + 128, Mo))
        assert np.isnan(c[rows]).all() if bad[bi] else np.array_equal(c[rows], ref[rows])


@pytest.mark.parametrize("tile", list(TILES))
def test_ring_empty_contraction(tile, monkeypatch):
    """Of such an output: other tiles take it."""
    Mo, No = _tiles(tile, 4096, False, monkeypatch)
    assert fq.fq_gemm_form(Mo, No, 0, falls_back=False)[0] not in FORM.values()
    e = lambda n: fq.fq_quantize(torch.empty((n, 0), dtype=torch.bfloat16, device="cuda"), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    gu.announce(f"ring {tile}: K = 0")
    assert (fq.fq_gemm(NT, e(Mo), e(No), out=torch.full((Mo, No), 3.0, device="cuda")) == 0).all().item()
