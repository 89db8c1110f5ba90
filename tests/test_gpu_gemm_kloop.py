"""GPU parity of the 256 x 256 / 128 x 384 tile kernel against the CPU oracle, bit for bit, where its
scalars and its tile plan have edges: contractions around the 64 k-blocks whose scales a wavefront
holds at a time, and a tail of 128 x 384 tiles along the last block rows.  FQ_GEMM_CUS, the number of
compute units the planner assumes, leads small problems to these tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from oracle import fqo
from paper_2503_08040_amd import synth
from tests import gpu_util as gu
from tests.test_gpu_gemm import _quant_pair
from tests.test_gpu_gemm_tile import _operands

NT, NN, TN = fq.FQ_OP_NT, fq.FQ_OP_NN, fq.FQ_OP_TN


def _compare(op, Mo, No, K, spikes, tag):
    a, b = _operands(op, Mo, No, K, K + op, spikes)
    # flagged blocks on both sides of the 64th and of the 128th k-block
    for k in (0, 62, 63, 64, 65, 127, 128):
        if k * 128 + 5 < K:
            i = (k * 37) % Mo
            a[(k * 128 + 5, i) if op == TN else (i, k * 128 + 5)] = 0x4300      # 128.0
    ga, gb, oa, ob = _quant_pair(a, b, fq.FQ_CRIT_ABSMAX_GT, 12.0)
    gu.announce(f"{tag} op={op} {Mo}x{No} K={K} flagged {int(oa.fb_count[0])}")
    ref, refb = fqo.gemm(op, oa, ob, want_bf16=True)
    assert np.array_equal(fq.fq_gemm(op, ga, gb).cpu().numpy(), ref)
    got = fq.fq_gemm(op, ga, gb, out_dtype=torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, refb)
    # the tolerance variant takes the same path through scales and plan; 1e-3 is what it promises
    assert np.abs(fq.fq_gemm_biased(op, ga, gb).cpu().numpy() - ref).max() <= 1e-3 * np.abs(ref).max()


@pytest.mark.parametrize("op,K", [(NT, 128), (NT, 8192), (NT, 8300), (NN, 8191), (TN, 8400), (TN, 16500)])
def test_scales_of_64_k_blocks_at_a_time(op, K, monkeypatch):
    monkeypatch.setenv("FQ_GEMM_CUS", "1")
    assert fq.fq_gemm_path(250, 256) == (fq.FQ_TILES_256x256, 1, 0, 0) == fq.fq_gemm_path(250, 256, biased=True)
    _compare(op, 250, 256, K, 20, "one tile")


@pytest.mark.parametrize("op,K", [(NT, 300), (TN, 640), (NN, 8400)])
def test_tail_along_the_last_block_rows(op, K, monkeypatch):
    # 10 x 2 blocks on two compute units: five 256 x 256 tiles would be three rounds; four of them and
    # two 128 x 384 tiles over the last two block rows are 2.75
    monkeypatch.setenv("FQ_GEMM_CUS", "2")
    assert fq.fq_gemm_path(1275, 253) == (fq.FQ_TILES_256x256, 4, 0, 2) == fq.fq_gemm_path(1275, 253, biased=True)
    _compare(op, 1275, 253, K, 30, "row tail")


def test_block_without_a_slot_behind_the_64th(monkeypatch):
    monkeypatch.setenv("FQ_GEMM_CUS", "1")
    assert fq.fq_gemm_path(256, 200)[0] == fq.FQ_TILES_256x256
    a, b = _operands(NT, 256, 200, 66 * 128, 1, 0)
    a[200, 65 * 128 + 3] = a[10, 65 * 128 + 3] = 0x4300          # both block rows flagged at k = 65
    ga = fq.fq_quantize(gu.to_device_bf16(a), fq.FQ_CRIT_ABSMAX_GT, 12.0, capacity=1)
    gb = fq.fq_quantize(gu.to_device_bf16(b), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    slots = ga.view("fb_slot").cpu().numpy()
    bad = (slots == -2).any(axis=1)
    assert bad.sum() == 1 and (slots[:, :64] == -1).all()
    gu.announce("block without a residual slot at k-block 65")
    c = fq.fq_gemm(NT, ga, gb).cpu().numpy()
    ref = fqo.gemm(NT, fqo.quantize(a, 128, fqo.CRIT_ABSMAX_GT, 12.0), fqo.quantize(b, 128, fqo.CRIT_NONE, 0.0))
    for bi in range(2):
        rows = slice(bi * 128, bi * 128 + 128)
        assert np.isnan(c[rows]).all() if bad[bi] else np.array_equal(c[rows], ref[rows])
