"""NaN inputs: their codes are unspecified, but they do not enter a block's scale or its fallback
decision, which come from the other values (as in the oracle)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from oracle import fqo
from paper_2503_08040_amd import synth
from tests import gpu_util as gu


@pytest.mark.parametrize("rows,cols", [(256, 384), (133, 270)])
def test_nan_does_not_enter_the_scale(rows, cols):
    rng = np.random.default_rng(rows)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    x[5, 7] = x[131, 3] = 100.0
    bits = synth.to_bf16_bits(x)
    bits[3, 200] = 0x7FC0                       # next to ordinary values
    bits[131, 140] = 0xFFFF
    bits[128:, :128][:, 64:] = 0x7F81           # half a block, beside its outlier
    gu.announce(f"NaN inputs {rows}x{cols}")
    o = fqo.quantize(bits, 128, fqo.CRIT_ABSMAX_GT, 12.0)
    g = fq.fq_quantize(gu.to_device_bf16(bits), fq.FQ_CRIT_ABSMAX_GT, 12.0)
    assert np.isfinite(o.scales).all()
    assert np.array_equal(g.view("scales").cpu().numpy(), o.scales)
    assert fq.fq_qtensor_check(g) == int(o.fb_count[0]) == 2
    s = fq.fq_quantize_sr(gu.to_device_bf16(bits), 11)
    assert np.array_equal(s.view("scales").cpu().numpy(), o.scales)
    t = fq.fq_quantize_topk(gu.to_device_bf16(bits), 2)
    assert np.array_equal(t.view("mask").cpu().numpy(), g.view("mask").cpu().numpy())
