"""The ascending list of flagged blocks around groups of 32 blocks: which workgroup counts a group last (a flagged block
counts before its residual, an unflagged one at its end) must not show in it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from tests import gpu_util as gu


@pytest.mark.parametrize("blocks", [31, 32, 33, 64, 65, 300])
@pytest.mark.parametrize("which", ["all", "all but one", "one", "last group", "even", "random"])
def test_list_of_flagged_blocks(blocks, which):
    rng = np.random.default_rng(blocks)
    flag = {"all": np.ones(blocks), "all but one": np.arange(blocks) != blocks // 2, "one": np.arange(blocks) == blocks - 1,
            "last group": np.arange(blocks) // 32 == (blocks - 1) // 32, "even": np.arange(blocks) % 2 == 0,
            "random": rng.random(blocks) < 0.2}[which].astype(bool)
    x = torch.ones((128, 128 * blocks), device="cuda")
    x.view(128, blocks, 128)[5, :, 7] += torch.from_numpy(99.0 * flag).float().cuda()
    x = x.bfloat16()
    q = fq.QTensor(128, 128 * blocks)
    gu.announce(f"list of {blocks} blocks, {which}")
    for _ in range(4):                      # the counters alternate from call to call
        q.view("fb_list").fill_(-7)
        fq.fq_quantize(x, fq.FQ_CRIT_ABSMAX_GT, 50.0, out=q)
        n = int(q.view("fb_count"))
        assert n == flag.sum()
        assert np.array_equal(q.view("fb_list").cpu().numpy()[:n], np.flatnonzero(flag))
        assert np.array_equal(q.view("mask").cpu().numpy()[0].astype(bool), flag)
        slots = q.view("fb_slot").cpu().numpy()[0]
        assert sorted(slots[flag]) == list(range(n)) and (slots[~flag] == -1).all()
