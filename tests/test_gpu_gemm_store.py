"""How the large tiles store: wavefronts inside the output take the unconditional form, those at its edges, or all of them
where the output allows no 16-byte stores, the general one.  Same bits, nothing beside the output written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2503_08040_amd as fq
from tests import gpu_util as gu

# rows, columns, compute units assumed: whole 256 x 256 tiles, one column or row more or less than a wavefront's 64 and 128,
# 128 x 384 tiles over the last block columns and the last block rows
SHAPES = [(256, 512, 2), (255, 256, 1), (256, 193, 1), (193, 256, 1), (129, 449, 1), (256, 1664, 4), (129, 1589, 4),
          (1280, 256, 2), (1275, 253, 2)]


@pytest.mark.parametrize("variant", ["exact", "residual items", "biased"])
@pytest.mark.parametrize("M,N,cus", SHAPES)
def test_stores(M, N, cus, variant, monkeypatch):
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    biased = variant == "biased"
    assert fq.fq_gemm_path(M, N, biased=biased)[0] == fq.FQ_TILES_256x256
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    x = torch.randn(M, 300, device="cuda", generator=g)
    if variant != "exact":
        x[M // 2, 150] = 90.0
    a = (fq.fq_quantize(x.bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0) if variant == "exact"
         else fq.fq_quantize(x.bfloat16(), fq.FQ_CRIT_ABSMAX_GT, 30.0))
    b = fq.fq_quantize(torch.randn(N, 300, device="cuda", generator=g).bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    product = fq.fq_gemm_biased if biased else fq.fq_gemm
    gu.announce(f"stores {variant} {M}x{N}")
    for dt in (torch.float32, torch.bfloat16):
        bits = torch.int32 if dt == torch.float32 else torch.int16
        pitch = -(-N // 8) * 8 + 16
        outs = []
        for shift in (0, 1):      # 16-byte stores, none
            buf = torch.full((M + 2, pitch), -77.0, device="cuda", dtype=dt)
            out = buf.view(-1)[pitch + shift:pitch + shift + M * pitch].view(M, pitch)[:, :N]
            product(fq.FQ_OP_NT, a, b, out=out)
            outs.append(out.clone())
            out.fill_(-77.0)
            assert (buf == -77.0).all(), "written beside the output"
        assert torch.equal(outs[0].view(bits), outs[1].view(bits))
        if dt == torch.float32:
            full = outs[0]
        else:
            assert torch.equal(outs[0].view(bits), full.bfloat16().view(bits))
    if not biased:                # the smaller tiles, which store otherwise
        monkeypatch.delenv("FQ_GEMM_CUS")
        assert torch.equal(product(fq.FQ_OP_NT, a, b), full)


# tail tiles: 20, 20, 32 and 32, of which 8 and 16 come before the main tiles (no fallback, binary32 output, up to 16 k-blocks)
@pytest.mark.parametrize("M,N,cus", [(1280, 1900, 24), (1280, 3000, 24), (2560, 3000, 32), (2048, 3000, 40)])
@pytest.mark.parametrize("K", [200, 2048, 2049])
def test_order_of_tail_tiles(M, N, cus, K, monkeypatch):
    monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
    path = fq.fq_gemm_path(M, N)
    assert path[0] == fq.FQ_TILES_256x256 and path[2] + path[3] >= 16
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    x = torch.randn(M, K, device="cuda", generator=g)
    x[::300, 150] = 90.0
    b = fq.fq_quantize(torch.randn(N, K, device="cuda", generator=g).bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    for a in (fq.fq_quantize(x.bfloat16(), fq.FQ_CRIT_ABSMAX_GT, 30.0),
              fq.fq_quantize(x.bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0)):
        gu.announce(f"order of tail tiles {M}x{N}x{K}")
        full = torch.full((M, N), float("nan"), device="cuda")
        fq.fq_gemm(fq.FQ_OP_NT, a, b, out=full)
        monkeypatch.setenv("FQ_GEMM_CUS", "0")           # 256 x 256 or smaller tiles only
        assert torch.equal(fq.fq_gemm(fq.FQ_OP_NT, a, b), full)
        monkeypatch.setenv("FQ_GEMM_CUS", str(cus))
        assert torch.equal(fq.fq_gemm(fq.FQ_OP_NT, a, b, out_dtype=torch.bfloat16), full.bfloat16())
