"""What the compiler made of csrc/fq_gemm_ring.hip (gfx950 assembly of this repository's own source): the
hand-written global -> LDS loads keep their wait states by themselves, the accumulators are kept once, nothing spills."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_08040_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc is not installed")
    out = tmp_path_factory.mktemp("asm") / "fq_gemm_ring.s"
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    r = subprocess.run([HIPCC, *flags, "--offload-device-only", "-S", "-o", str(out),
                        os.path.join(build.CSRC, "fq_gemm_ring.hip")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def test_direct_loads_keep_their_wait_states(assembly):
    blocks, inside = [], None
    for line in assembly.splitlines():
        line = line.strip() if line.strip().startswith(";;#") else line.split(";")[0].strip()
        if line == ";;#ASMSTART":
            inside = []
        elif line == ";;#ASMEND":
            if any("global_load_lds" in s for s in inside):
                blocks.append(inside)
            inside = None
        elif inside is not None:
            inside.append(line)
        else:
            assert "global_load_lds" not in line and not re.search(r"\bm0\b", line), line
    assert len(blocks) > 20
    for b in blocks:
        # m0, then the base moved by the scalar unit (which is also the wait state behind m0), then loads only
        assert re.fullmatch(r"s_mov_b32 m0, s\d+", b[0]), b
        base = re.fullmatch(r"s_mov_b64 (s\[\d+:\d+\]), \1", b[1])
        assert base, b
        for n, s in enumerate(b[2:]):
            m = re.fullmatch(r"global_load_lds_dword(x4)? v\d+, (s\[\d+:\d+\])(?: offset:(\d+))?", s)
            assert m and m.group(2) == base.group(1) and int(m.group(3) or 0) == 1024 * n, b


def test_registers(assembly):
    kernels = re.findall(r"\.name:\s+(\S*gemm_ring_kernel\S*)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)\n\s+\.vgpr_spill_count: (\d+)",
                         assembly)
    assert len(kernels) == 3
    # 168 registers are what three wavefronts of a SIMD may have, 128 what four may
    assert sorted(int(v) <= 128 for _, v, _ in kernels) == [False, True, True], kernels
    assert all(int(v) <= 168 and s == "0" for _, v, s in kernels), kernels
