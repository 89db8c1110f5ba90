"""What the compiler made of csrc/fq_gemm.hip (gfx950 assembly of this repository's own source).

The global -> LDS loads are written as assembly, which the compiler's hazard pass does not look into:
a load may not follow the write of its base address by a vector instruction within five wait states, nor
the write of m0 within one, and m0 may hold nothing of the compiler's."""
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
    out = tmp_path_factory.mktemp("asm") / "fq_gemm.s"
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    r = subprocess.run([HIPCC, *flags, "--offload-device-only", "-S", "-o", str(out),
                        os.path.join(build.CSRC, "fq_gemm.hip")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return out.read_text().splitlines()


def test_direct_loads_keep_their_wait_states_by_themselves(assembly):
    blocks, inside = [], None
    for line in assembly:
        line = line.split(";")[0].strip() if not line.strip().startswith(";;#") else line.strip()
        if line == ";;#ASMSTART":
            inside = []
        elif line == ";;#ASMEND":
            if any("global_load_lds" in s for s in inside):
                blocks.append(inside)
            inside = None
        elif inside is not None:
            inside.append(line)
        else:
            assert "global_load_lds" not in line, line
            assert not re.search(r"\bm0\b", line), f"the compiler uses m0 itself: {line}"
    assert len(blocks) > 20
    for b in blocks:
        first = next(i for i, s in enumerate(b) if s.startswith("global_load_lds"))
        loads = [re.fullmatch(r"global_load_lds_dwordx4 v\d+, (s\[\d+:\d+\])(?: offset:\d+)?", s) for s in b[first:]]
        assert len(loads) == 4 and all(loads), b
        base = {m.group(1) for m in loads}
        assert len(base) == 1, b
        before = b[:first]
        m0 = [i for i, s in enumerate(before) if s.startswith("s_mov_b32 m0,")]
        assert m0 and first - m0[-1] >= 2, f"no wait state between m0 and its use: {b}"
        assert any(s.startswith(f"s_mov_b64 {next(iter(base))},") for s in before), \
            f"the base may come straight from a vector instruction: {b}"

