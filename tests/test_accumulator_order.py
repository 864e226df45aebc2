"""The square GEMM tiles multiply in inline assembly, so the compiler knows nothing of the cycles until a product arrives:
the wait behind the K loop is a statement of the source, and every read of an accumulator has to hang on it.  Compiles the
SwiGLU kernels to LLVM IR and follows each read back to its origin; no GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2602_07306_amd import build as B

READ = re.compile(r"^\s*(%\S+) = .*asm \"v_accvgpr_read_b32[^\"]*\", \"=v,a\"\(float (%\S+)\)")
ELEMENT = re.compile(r"^\s*(%\S+) = extractelement <4 x float> (%\S+), ")
TIED = re.compile(r"^\s*(%\S+) = .*asm sideeffect \"\", \"=a,0[^\"]*\"\(<4 x float> ")


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not found")
def test_accumulators_are_read_behind_the_wait(tmp_path):
    out = tmp_path / "swiglu.ll"
    cmd = [B.HIPCC] + B.COMMON + ["--cuda-device-only", "-emit-llvm", "-S", os.path.join(B.CSRC, "kernels_gemm_mfma_swiglu.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = 0
    for body in out.read_text().split("\ndefine ")[1:]:
        if "v_mfma_f32_16x16x32_bf16" not in body:
            continue
        kernels += 1
        origin, tied, reads = {}, set(), []
        for line in body.splitlines():
            for pattern, keep in ((READ, lambda m: reads.append(m[2])), (ELEMENT, lambda m: origin.__setitem__(m[1], m[2])),
                                  (TIED, lambda m: tied.add(m[1]))):
                m = pattern.match(line)
                if m:
                    keep(m)
        loose = [x for x in reads if origin.get(x) not in tied]
        assert reads and not loose, (body.split("(")[0][-80:], len(reads), len(loose))
        assert body.rindex("s_nop 15") < body.index('asm sideeffect "", "=a,0')
    assert kernels >= 3   # 256 x 256, 128 x 128, and its form with four K steps in flight
