"""The multi-token kernel's tilings, chosen by defines, compile (the device pass for gfx950,
without code generation)."""
import os
import subprocess

import pytest

from paper_2607_09207_amd import build as B


@pytest.mark.parametrize("defines", [[], ["RLDA_MQ_TILES=2"], ["RLDA_MQ_KEY_TILES=2"], ["RLDA_MQ_DMA=0", "RLDA_MQ_PREFETCH=2"]],
                         ids=lambda d: "+".join(d) or "default")
def test_tilings_compile(defines):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    src = os.path.join(B.CSRC, "rlda_multi.hip")
    cmd = [B.HIPCC] + [f for f in B.FLAGS if f != "-shared"] + ["--cuda-device-only", "-fsyntax-only", src]
    r = subprocess.run(cmd + ["-D" + d for d in defines], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
