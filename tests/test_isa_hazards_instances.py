"""The wait-state checks of test_isa_hazards.py over every instance of a kernel template that
writes its MFMAs in assembly (that test reads the first instance of each)."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2509_21081_amd import build as B
from tests import test_isa_hazards as hz


@pytest.mark.parametrize("source,kernel,count", [("tmla_prefix_mfma.hip", "prefix_attn_pipelined_kernel", 2),
                                                 ("tmla_absorb128_mfma.hip", "absorb128_kernel", 2),
                                                 ("tmla_expand_mfma.hip", "expand_gemm_kernel", 2)])
@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_every_instance_keeps_the_wait_states(source, kernel, count):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        subprocess.run([B.HIPCC, *B.FLAGS, "-S", "--cuda-device-only", "-o", out,
                        os.path.join(B.CSRC, source)], check=True, capture_output=True)
        text = open(out).read()
    starts = [m.start() for m in re.finditer(r"\n_ZN4tmla%d%sI[^:\s]*:" % (len(kernel), kernel), text)]
    assert len(starts) == count
    for start in starts:
        instrs, labels = [], {}
        for raw in text[start:text.index("\n.Lfunc_end", start)].split("\n"):
            t = raw.split(";")[0].strip()
            if t.endswith(":"):
                labels[t[:-1]] = len(instrs)
            elif t and not t.startswith("."):
                instrs.append(t)
        for where, seq in hz._sequences(instrs, labels):
            n = hz._check_valu_to_mfma(seq, where)
            hz._check_mfma_result(seq, where)
            assert where != "text order" or n > 100
