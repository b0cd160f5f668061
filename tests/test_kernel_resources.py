"""Registers of the attention kernels as the compiler reports them: none keeps anything in scratch
memory, which its loops would reload after every barrier."""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2305_19370_amd import build


def _report(src):
    cmd = [build._hipcc(), *build.HIP_FLAGS, *build.EXTRA_FLAGS.get(src, []), "--cuda-device-only", "-c",
           "-Rpass-analysis=kernel-resource-usage", os.path.join(build.CSRC, src), "-o", os.devnull]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return dict(zip(re.findall(r"Function Name: (\S+)", r.stderr), map(int, re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr))))


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
def test_attention_kernels_use_no_scratch():
    srcs = ["attn_fwd.hip", "attn_bwd_dkdv.hip", "attn_bwd_dq.hip"]
    with concurrent.futures.ThreadPoolExecutor(3) as ex:
        for src, got in zip(srcs, ex.map(_report, srcs)):
            assert len(got) == 6, (src, got)          # bf16: two head sizes of 4 and 8 waves; fp32: two
            assert not any(got.values()), (src, got)
