"""The build refuses kernels of the wide attention source that spill."""
import subprocess

import pytest

from paper_2607_24260_amd import build as B

REMARKS = """\
attn_wide.hip:420:0: remark: Function Name: k1 [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark:     ScratchSize [bytes/lane]: {} [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark:     SGPRs Spill: 5 [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark:     VGPRs Spill: {} [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark: Function Name: k2 [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]
attn_wide.hip:420:0: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]
"""


@pytest.mark.parametrize("scratch,regs", [(0, 0), (0, 3), (36, 0), (24, 7)])
def test_spilling_kernels_stop_the_build(monkeypatch, scratch, regs):
    text = REMARKS.format(scratch, regs)
    want = [("k1", regs, scratch)] if scratch or regs else []
    assert B.spills(text) == want
    run = lambda cmd, **kw: subprocess.CompletedProcess(cmd, 0, "", text)
    monkeypatch.setattr(B.subprocess, "run", run)
    if want:
        with pytest.raises(RuntimeError, match="spills"):
            B._compile("/x/attn_wide.hip", False)
    else:
        B._compile("/x/attn_wide.hip", False)
    B._compile("/x/decode_fast.hip", False)      # not checked


def test_a_build_without_remarks_is_refused(monkeypatch):
    run = lambda cmd, **kw: subprocess.CompletedProcess(cmd, 0, "", "")
    monkeypatch.setattr(B.subprocess, "run", run)
    with pytest.raises(RuntimeError, match="unknown"):
        B._compile("/x/attn_wide.hip", False)
