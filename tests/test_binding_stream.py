"""The stream that the binding launches on, by torch's private and public names."""

import subprocess
import sys

import pytest
import torch

from gpu_helpers import require_gpu, say

import paper_2609_19868_amd as Z


def test_binding_needs_no_private_name_of_torch():
    code = ("import torch; del torch._C._cuda_getCurrentRawStream; import paper_2609_19868_amd as Z; "
            "assert Z._raw_stream is Z._public_raw_stream")
    had = "import torch; assert hasattr(torch._C, '_cuda_getCurrentRawStream'); "
    subprocess.run([sys.executable, "-c", (had if Z._raw_stream is not Z._public_raw_stream else "") + code], check=True,
                   timeout=300)


@pytest.mark.gpu
@pytest.mark.parametrize("public", [False, True])
def test_calls_follow_the_current_stream(public, monkeypatch):
    dev = require_gpu()
    if public:
        monkeypatch.setattr(Z, "_raw_stream", Z._public_raw_stream)
    conf = torch.rand((4, 8, 8), device=dev)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    say(f"select_slots on a side stream, public name {public}")
    with torch.cuda.stream(side):
        assert Z._raw_stream(0) == side.cuda_stream
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):  # a launch elsewhere would not be recorded
            out = Z.select_slots(conf)
        for t in out:
            t.zero_()
        g.replay()
    torch.cuda.synchronize()
    for a, b in zip(out, Z.select_slots(conf)):
        assert torch.equal(a, b)
    torch.cuda.synchronize()
