"""GPU parity of the output-layer kernel's two work splits against the oracle:
a workgroup per lane (its four waves on consecutive 16-step chunks) up to 512
lanes, four lanes per workgroup beyond and where the workspace holds partials
for no more.  Unrolls at the edges of a wave's and a workgroup's chunks, so that
some waves lie wholly before t = 0; several lane groups per workgroup.  Bounds
as in test_gpu_head.py."""

import math

import numpy as np
import pytest
import torch

import paper_1802_01561_amd as vt
from gpu_util import log_case, require_gpu
from synth import Params, make_head
from test_gpu_head import check_head, head_to_device, run_head

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("T", [17, 32, 33, 63, 64, 65, 129])
@pytest.mark.parametrize("A,H", [(9, 64), (18, 256)])
def test_one_lane_per_workgroup(T, A, H):
    hb = make_head(T, 5, A, H, 30000 + T + H, end_prob=0.05)
    dev = head_to_device(hb)
    for p in (Params(1.0, 0.5, 0.95), Params(math.inf, math.inf, 1.0)):
        log_case(f"head split T={T} B=5 A={A} H={H} {p.label()}")
        check_head(hb, p, run_head(dev, p))


@pytest.mark.parametrize("T,B", [(33, 512), (33, 513), (20, 256), (20, 257)])
def test_split_boundaries(T, B):
    hb = make_head(T, B, 9, 128, 31000 + T + B, end_prob=0.05)
    dev = head_to_device(hb)
    log_case(f"head split boundary T={T} B={B}")
    check_head(hb, Params(1.0, 1.0, 1.0), run_head(dev, Params(1.0, 1.0, 1.0), grad_dtype=torch.bfloat16),
               grad_bf16=True)


def test_several_groups_of_several_chunks():
    """Lane groups beyond the workgroup count, each of more than one chunk: a
    group's first chunk and bootstrap values load during the previous group's
    last chunk."""
    hb = make_head(40, 2101, 9, 64, 32000, end_prob=0.05)
    p = Params(1.0, 1.0, 1.0)
    log_case("head T=40 B=2101: several groups per workgroup")
    check_head(hb, p, run_head(head_to_device(hb), p))


def test_workspace_of_four_lane_groups():
    """A workspace with partials for a workgroup per four lanes is enough."""
    T, B, A, H = 70, 30, 18, 64
    hb = make_head(T, B, A, H, 33000, end_prob=0.05)
    dev = head_to_device(hb)
    ws = vt.Workspace(T, B, A, H=H)
    groups = -(-B // 4)
    least = 256 + -(-groups * 24 // 256) * 256 + 4 * groups * (H + 1) * 32
    assert least < ws.nbytes
    small = vt.Workspace(T, B, A, H=H)
    small.tensor, small.nbytes = small.tensor[:least].clone(), least
    p = Params(1.0, 1.0, 1.0)
    log_case("head, small workspace")
    check_head(hb, p, run_head(dev, p, workspace=small))
    small.nbytes = least - 1
    with pytest.raises(vt.VtraceError, match="WORKSPACE"):
        run_head(dev, p, workspace=small)


def test_captured_replays():
    hb = make_head(100, 32, 9, 256, 34000)
    dev = head_to_device(hb)
    p = Params(1.0, 1.0, 1.0)
    ws = vt.Workspace(hb.T, hb.B, hb.A, H=hb.H)
    log_case("head captured")
    eager = run_head(dev, p, workspace=ws)
    out = run_head(dev, p, workspace=ws)
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            vt.vtrace_head_loss_grad(**dev, rho_bar=1.0, c_bar=1.0, lam=1.0, workspace=ws, out=out)
    for _ in range(3):
        for x in out:
            x.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        for name, x, y in zip(out._fields, out, eager):
            assert torch.equal(x, y), name
        run_head(dev, Params(1.0, 0.5, 0.95), workspace=ws)  # eager work between replays
