"""GPU parity of the row-split kernel (20 < A <= 256) against the oracle: the
edges of its column split (A at and around multiples of 16 and 64 per-thread
columns, an A that leaves the last threads overlapping), of its 64- and 16-step
chunks, more lanes than workgroups, and every variant switch; and an action
count beyond it, which keeps the generic kernel.  Element-wise bound
1e-5 + 1e-4 |o|, as for every other kernel."""

import math

import numpy as np
import pytest
import torch

import oracle
import paper_1802_01561_amd as vt
from gpu_util import assert_close, log_case, np_out, oracle_args, require_gpu, to_device
from synth import Params, make_random, subset_lanes
from test_gpu_variants import check_io_variant

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("A", [21, 31, 32, 33, 48, 49, 64, 65, 127, 128, 129, 193, 256, 257])
@pytest.mark.parametrize("bf16", [False, True])
def test_action_counts(A, bf16):
    for T, B, p in ((65, 5, Params(1.0, 1.0, 1.0)), (17, 3, Params(math.inf, math.inf, 1.0))):
        tr = make_random(T, B, A, 8000 + A + T, noise_std=1.0, end_prob=0.05, bf16=bf16)
        log_case(f"rows A={A} T={T} B={B} bf16={bf16} {p.label()}")
        check_io_variant(tr, p)


@pytest.mark.parametrize("T", [1, 15, 16, 63, 64, 128, 130])
@pytest.mark.parametrize("A", [40, 100])
def test_unroll_lengths(T, A):
    tr = make_random(T, 7, A, 8100 + A + T, noise_std=1.0, end_prob=0.05)
    log_case(f"rows A={A} T={T} B=7")
    check_io_variant(tr, Params(1.0, 0.5, 0.95))


@pytest.mark.parametrize("correction", ["vtrace", "none", "epsilon", "one_step_is"])
@pytest.mark.parametrize("log_probs,transform,grad_bf16,q_estimate",
                         [(False, "asymmetric", True, "vtrace"), (True, "clip", False, "baseline"),
                          (True, None, True, "vtrace")])
def test_variants(correction, log_probs, transform, grad_bf16, q_estimate):
    for A, bf16 in ((37, True), (70, False)):
        tr = make_random(70, 9, A, 8200 + A, noise_std=1.0, end_prob=0.05, bf16=bf16)
        tr.rewards = (tr.rewards * 2.5).astype(np.float32)
        log_case(f"rows A={A} {correction}/{q_estimate} lp={log_probs} r={transform} bf16 grads={grad_bf16}")
        check_io_variant(tr, Params(2.0, 1.0, 0.9), correction=correction, log_probs=log_probs,
                         reward_transform=transform, grad_bf16=grad_bf16, q_estimate=q_estimate)


def test_more_lanes_than_workgroups():
    B = 4099
    tr = make_random(9, B, 22, 8300, noise_std=1.0, end_prob=0.05)
    log_case("rows, lanes beyond the workgroup count")
    check_io_variant(tr, Params(1.0, 1.0, 1.0), lanes=[0, 1, 4094, 4095, 4096, 4097, B - 1])


@pytest.mark.parametrize("T,B,A", [(1, 1023, 21), (1, 1024, 21), (2, 1024, 21), (1, 2049, 22), (3, 4098, 21),
                                   (7, 8191, 22), (1, 8200, 113), (4, 16384, 40), (1, 20000, 220)])
def test_short_unrolls_of_many_lanes(T, B, A):
    """Both sides of the rule that gives short unrolls one thread per lane, and
    lanes beyond either kernel's workgroups."""
    tr = make_random(T, B, A, 8500 + A + T, noise_std=1.0, end_prob=0.05)
    log_case(f"rows or one thread per lane, T={T} B={B} A={A}")
    lanes = sorted({0, 1, 63, 64, *range(B - 3, B), *(i for i in (2047, 2048, 4095, 4096) if i < B)})
    check_io_variant(tr, Params(1.0, 1.0, 1.0), lanes=lanes)
    vs, pg = vt.vtrace_targets(**to_device(tr))
    sub = subset_lanes(tr, lanes)
    o = oracle.vtrace(*oracle_args(sub), 1.0, 1.0, 1.0)
    assert_close("targets.vs", np_out(vs)[:, lanes], o.vs)
    assert_close("targets.pg_advantages", np_out(pg)[:, lanes], o.pg_advantages)


def test_bad_values_stay_in_their_lane():
    """A NaN logit and an action out of range poison only their lane's earlier
    steps, and the action raises the flag."""
    T, B, A = 70, 6, 50
    tr = make_random(T, B, A, 8400, noise_std=1.0)
    ref = vt.vtrace_loss_grad(**to_device(tr), with_vs=True)
    tr.target_logits[40, 1, A - 1] = np.nan
    tr.actions[10, 3] = A
    log_case("rows, NaN logit and out-of-range action")
    ws = vt.Workspace(T, B, A)
    out = vt.vtrace_loss_grad(**to_device(tr), with_vs=True, workspace=ws)
    assert vt.vtrace_error_flag(ws) == 1
    keep = [0, 2, 4, 5]
    for name in ("vs", "d_logits", "d_values"):
        x, y = np_out(getattr(out, name)), np_out(getattr(ref, name))
        assert np.array_equal(x[:, keep], y[:, keep]), name
        assert np.array_equal(x[41:, 1], y[41:, 1]) and np.array_equal(x[11:, 3], y[11:, 3]), name
    assert np.isnan(np_out(out.d_logits)[40, 1]).all() and np.isnan(np_out(out.d_logits)[10, 3]).all()
    torch.cuda.synchronize()
