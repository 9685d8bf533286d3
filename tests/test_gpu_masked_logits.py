"""GPU parity with masked actions and large logits: rows with some logits at a
large negative finite value (how illegal actions are often masked), in the target
policy, the behaviour policy or both, and rows shifted as a whole.  A softmax
does not change under a shift, so rows of masks alone must give what rows of
zeros give; the oracle's float64 log-softmax of a shift of 1e9 is within 2e-7.
Element-wise bound 1e-5 + 1e-4 |o|, as everywhere."""

import math

import numpy as np
import pytest
import torch

import oracle
import paper_1802_01561_amd as vt
from gpu_util import assert_close, call_params, log_case, np_out, oracle_args, require_gpu, to_device
from synth import Params, make_random
from test_gpu_parity import check_against_oracle, run_loss_grad

pytestmark = pytest.mark.gpu

F32_LOWEST = float(np.finfo(np.float32).min)
BF16_LOWEST = -float.fromhex("0x1.fep127")
# Multiples of a unit of bfloat16 at these magnitudes: the values are the same in both types.
MASKS = [-float.fromhex("0x1.dcp29"), -2.0 ** 31, -float.fromhex("0x1.94p99"), None]  # about -1e9, ..., -1e30


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def masked_batch(T, B, A, seed, mask, bf16, rows=0.5):
    """Some rows with about half of the actions not taken masked, in one policy or both."""
    tr = make_random(T, B, A, seed, noise_std=1.0, end_prob=0.05, bf16=bf16)
    rng = np.random.default_rng(seed)
    if mask is None:
        mask = BF16_LOWEST if bf16 else F32_LOWEST
    hit = (rng.random((T, B, A)) < 0.5) & (np.arange(A) != tr.actions[..., None])
    for logits in (tr.target_logits, tr.behaviour_logits):
        logits[hit & (rng.random((T, B, 1)) < rows)] = mask
    return changed(tr)


def changed(tr):
    """The batch after a change of its float32 logits."""
    if tr.dtype == "bf16":
        tr.target_bits, tr.behaviour_bits = (np.ascontiguousarray(x).view(np.uint32).__rshift__(16).astype(np.uint16)
                                             for x in (tr.target_logits, tr.behaviour_logits))
    return tr


# On a 256-CU part 16, 8, 2 and 1 lanes per tile, the row-split and the generic kernel.
@pytest.mark.parametrize("T,B,A,bf16", [(20, 8200, 2, False), (20, 8200, 9, True), (33, 3601, 6, False),
                                        (100, 37, 9, False), (100, 37, 20, True), (257, 37, 18, False),
                                        (257, 37, 20, False), (70, 37, 21, False), (70, 37, 48, True),
                                        (20, 37, 100, False), (10, 7, 300, False)])
@pytest.mark.parametrize("mask", MASKS)
def test_masked_actions(T, B, A, bf16, mask):
    tr = masked_batch(T, B, A, 9500 + A + T, mask, bf16)
    dev = to_device(tr)
    lanes = sorted({0, 1, B // 2, *range(max(0, B - 20), B)})
    # (An entropy cost above 1 times the lowest value leaves float32's range.)
    for p in (Params(1.0, 1.0, 1.0), Params(math.inf, math.inf, 0.9, 0.5, 2.0)):
        log_case(f"masked T={T} B={B} A={A} bf16={bf16} mask={mask} {p.label()}")
        check_against_oracle(tr, p, run_loss_grad(dev, p), lanes=lanes)
        vs, pg = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
        q = call_params(p)
        o = oracle.vtrace(*oracle_args(tr), q.rho_bar, q.c_bar, q.lam)
        assert_close("targets.vs", np_out(vs), o.vs)
        assert_close("targets.pg_advantages", np_out(pg), o.pg_advantages)


@pytest.mark.parametrize("A,bf16", [(2, True), (9, False), (18, False), (20, True), (21, False), (48, True), (100, False),
                                    (300, False)])
@pytest.mark.parametrize("variant", [{}, dict(correction="one_step_is", reward_transform="clip")])
def test_rows_of_masks_are_uniform(A, bf16, variant):
    """Every logit of a row at one value, of any size, gives what zeros give."""
    T, B = 40, 70
    for value in (2.0 ** 21, -2.0 ** 30, 2.0 ** 100, -2.0 ** 127):
        tr = make_random(T, B, A, 9600 + A, noise_std=1.0, end_prob=0.05, bf16=bf16)
        rows = np.random.default_rng(A).random((2, T, B)) < 0.3
        out = []
        for x in (0.0, value):
            tr.target_logits[rows[0]] = x
            tr.behaviour_logits[rows[1]] = x
            dev = to_device(changed(tr))
            p = Params(2.0, 1.0, 0.9)
            res = run_loss_grad(dev, p, **variant)
            out.append([np_out(t) for t in (*res, *vt.vtrace_targets(**dev, rho_bar=p.rho_bar, **variant))])
        log_case(f"rows of {value}, A={A} bf16={bf16} {variant}")
        for got, expect in zip(out[1], out[0]):
            assert_close(f"rows of {value}", got, expect)


@pytest.mark.parametrize("A", [9, 18, 21, 48, 100, 300])
def test_shifted_rows(A):
    """Rows shifted by a large common offset (a multiple of the logits' spacing there)."""
    T, B = 40, 70
    rng = np.random.default_rng(A)
    for offset in (100.0, -3000.0, 2.0 ** 17, -2.0 ** 22):
        tr = make_random(T, B, A, 9700 + A, noise_std=1.0, end_prob=0.05)
        for logits in (tr.target_logits, tr.behaviour_logits):
            logits[rng.random((T, B)) < 0.5] += np.float32(offset)
        log_case(f"rows shifted by {offset}, A={A}")
        p = Params(1.0, 1.0, 1.0)
        check_against_oracle(tr, p, run_loss_grad(to_device(tr), p))


def test_infinite_masks_pass_through():
    """-inf logits of actions not taken: targets as for probability 0, and NaN in
    that row's gradient and in the entropy, for every action count."""
    T, B = 40, 70
    for A in (9, 20, 21, 100, 300):
        tr = masked_batch(T, B, A, 9800 + A, -2.0 ** 30, False)
        p = Params(2.0, 1.0, 0.9)
        ref = run_loss_grad(to_device(tr), p)
        hit = [(x == -2.0 ** 30) for x in (tr.target_logits, tr.behaviour_logits)]
        tr.target_logits[hit[0]] = tr.behaviour_logits[hit[1]] = -np.inf
        log_case(f"-inf logits, A={A}")
        out = run_loss_grad(to_device(tr), p)
        for name in ("vs", "pg_advantages", "d_values"):
            assert torch.equal(getattr(out, name), getattr(ref, name)), name
        rows = hit[0].any(-1)
        assert np.isnan(np_out(out.d_logits)[rows]).all() and np.isnan(np_out(out.losses)[3])
        assert np.array_equal(np_out(out.d_logits)[~rows], np_out(ref.d_logits)[~rows])
