"""GPU parity: the HIP path through the C ABI against the fp64 oracle.

fp32 outputs must satisfy |g - o| <= 1e-5 + 1e-4 |o| element by element;
gathers must be bit-exact.  The oracle sees the same seeded inputs.
"""

import math

import numpy as np
import pytest
import torch

import oracle
import paper_1802_01561_amd as vt
from gpu_util import assert_close, call_params, log_case, np_out, oracle_args, require_gpu, to_device
from synth import PARAM_SETS, make_config, make_random, subset_lanes
from synth.trajectories import STRESS_SUBSET

pytestmark = pytest.mark.gpu


def run_loss_grad(dev, p, **kw):
    out = vt.vtrace_loss_grad(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam,
                              baseline_cost=p.baseline_cost, entropy_cost=p.entropy_cost,
                              with_vs=True, with_pg_advantages=True, with_lane_losses=True, **kw)
    torch.cuda.synchronize()
    return out


def check_against_oracle(tr, p, out, lanes=None):
    """Compare every output of a loss_grad call with the oracle (optionally on a
    subset of lanes, where the oracle runs on those lanes alone)."""
    sub = tr if lanes is None else subset_lanes(tr, lanes)
    q = call_params(p)
    o = oracle.loss_and_grads(*oracle_args(sub), q.rho_bar, q.c_bar, q.lam,
                              q.baseline_cost, q.entropy_cost)
    pick = (lambda x: x) if lanes is None else (lambda x: x[:, lanes])
    assert_close("vs", pick(np_out(out.vs)), o.vs)
    assert_close("pg_advantages", pick(np_out(out.pg_advantages)), o.pg_advantages)
    assert_close("d_values", pick(np_out(out.d_values)), o.d_values)
    assert_close("d_logits", pick(np_out(out.d_logits)), o.d_logits)
    lane = np_out(out.lane_losses)
    assert_close("lane_losses", lane if lanes is None else lane[lanes], o.lane_losses)
    if lanes is None:
        assert_close("losses", np_out(out.losses), o.losses)
    return o


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("cfg,bf16", [(0, False), (1, False), (2, False), (3, False), (3, True),
                                      (0, True), (2, True)])
def test_config_matches_oracle(cfg, bf16):
    tr = make_config(cfg, bf16=bf16)
    for p in PARAM_SETS[cfg]:
        log_case(f"config {cfg} ({tr.name}) {p.label()} T={tr.T} B={tr.B} A={tr.A}")
        dev = to_device(tr)
        out = run_loss_grad(dev, p)
        check_against_oracle(tr, p, out)
        vs, pg = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
        torch.cuda.synchronize()
        q = call_params(p)
        o = oracle.vtrace(*oracle_args(tr), q.rho_bar, q.c_bar, q.lam)
        assert_close("targets.vs", np_out(vs), o.vs)
        assert_close("targets.pg_advantages", np_out(pg), o.pg_advantages)
        g = vt.vtrace_gather_logits(dev["target_logits"], dev["behaviour_logits"], dev["actions"])
        torch.cuda.synchronize()
        zt, yt = tr.logits_for_device()
        expect = oracle.gather_action_logits(zt, yt, tr.actions)
        got = g.cpu().view(torch.int16).numpy() if bf16 else g.cpu().numpy()
        assert got.tobytes() == np.ascontiguousarray(expect).tobytes()


@pytest.fixture(scope="module")
def stress():
    log_case("generating the stress batch T=1000 B=16384 A=18")
    tr = make_config(4)
    dev = to_device(tr)
    return tr, dev


@pytest.mark.parametrize("pidx", [0, 1, 2])
def test_stress_subset_matches_oracle(stress, pidx):
    tr, dev = stress
    p = PARAM_SETS[4][pidx]
    log_case(f"stress T=1000 B=16384 A=18 {p.label()}: full launch, oracle on 64 lanes")
    out = run_loss_grad(dev, p)
    check_against_oracle(tr, p, out, lanes=STRESS_SUBSET)
    # the totals are the fixed-order sums of the per-lane partials
    lane = np_out(out.lane_losses).astype(np.float64)
    losses = np_out(out.losses).astype(np.float64)
    assert_close("losses vs lane sums", losses[1:], lane.sum(axis=0), rtol=1e-4, atol=1e-3)
    assert losses[0] == pytest.approx(losses[1:].sum(), rel=1e-6)


@pytest.mark.parametrize("pidx", [0, 1, 2])
def test_stress_every_lane_matches_oracle(stress, pidx):
    """The full stress launch (T=1000, B=16384, A=18) with each parameter set
    (every one forms its exponent sums in float64), every output element
    against the oracle, which runs on 2048 lanes at a time to bound host memory;
    the totals against the fp64 sum of the oracle's lane losses.  Lane losses
    and totals are held to the element-wise bound: the policy-gradient loss of
    some lanes is a few hundredths from a thousand terms of order one."""
    tr, dev = stress
    p = PARAM_SETS[4][pidx]
    log_case(f"stress T=1000 B=16384 A=18 {p.label()}, every lane against the oracle")
    out = run_loss_grad(dev, p)
    got = {k: np_out(getattr(out, k)) for k in ("vs", "pg_advantages", "d_values", "d_logits")}
    lane = np_out(out.lane_losses)
    o_lane = []
    for l0 in range(0, tr.B, 2048):
        lanes = list(range(l0, min(tr.B, l0 + 2048)))
        q = call_params(p)
        o = oracle.loss_and_grads(*oracle_args(subset_lanes(tr, lanes)), q.rho_bar, q.c_bar, q.lam,
                                  q.baseline_cost, q.entropy_cost)
        for k, ov in (("vs", o.vs), ("pg_advantages", o.pg_advantages), ("d_values", o.d_values),
                      ("d_logits", o.d_logits)):
            assert_close(f"{k} lanes {l0}..", got[k][:, l0:l0 + len(lanes)], ov)
        assert_close(f"lane_losses {l0}..", lane[l0:l0 + len(lanes)], o.lane_losses)
        o_lane.append(o.lane_losses.astype(np.float64))
    tot = np.concatenate(o_lane).sum(axis=0)
    assert_close("losses", np_out(out.losses)[1:], tot)


EDGE_SHAPES = [
    (1, 1, 1), (1, 5, 9), (2, 1, 18), (15, 3, 9), (16, 16, 18), (17, 17, 18), (33, 15, 9),
    (31, 33, 9), (7, 64, 9), (5, 65, 18), (40, 31, 2), (9, 7, 3), (12, 10, 7), (20, 9, 17),
    (11, 6, 33), (3, 4, 100), (65, 2, 5), (8, 129, 18), (24, 40, 9),
]


@pytest.mark.parametrize("T,B,A", EDGE_SHAPES)
def test_edge_shapes(T, B, A):
    tr = make_random(T, B, A, 1000 + T * 7 + B * 3 + A, noise_std=1.0, end_prob=0.05)
    for p in (PARAM_SETS[4][1], PARAM_SETS[4][2]):
        log_case(f"edge T={T} B={B} A={A} {p.label()}")
        out = run_loss_grad(to_device(tr), p)
        check_against_oracle(tr, p, out)


@pytest.mark.parametrize("bf16", [False, True])
def test_edge_shapes_bf16(bf16):
    for (T, B, A) in [(17, 65, 9), (5, 3, 18), (33, 130, 9)]:
        tr = make_random(T, B, A, 77 + T, noise_std=1.0, bf16=bf16)
        p = PARAM_SETS[4][0]
        log_case(f"edge bf16={bf16} T={T} B={B} A={A}")
        check_against_oracle(tr, p, run_loss_grad(to_device(tr), p))


@pytest.mark.parametrize("case", ["extreme_logits", "all_ends", "lambda0", "no_clip", "cbar0",
                                  "action0", "actionlast", "on_policy"])
def test_degenerate_cases(case):
    T, B, A = 37, 40, 18
    kw = dict(noise_std=1.0)
    if case == "extreme_logits":
        kw["logit_scale"] = 80.0
    tr = make_random(T, B, A, 4242, **kw)
    p = PARAM_SETS[4][0]
    if case == "all_ends":
        tr.discounts[:] = 0.0
    if case == "lambda0":
        p = type(p)(1.0, 1.0, 0.0)
    if case == "no_clip":
        p = type(p)(math.inf, math.inf, 1.0)
    if case == "cbar0":
        p = type(p)(2.0, 0.0, 1.0)
    if case == "action0":
        tr.actions[:] = 0
    if case == "actionlast":
        tr.actions[:] = A - 1
    if case == "on_policy":
        tr.behaviour_logits = tr.target_logits.copy()
    log_case(f"degenerate {case}")
    out = run_loss_grad(to_device(tr), p)
    check_against_oracle(tr, p, out)
    if case == "all_ends":
        pg = np_out(out.pg_advantages)
        assert np.all(np.isfinite(pg))


def test_out_of_range_actions_give_nan_and_flag():
    tr = make_random(12, 10, 9, 5)
    tr.actions[5, 3] = 9
    tr.actions[2, 7] = -1
    dev = to_device(tr)
    ws = vt.Workspace(12, 10, 9)
    log_case("out-of-range actions")
    assert vt.vtrace_error_flag(ws) == 0
    out = vt.vtrace_loss_grad(**dev, workspace=ws, with_vs=True, with_pg_advantages=True)
    torch.cuda.synchronize()
    assert vt.vtrace_error_flag(ws) == 1
    dl = np_out(out.d_logits)
    assert np.all(np.isnan(dl[5, 3])) and np.all(np.isnan(dl[2, 7]))
    vs = np_out(out.vs)
    assert np.isnan(vs[5, 3]) and np.all(np.isnan(vs[:5, 3]))
    assert np.all(np.isfinite(vs[6:, 3]))  # later steps are untouched
    good = [b for b in range(10) if b not in (3, 7)]
    assert np.all(np.isfinite(vs[:, good]))
    losses = np_out(out.losses)
    assert np.isnan(losses[:3]).all() and np.isfinite(losses[3])  # entropy ignores actions
    g = vt.vtrace_gather_logits(dev["target_logits"], dev["behaviour_logits"], dev["actions"])
    gb = g.cpu().numpy().view(np.uint32)
    assert gb[5, 3, 0] == 0xFFFFFFFF and gb[2, 7, 1] == 0xFFFFFFFF
    # a cleared workspace starts without the flag; valid data does not raise it
    ws2 = vt.Workspace(12, 10, 9)
    tr.actions[5, 3] = 0
    tr.actions[2, 7] = 0
    vt.vtrace_loss_grad(**to_device(tr), workspace=ws2)
    assert vt.vtrace_error_flag(ws2) == 0


@pytest.mark.parametrize("T,B,A", [(40, 64, 18), (1000, 16384, 18), (100, 4096, 9)])
def test_nonfinite_logit_rows_leave_the_other_lanes_exact(T, B, A):
    """A NaN target logit in one lane's row and a NaN behaviour logit in
    another's.  Those rows' statistics are NaN (so are the recursion's values
    at and before them, and the two lanes' losses), and every wave holding
    such a row forms its exponent sums with the terms clamped against
    non-finite logits; the other lanes of those waves, and all other lanes,
    still match the oracle element by element (shapes: 16-step tiles, the
    32 x 8 loss tiles of the stress batch, A = 9)."""
    tr = make_random(T, B, A, 1234, noise_std=1.0)
    bz, tz, by, ty = 5, T // 2, B - 3, T // 3
    tr.target_logits[tz, bz, 3] = np.nan
    tr.behaviour_logits[ty, by, A - 2] = np.nan
    p = PARAM_SETS[4][0]
    log_case(f"non-finite logits T={T} B={B} A={A}")
    out = run_loss_grad(to_device(tr), p)
    lane = np_out(out.lane_losses)
    assert np.isnan(lane[bz, 0]) and np.isnan(lane[by, 0])
    vs = np_out(out.vs)
    assert np.all(np.isnan(vs[:tz + 1, bz])) and np.all(np.isfinite(vs[tz + 1:, bz]))
    assert np.all(np.isnan(vs[:ty + 1, by])) and np.all(np.isfinite(vs[ty + 1:, by]))
    assert np.all(np.isnan(np_out(out.d_logits)[tz, bz]))
    # the lanes that share a 64-lane neighbourhood with the two rows (their
    # waves' other lanes in every tile shape), else a spread of lanes
    near = [b for b in list(range(0, 64)) + list(range(B - 64, B)) if b not in (bz, by)]
    lanes = sorted(set(near + (list(range(64, B - 64, max(1, (B - 128) // 64))) if B > 128 else [])))
    check_against_oracle(tr, p, out, lanes=lanes)


def test_deterministic_and_workspace_reuse():
    tr = make_config(3)
    dev = to_device(tr)
    ws = vt.Workspace(tr.T, tr.B, tr.A)
    p = PARAM_SETS[3][0]
    log_case("determinism, 30-task batch T=100 B=4096 A=9")
    a = run_loss_grad(dev, p, workspace=ws)
    b = run_loss_grad(dev, p, workspace=ws)
    for x, y in zip(a, b):
        assert np_out(x).tobytes() == np_out(y).tobytes()


@pytest.mark.parametrize("T,B,A", [(16, 4096, 9), (100, 4096, 9), (20, 24576, 18)])
def test_loss_reduction_across_back_to_back_calls(T, B, A):
    """The cross-workgroup loss reduction publishes each workgroup's partial
    before its ticket; a partial read before it landed would still hold the
    previous call's value.  Two different batches of the same shape alternate
    on one workspace, 200 calls back to back on one stream, each writing its
    own losses buffer: every call must reproduce its batch's losses bit for
    bit."""
    trs = [make_random(T, B, A, 4000 + k, noise_std=1.0, end_prob=0.03) for k in range(2)]
    devs = [to_device(tr) for tr in trs]
    p = PARAM_SETS[4][0]
    ws = vt.Workspace(T, B, A)
    log_case(f"back-to-back loss reductions T={T} B={B} A={A}")
    ref = [np_out(run_loss_grad(d, p, workspace=ws).losses) for d in devs]
    assert not np.array_equal(ref[0], ref[1])
    first = run_loss_grad(devs[0], p, workspace=ws)
    n = 200
    losses = [torch.empty(4, dtype=torch.float32, device="cuda") for _ in range(n)]
    for i in range(n):
        out = first._replace(losses=losses[i])
        vt.vtrace_loss_grad(**devs[i % 2], rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam,
                            baseline_cost=p.baseline_cost, entropy_cost=p.entropy_cost,
                            workspace=ws, out=out)
    torch.cuda.synchronize()
    for i in range(n):
        assert np_out(losses[i]).tobytes() == ref[i % 2].tobytes(), f"call {i}"


@pytest.mark.parametrize("T,B,A", [(100, 32, 9), (100, 4096, 9), (20, 16384, 18)])
def test_graph_capture_replays(T, B, A):
    """The call captured in a HIP graph (the time-parallel, tiled and
    multi-tile kernels by shape) and replayed several times, with eager calls
    on other inputs and synchronisations in between: every replay must equal
    the eager result bit for bit (the loss ticket rearms itself; nothing in
    the call is a memset)."""
    trs = [make_random(T, B, A, 5000 + k, noise_std=1.0, end_prob=0.03) for k in range(2)]
    devs = [to_device(tr) for tr in trs]
    p = PARAM_SETS[4][0]
    ws = vt.Workspace(T, B, A)
    log_case(f"graph capture T={T} B={B} A={A}")
    eager = run_loss_grad(devs[0], p, workspace=ws)
    ref = {k: np_out(getattr(eager, k)).tobytes() for k in ("losses", "d_logits", "d_values", "vs")}
    out = vt.vtrace_loss_grad(**devs[0], rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam,
                              with_vs=True, with_pg_advantages=True, with_lane_losses=True,
                              workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            vt.vtrace_loss_grad(**devs[0], rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam,
                                workspace=ws, out=out)
    torch.cuda.synchronize()
    for rep in range(4):
        for k in ("losses", "d_logits", "d_values", "vs"):
            getattr(out, k).fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        for k in ("losses", "d_logits", "d_values", "vs"):
            assert np_out(getattr(out, k)).tobytes() == ref[k], f"replay {rep}: {k}"
        other = run_loss_grad(devs[1], p, workspace=ws)  # eager work between replays
        assert not np.array_equal(np_out(other.losses), np_out(eager.losses))


def test_lane_permutation_is_bit_exact():
    tr = make_random(50, 96, 9, 8)
    perm = np.random.default_rng(0).permutation(96)
    p = PARAM_SETS[4][1]
    log_case("lane permutation")
    a = run_loss_grad(to_device(tr), p)
    b = run_loss_grad(to_device(subset_lanes(tr, perm)), p)
    for name in ("vs", "pg_advantages", "d_values", "d_logits"):
        x, y = np_out(getattr(a, name)), np_out(getattr(b, name))
        assert x[:, perm].tobytes() == y.tobytes(), name
    assert np_out(a.lane_losses)[perm].tobytes() == np_out(b.lane_losses).tobytes()


def test_episode_cut_is_bit_exact():
    T, B, A = 40, 33, 18
    tr = make_random(T, B, A, 21, end_prob=0.0)
    tcut = 17
    tr.discounts[tcut] = 0.0
    p = PARAM_SETS[4][1]
    log_case("episode cut")
    a = run_loss_grad(to_device(tr), p)
    other = make_random(T, B, A, 22)
    for name in ("target_logits", "behaviour_logits", "actions", "rewards", "discounts", "values"):
        arr = getattr(tr, name).copy()
        arr[tcut + 1:] = getattr(other, name)[tcut + 1:]
        setattr(tr, name, arr)
    tr.bootstrap_value = other.bootstrap_value
    b = run_loss_grad(to_device(tr), p)
    for name in ("vs", "pg_advantages", "d_values", "d_logits"):
        x, y = np_out(getattr(a, name)), np_out(getattr(b, name))
        assert x[:tcut + 1].tobytes() == y[:tcut + 1].tobytes(), name


def test_gradient_invariants():
    tr = make_random(30, 50, 18, 9, noise_std=1.0)
    dev = to_device(tr)
    p = type(PARAM_SETS[4][0])(1.0, 1.0, 1.0, 0.5, 0.0)
    log_case("gradient invariants (entropy cost 0)")
    out = run_loss_grad(dev, p)
    dl = np_out(out.d_logits).astype(np.float64)
    adv = np_out(out.pg_advantages).astype(np.float64)
    np.testing.assert_allclose(dl.sum(-1), 0.0, atol=1e-5 + 1e-5 * np.abs(adv).max())
    taken = np.take_along_axis(dl, tr.actions[..., None].astype(np.int64), -1)[..., 0]
    nz = adv != 0
    assert np.all(np.sign(taken[nz]) == -np.sign(adv[nz]))
    # shifting each row of target logits by a constant leaves everything unchanged
    shifted = tr.target_logits + np.float32(3.0)
    tr2 = make_random(30, 50, 18, 9, noise_std=1.0)
    tr2.target_logits = shifted
    tr2.behaviour_logits = tr.behaviour_logits + np.float32(-2.0)
    out2 = run_loss_grad(to_device(tr2), p)
    for name in ("vs", "pg_advantages", "d_values", "d_logits"):
        assert_close(f"shift {name}", np_out(getattr(out2, name)), np_out(getattr(out, name)))
    # a single action: no policy gradient
    tr1 = make_random(10, 8, 1, 10)
    out1 = run_loss_grad(to_device(tr1), PARAM_SETS[0][0])
    assert np.all(np_out(out1.d_logits) == 0.0)


@pytest.mark.parametrize("kernel", ["tiled", "wide"])
@pytest.mark.parametrize("pidx", [0, 1])
def test_kernels_agree(monkeypatch, pidx, kernel):
    """The tiled and the time-parallel kernel each give the generic lane-serial
    kernel's results: tightly where every weight is at most 1 (nothing
    amplifies rounding), to the oracle's tolerance where the weights are
    unclipped."""
    p = PARAM_SETS[4][pidx]
    tight = pidx == 0
    for (T, B, A, bf16) in [(100, 4096, 9, False), (60, 1000, 18, False), (50, 777, 9, True),
                            (40, 1000, 18, True), (20, 32, 18, True)]:
        tr = make_random(T, B, A, 31 + A, noise_std=1.0, bf16=bf16)
        dev = to_device(tr)
        log_case(f"kernel agreement {kernel} T={T} B={B} A={A} bf16={bf16} {p.label()}")
        monkeypatch.setenv("VTRACE_KERNEL", kernel)
        a = run_loss_grad(dev, p)
        monkeypatch.setenv("VTRACE_KERNEL", "lane_serial")
        b = run_loss_grad(dev, p)
        monkeypatch.delenv("VTRACE_KERNEL")
        for name in ("vs", "pg_advantages", "d_values", "d_logits"):
            kw = dict(rtol=2e-5, atol=2e-6) if tight else {}
            assert_close(f"{kernel} vs lane_serial {name}", np_out(getattr(a, name)),
                         np_out(getattr(b, name)), **kw)
        # loss sums cancel (advantages of both signs): the oracle's tolerance
        for name in ("lane_losses", "losses"):
            assert_close(f"{kernel} vs lane_serial {name}", np_out(getattr(a, name)),
                         np_out(getattr(b, name)))


def _bits(t):
    return t.view(torch.int16 if t.element_size() == 2 else torch.int32).cpu().numpy()


@pytest.mark.parametrize("A,bf16,grad", [(18, False, "float32"), (18, False, "bfloat16"),
                                         (9, True, "bfloat16"), (9, True, "float32")])
def test_multi_tile_walk_matches_single_tile(A, bf16, grad, monkeypatch):
    """With the 16-step tiles (VTRACE_KERNEL=tiled_short), a batch whose tile
    count is a whole multiple (at least two) of the workgroups the chip holds
    at once runs the tiled kernel's multi-tile walk (for the kernels that fit
    two or more workgroups per CU: fp32 logits with A = 18 and bf16 logits with
    A = 9; fp32 A = 9 takes 32-lane tiles at this size and bf16 A = 18 fits one
    workgroup per CU); on a 256-CU part B = 24576 is such a batch.
    Every per-step and per-lane output must be bit-identical to the walk with
    one workgroup per tile (the same arithmetic per lane; only the order of the
    batch totals differs), the totals must agree within the sum tolerance, and
    sampled lanes must match the oracle.  The targets-only call likewise."""
    T, B = 40, 24576
    tr = make_random(T, B, A, 77 + A, noise_std=1.0, end_prob=0.02, bf16=bf16)
    dev = to_device(tr)
    gd = torch.bfloat16 if grad == "bfloat16" else torch.float32
    lanes = sorted(set([0, 1, 15, 16, 17, B // 3, B // 2, B - 17, B - 16, B - 1]
                       + list(range(511, B, 4093))))
    for p in (PARAM_SETS[4][0], PARAM_SETS[4][2]):
        log_case(f"multi-tile walk T={T} B={B} A={A} bf16={bf16} grad={grad} {p.label()}")
        monkeypatch.setenv("VTRACE_KERNEL", "tiled_short")
        a = run_loss_grad(dev, p, grad_dtype=gd)
        ta = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
        monkeypatch.setenv("VTRACE_KERNEL", "tiled_short_single")
        b = run_loss_grad(dev, p, grad_dtype=gd)
        tb = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
        torch.cuda.synchronize()
        monkeypatch.delenv("VTRACE_KERNEL")
        for name in ("vs", "pg_advantages", "d_values", "d_logits", "lane_losses"):
            x, y = getattr(a, name), getattr(b, name)
            assert np.array_equal(_bits(x), _bits(y)), f"{name} differs between the two walks"
        for x, y in zip(ta, tb):
            assert np.array_equal(_bits(x), _bits(y)), "targets differ between the two walks"
        assert_close("losses, multi vs single", np_out(a.losses), np_out(b.losses), rtol=1e-4,
                     atol=1e-3)
        lane = np_out(a.lane_losses).astype(np.float64)
        assert_close("losses vs lane sums", np_out(a.losses)[1:].astype(np.float64),
                     lane.sum(axis=0), rtol=1e-4, atol=1e-3)
        if gd == torch.float32:
            check_against_oracle(tr, p, a, lanes=lanes)
    del dev
    torch.cuda.empty_cache()


OTHER_ACTION_COUNTS = [2, 3, 4, 5, 6, 7, 8, 10, 11, 12, 13, 14, 15, 16, 17, 19, 20]


@pytest.mark.parametrize("A", OTHER_ACTION_COUNTS)
def test_tiled_other_action_counts(A, monkeypatch):
    """Every action count 2 <= A <= 20 takes the tiled kernel: ragged shapes
    against the oracle (fp32 and bf16 logits, weights clipped at 1 and
    unclipped), and a 16384-lane batch (which takes the multi-tile walk where
    it fits) against the generic lane-serial kernel and, on sampled lanes, the
    oracle."""
    for bf16 in (False, True):
        tr = make_random(37, 45, A, 1100 + A, noise_std=1.0, end_prob=0.05, bf16=bf16)
        for p in (PARAM_SETS[4][0], PARAM_SETS[4][1]):
            log_case(f"tiled A={A} T=37 B=45 bf16={bf16} {p.label()}")
            check_against_oracle(tr, p, run_loss_grad(to_device(tr), p))
    T, B = 20, 16384
    tr = make_random(T, B, A, 1200 + A, noise_std=1.0, end_prob=0.03)
    dev = to_device(tr)
    p = PARAM_SETS[4][0]
    log_case(f"tiled A={A} T={T} B={B} against lane_serial")
    monkeypatch.delenv("VTRACE_KERNEL", raising=False)
    a = run_loss_grad(dev, p)
    check_against_oracle(tr, p, a, lanes=[0, 15, 16, B // 2, B - 1])
    monkeypatch.setenv("VTRACE_KERNEL", "lane_serial")
    b = run_loss_grad(dev, p)
    monkeypatch.delenv("VTRACE_KERNEL")
    for name in ("vs", "pg_advantages", "d_values", "d_logits"):
        assert_close(f"A={A} tiled vs lane_serial {name}", np_out(getattr(a, name)),
                     np_out(getattr(b, name)), rtol=2e-5, atol=2e-6)
    for name in ("lane_losses", "losses"):
        assert_close(f"A={A} tiled vs lane_serial {name}", np_out(getattr(a, name)),
                     np_out(getattr(b, name)))


@pytest.mark.parametrize("T,B", [(40, 8192), (33, 24576 + 32), (17, 65536)])
def test_wide_tiles_for_nine_actions(T, B, monkeypatch):
    """fp32 logits with A = 9 take 32-lane tiles once they cover every CU
    (B >= 8192 on a 256-CU part): the same results as the generic lane-serial
    kernel (tightly, weights <= 1) and, on sampled lanes, as the oracle."""
    A = 9
    tr = make_random(T, B, A, 700 + T, noise_std=1.0, end_prob=0.03)
    dev = to_device(tr)
    for p in (PARAM_SETS[4][0], PARAM_SETS[4][1]):
        log_case(f"32-lane tiles T={T} B={B} A={A} {p.label()}")
        monkeypatch.delenv("VTRACE_KERNEL", raising=False)
        a = run_loss_grad(dev, p)
        check_against_oracle(tr, p, a, lanes=[0, 31, 32, B // 2, B - 33, B - 1])
        if p is PARAM_SETS[4][0]:
            monkeypatch.setenv("VTRACE_KERNEL", "lane_serial")
            b = run_loss_grad(dev, p)
            monkeypatch.delenv("VTRACE_KERNEL")
            for name in ("vs", "pg_advantages", "d_values", "d_logits"):
                assert_close(f"32-lane vs lane_serial {name}", np_out(getattr(a, name)),
                             np_out(getattr(b, name)), rtol=2e-5, atol=2e-6)
            for name in ("lane_losses", "losses"):
                assert_close(f"32-lane vs lane_serial {name}", np_out(getattr(a, name)),
                             np_out(getattr(b, name)))
    del dev
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T", [1, 5, 16, 17, 33])
def test_multi_tile_walk_unroll_lengths(T, monkeypatch):
    """The multi-tile walk where a tile is one chunk (T <= 16: its carry reset
    and its lane totals fall in the same iteration), exactly one chunk, and a
    ragged second or third chunk: bit-identical to one workgroup per tile, and
    sampled lanes against the oracle."""
    B, A = 24576, 18
    tr = make_random(T, B, A, 500 + T, noise_std=1.0, end_prob=0.05)
    dev = to_device(tr)
    p = PARAM_SETS[4][0]
    log_case(f"multi-tile walk T={T} B={B} A={A}")
    monkeypatch.setenv("VTRACE_KERNEL", "tiled_short")
    a = run_loss_grad(dev, p)
    monkeypatch.setenv("VTRACE_KERNEL", "tiled_short_single")
    b = run_loss_grad(dev, p)
    monkeypatch.delenv("VTRACE_KERNEL")
    for name in ("vs", "pg_advantages", "d_values", "d_logits", "lane_losses"):
        assert np.array_equal(_bits(getattr(a, name)), _bits(getattr(b, name))), name
    check_against_oracle(tr, p, a, lanes=[0, 15, 16, 8191, 8192, B - 17, B - 1])


@pytest.mark.parametrize("A,bf16", [(18, False), (9, False), (18, True), (9, True)])
@pytest.mark.parametrize("lanes_per_cu", [64, 128, 192, 256])
def test_long_run_tile_shapes(A, bf16, lanes_per_cu, monkeypatch):
    """Batches of 64, 128, 192 and 256 lanes per CU take the long-run tile
    shapes: the loss call with A = 18 the 32 x 8 loss tiles (one to four
    whole generations of them), with A = 9 64 x 4 (128 and 256 lanes per CU)
    or 32 x 8 (64 and 192 lanes per CU), the targets-only
    call in the float32 ratio mode 64 x 8, 128 x 4 or 64 x 4 lanes x steps per
    chunk (32 x 8 or 64 x 4 for bf16 logits with A = 9; 64 x 4 through the
    multi-tile walk where the batch is a whole number of its generations; 192
    lanes per CU as three generations of 64 x 8 for fp32 logits), and with
    unclipped weights (float64 sums) the 16-step tiles.  T = 37 leaves every
    chunk length a ragged last chunk.  Every output against the oracle, with
    weights clipped at 1, with (1, 0.5, 0.95) and unclipped; the targets-only
    call against the oracle; the 16-step tiles (VTRACE_KERNEL=tiled_short)
    within the tolerance; and one workgroup per tile (tiled_single, the same
    shape without the multi-tile walk) bit-identical per step and per lane."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T, B = 37, lanes_per_cu * cus
    tr = make_random(T, B, A, 3000 + A + lanes_per_cu, noise_std=1.0, end_prob=0.03, bf16=bf16)
    dev = to_device(tr)
    for p in (PARAM_SETS[4][0], PARAM_SETS[4][2], PARAM_SETS[4][1]):
        log_case(f"long-run tiles T={T} B={B} A={A} bf16={bf16} {p.label()}")
        monkeypatch.delenv("VTRACE_KERNEL", raising=False)
        a = run_loss_grad(dev, p)
        o = check_against_oracle(tr, p, a)
        tv, tp = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
        torch.cuda.synchronize()
        assert_close("targets vs", np_out(tv), o.vs)
        assert_close("targets pg_advantages", np_out(tp), o.pg_advantages)
        monkeypatch.setenv("VTRACE_KERNEL", "tiled_short")
        b = run_loss_grad(dev, p)
        monkeypatch.setenv("VTRACE_KERNEL", "tiled_single")
        c = run_loss_grad(dev, p)
        monkeypatch.delenv("VTRACE_KERNEL")
        for name in ("vs", "pg_advantages", "d_values", "d_logits"):
            assert_close(f"long-run vs 16-step tiles {name}", np_out(getattr(a, name)),
                         np_out(getattr(b, name)), rtol=2e-5, atol=2e-6)
        for name in ("vs", "pg_advantages", "d_values", "d_logits", "lane_losses"):
            assert np.array_equal(_bits(getattr(a, name)), _bits(getattr(c, name))), \
                f"{name} differs between the multi-tile walk and one workgroup per tile"
    del dev
    torch.cuda.empty_cache()


@pytest.mark.parametrize("lanes_per_cu,T", [(64, 1), (64, 7), (64, 8), (64, 9), (128, 1), (128, 3),
                                             (128, 4), (128, 5), (256, 1), (256, 4), (256, 5)])
def test_long_run_tile_shapes_short_unrolls(lanes_per_cu, T, monkeypatch):
    """Unrolls of at most one chunk of the long-run shapes (fp32 logits, A = 18:
    64 x 8 at 64 lanes per CU, 128 x 4 at 128, 64 x 4 with the multi-tile walk
    at 256), exactly one chunk, and one step more: the only chunk starting
    before t = 0, and in the multi-tile walk a tile's carry reset and lane
    totals in the same iteration.  Every output against the oracle, and the
    multi-tile walk bit-identical per step and per lane to one workgroup per
    tile."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    A, B = 18, lanes_per_cu * cus
    tr = make_random(T, B, A, 3100 + T + lanes_per_cu, noise_std=1.0, end_prob=0.05)
    dev = to_device(tr)
    p = PARAM_SETS[4][0]
    log_case(f"long-run tiles, short unroll T={T} B={B} A={A}")
    monkeypatch.delenv("VTRACE_KERNEL", raising=False)
    a = run_loss_grad(dev, p)
    check_against_oracle(tr, p, a)
    monkeypatch.setenv("VTRACE_KERNEL", "tiled_single")
    b = run_loss_grad(dev, p)
    monkeypatch.delenv("VTRACE_KERNEL")
    for name in ("vs", "pg_advantages", "d_values", "d_logits", "lane_losses"):
        assert np.array_equal(_bits(getattr(a, name)), _bits(getattr(b, name))), name
    del dev
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,B,A,bf16", [(512, 4096, 18, False), (513, 4096, 18, False), (544, 4091, 18, True),
                                         (1000, 2048, 18, False), (543, 1000, 18, True)])
def test_two_row_chunks(T, B, A, bf16):
    """Long unrolls of at most 16 lanes per CU take tiles of 8 lanes by 32 steps
    (two lanes per wave, each on two DPP rows joined by one cross-row step of
    the scan), or fewer lanes by more steps: whole chunks, one step more than
    whole chunks, a last lane tile moved back over its neighbour, bf16 logits,
    every output against the oracle, for the loss call and the targets-only
    call."""
    tr = make_random(T, B, A, 5100 + T + B, noise_std=1.0, end_prob=0.02, bf16=bf16)
    dev = to_device(tr)
    p = PARAM_SETS[4][1] if T == 513 else PARAM_SETS[4][0]
    log_case(f"32-step chunks T={T} B={B} A={A} bf16={bf16}")
    check_against_oracle(tr, p, run_loss_grad(dev, p))
    vs, pg = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
    torch.cuda.synchronize()
    q = call_params(p)
    ot = oracle.vtrace(*oracle_args(tr), q.rho_bar, q.c_bar, q.lam)
    assert_close("targets.vs", np_out(vs), ot.vs)
    assert_close("targets.pg_advantages", np_out(pg), ot.pg_advantages)
    del dev
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kernel", ["tiled", "wide"])
@pytest.mark.parametrize("cfg,bf16", [(0, False), (1, False), (2, False), (3, False), (3, True),
                                      (2, True)])
def test_config_each_kernel(cfg, bf16, kernel, monkeypatch):
    """Configs 0-3 through each of the two fast kernels (the automatic choice
    takes the time-parallel one for configs 0-2, the tiled one for config 3)."""
    monkeypatch.setenv("VTRACE_KERNEL", kernel)
    tr = make_config(cfg, bf16=bf16)
    dev = to_device(tr)
    for p in (PARAM_SETS[cfg][0], PARAM_SETS[4][1], PARAM_SETS[4][2]):
        log_case(f"config {cfg} bf16={bf16} kernel={kernel} {p.label()}")
        check_against_oracle(tr, p, run_loss_grad(dev, p))


# (T, B, A, bf16 logits, kernel the automatic choice takes): the paper's
# learner batches and shapes on both sides of the measured crossover, each
# with a different workgroup count under the two kernels.
CHOICE_CASES = [(100, 32, 9, False, "wide"), (20, 32, 18, False, "wide"), (48, 8, 18, False, "wide"),
                (64, 1024, 18, False, "wide"), (16, 32, 18, True, "tiled"), (64, 1024, 9, False, "tiled"),
                (100, 4096, 9, False, "tiled"), (300, 32, 9, False, "tiled")]
_PARTIAL_SENTINEL = 0x7FF4DEADBEEF0001  # a NaN no partial sum can take


def _call_counting_workgroups(dev, p, T, B, A):
    """One loss call on a fresh workspace whose partials are preset to a
    sentinel; returns the outputs and the number of workgroups that wrote a
    loss partial.  (The workspace is a 256-byte header followed by three
    float64 partials per workgroup, the layout VTRACE_STATIC_WORKSPACE_BYTES
    states; a single-workgroup grid writes none.)"""
    ws = vt.Workspace(T, B, A, device="cuda")
    parts = ws.tensor[256:].view(torch.int64)
    parts.fill_(_PARTIAL_SENTINEL)
    out = run_loss_grad(dev, p, workspace=ws)
    written = int((parts != _PARTIAL_SENTINEL).sum().item())
    assert written % 3 == 0
    return out, written // 3


@pytest.mark.parametrize("T,B,A,bf16,kernel", CHOICE_CASES)
def test_automatic_kernel_choice(T, B, A, bf16, kernel, monkeypatch):
    """The automatic choice between the time-parallel and the tiled kernel.
    The two give the same float32 outputs (their float64 sums differ only far
    below float32 resolution), so they are told apart by their grids: the
    automatic call runs as many workgroups as the forced kernel and a
    different number from the other one, and matches the forced kernel bit
    for bit."""
    tr = make_random(T, B, A, 7000 + T + B + A, noise_std=1.0, end_prob=0.02, bf16=bf16)
    dev = to_device(tr)
    p = PARAM_SETS[4][0]
    log_case(f"kernel choice T={T} B={B} A={A} bf16={bf16} -> {kernel}")
    monkeypatch.delenv("VTRACE_KERNEL", raising=False)
    auto, n_auto = _call_counting_workgroups(dev, p, T, B, A)
    monkeypatch.setenv("VTRACE_KERNEL", kernel)
    forced, n_forced = _call_counting_workgroups(dev, p, T, B, A)
    if T <= 256:
        monkeypatch.setenv("VTRACE_KERNEL", "tiled" if kernel == "wide" else "wide")
        _, n_other = _call_counting_workgroups(dev, p, T, B, A)
        assert n_other != n_forced, "the two kernels run as many workgroups: the case cannot tell them apart"
    monkeypatch.delenv("VTRACE_KERNEL")
    assert n_auto == n_forced, f"the automatic call ran {n_auto} workgroups, the {kernel} kernel {n_forced}"
    for name in ("vs", "pg_advantages", "d_values", "d_logits", "lane_losses", "losses"):
        assert np.array_equal(_bits(getattr(auto, name)), _bits(getattr(forced, name))), name


WIDE_SHAPES = [(1, 1, 9), (1, 300, 18), (16, 16, 18), (17, 7, 9), (31, 5, 18), (64, 9, 9),
               (100, 33, 18), (128, 4, 9), (129, 3, 9), (200, 2, 18), (256, 3, 9), (255, 1, 18)]


@pytest.mark.parametrize("T,B,A", WIDE_SHAPES)
def test_wide_kernel_shapes(T, B, A, monkeypatch):
    """The time-parallel kernel at every lane packing (T up to 16, 32, ..., 256:
    16 to 1 lanes per workgroup), ragged T and B, fp32 and bf16 logits."""
    monkeypatch.setenv("VTRACE_KERNEL", "wide")
    for bf16 in (False, True):
        tr = make_random(T, B, A, 2000 + T + B + A, noise_std=1.0, end_prob=0.05, bf16=bf16)
        for p in (PARAM_SETS[4][0], PARAM_SETS[4][1]):
            log_case(f"wide T={T} B={B} A={A} bf16={bf16} {p.label()}")
            check_against_oracle(tr, p, run_loss_grad(to_device(tr), p))


@pytest.mark.parametrize("B", [(1 << 20) + 8, 1 << 20])
def test_offsets_beyond_four_gib(B):
    """Logit tensors larger than 2^32 bytes (T=64, B=2^20+8 or 2^20, A=18:
    4.8 GB each): byte offsets need more than 32 bits, signed or not.  With
    2^20 + 8 lanes the 16-step tiles run it, the last one moved back by half a
    tile; 2^20 lanes are a whole
    number of generations of the 64 x 4 long-run tiles, which take the
    multi-tile walk (on a 256-CU part).  The oracle checks lanes spread over
    the batch, including the last ones, whose elements lie beyond 2^32 bytes."""
    T, A = 64, 18
    assert T * B * A * 4 > 2**32
    log_case(f"large batch T={T} B={B} A={A} ({T * B * A * 4 / 2**30:.2f} GiB per logit tensor)")
    tr = make_random(T, B, A, 4321, noise_std=1.0, end_prob=0.01)
    dev = to_device(tr)
    lanes = sorted(set([0, 1, B // 2, B - 17, B - 9, B - 8, B - 2, B - 1] + list(range(B - 64, B, 7))))
    for p in (PARAM_SETS[4][0], PARAM_SETS[4][1]):
        out = run_loss_grad(dev, p)
        check_against_oracle(tr, p, out, lanes=lanes)
        del out
    del dev
    torch.cuda.empty_cache()
