"""GPU parity of the tiled kernel's shapes for small and ragged batches: 8, 4, 2
and 1 lanes by 32, 64, 128 and 256 steps, and time rows that start at any
alignment.  Each batch has a last tile moved back over the tile before it; its
shared lanes must be written right and counted once in the loss totals.  Sizes
are the edges of the chunks (one step more than whole chunks, one chunk cut
short) and odd action counts, whose rows allow only 4- and 8-byte vectors.
Element-wise bound 1e-5 + 1e-4 |o|, as for every other kernel; the totals
against the float64 sum of the lane losses (each rounded to float32, 2^-24, in a
sum of at most 3601 of them: within 1e-5 of their root-sum-square)."""

import math

import numpy as np
import pytest
import torch

import oracle
import paper_1802_01561_amd as vt
from gpu_util import assert_close, call_params, log_case, np_out, oracle_args, require_gpu, to_device
from synth import Params, make_random, subset_lanes
from test_gpu_parity import check_against_oracle, run_loss_grad
from test_gpu_variants import check_io_variant

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# (T, B): on a 256-CU part 1, 1, 2, 2, 4, 8 and 16 lanes per tile.
SHAPES = [(257, 37), (600, 3), (100, 37), (385, 461), (321, 901), (97, 1803), (33, 3601)]


@pytest.mark.parametrize("T,B", SHAPES)
@pytest.mark.parametrize("A,bf16", [(2, True), (3, False), (7, True), (9, False), (13, True), (18, False), (20, True)])
def test_shapes(T, B, A, bf16):
    tr = make_random(T, B, A, 9000 + T + B + A, noise_std=1.0, end_prob=0.03, bf16=bf16)
    dev = to_device(tr)
    lanes = sorted({0, 1, B // 2, *range(max(0, B - 20), B)})
    for p in (Params(1.0, 1.0, 1.0), Params(1.0, 0.5, 0.95)):
        log_case(f"tile shapes T={T} B={B} A={A} bf16={bf16} {p.label()}")
        out = run_loss_grad(dev, p)
        check_against_oracle(tr, p, out, lanes=lanes)
        lane = np_out(out.lane_losses).astype(np.float64)
        rss = np.sqrt((lane ** 2).sum(axis=0))
        assert np.all(np.abs(np_out(out.losses)[1:] - lane.sum(axis=0)) <= 1e-5 * rss + 1e-5)
        vs, pg = vt.vtrace_targets(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam)
        q = call_params(p)
        o = oracle.vtrace(*oracle_args(subset_lanes(tr, lanes)), q.rho_bar, q.c_bar, q.lam)
        assert_close("targets.vs", np_out(vs)[:, lanes], o.vs)
        assert_close("targets.pg_advantages", np_out(pg)[:, lanes], o.pg_advantages)


# Both sides of the lines between 8, 16 and 32 lanes (on a 256-CU part).
@pytest.mark.parametrize("T,B,A,bf16", [(125, 4093, 4, False), (100, 4090, 8, False), (100, 4096, 9, False),
                                        (48, 4096, 18, True), (300, 8200, 10, False), (340, 9001, 9, True),
                                        (64, 24600, 5, False), (20, 4096, 15, True), (16, 7999, 9, False),
                                        (9, 16001, 9, False), (17, 8192, 9, False), (130, 15900, 9, False)])
def test_shapes_of_full_chips(T, B, A, bf16):
    test_shapes(T, B, A, bf16)


@pytest.mark.parametrize("T,B", [(257, 37), (385, 461), (70, 9), (40, 19)])
@pytest.mark.parametrize("correction,log_probs,transform", [("vtrace", True, "clip"), ("epsilon", False, None),
                                                            ("one_step_is", False, "asymmetric")])
def test_variants(T, B, correction, log_probs, transform):
    for A, bf16 in ((5, True), (9, False), (18, True)):
        tr = make_random(T, B, A, 9100 + T + B + A, noise_std=1.0, end_prob=0.03, bf16=bf16)
        tr.rewards = (tr.rewards * 2.5).astype(np.float32)
        log_case(f"tile shapes T={T} B={B} A={A} bf16={bf16} {correction} lp={log_probs} r={transform}")
        check_io_variant(tr, Params(2.0, 1.0, 0.9), correction=correction, log_probs=log_probs,
                         reward_transform=transform, grad_bf16=True)


@pytest.mark.parametrize("T,B,log_probs,bf16", [(20, 16384, True, False), (17, 32768, False, True),
                                                (9, 49152, True, True), (5, 65536, False, False)])
def test_whole_generations_of_two_or_three(T, B, log_probs, bf16):
    """A = 9 batches that are whole generations of two workgroups a CU, or of the
    three that fit some of the long-run kernels."""
    tr = make_random(T, B, 9, 9150 + T, noise_std=1.0, end_prob=0.03, bf16=bf16)
    log_case(f"long-run tiles T={T} B={B} lp={log_probs} bf16={bf16}")
    check_io_variant(tr, Params(1.0, 1.0, 1.0), log_probs=log_probs, reward_transform="clip", grad_bf16=bf16,
                     lanes=[0, 1, 31, 32, B // 2, B // 3, B - 33, B - 1])


@pytest.mark.parametrize("T,B,A", [(300, 40, 9), (385, 461, 7)])
def test_unclipped_weights_and_replays(T, B, A):
    """(inf, inf, 1) through several waves per lane, and the captured call equal
    to the eager one bit for bit on every replay."""
    tr = make_random(T, B, A, 9200 + T, noise_std=0.3, end_prob=0.05)
    dev = to_device(tr)
    p = Params(math.inf, math.inf, 1.0)
    ws = vt.Workspace(T, B, A)
    log_case(f"tile shapes T={T} B={B} A={A} unclipped, captured")
    eager = run_loss_grad(dev, p, workspace=ws)
    check_against_oracle(tr, p, eager)
    out = run_loss_grad(dev, p, workspace=ws)
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            vt.vtrace_loss_grad(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam, workspace=ws, out=out)
    for _ in range(3):
        for x in out:
            x.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        for name, x, y in zip(out._fields, out, eager):
            assert torch.equal(x, y), name
        run_loss_grad(dev, Params(1.0, 1.0, 1.0), workspace=ws)  # eager work between replays


@pytest.mark.parametrize("T,B,A,bf16,variant", [
    (18, 2 ** 22 + 37, 18, False, {}),
    (5, 2 ** 26 // 20 + 3, 20, True, dict(grad_dtype=torch.bfloat16)),
    (37, 2 ** 25 + 1, 2, False, {}),  # the loss call tiled, the targets one thread per lane
    (8, 2 ** 23 + 5, 9, False, dict(behaviour="log_probs", reward_transform="clip")),
    (2, 2 ** 23 + 5, 9, True, {})])  # one thread per lane
def test_time_rows_beyond_32_bit_offsets(T, B, A, bf16, variant):
    """Time rows of 2^26 elements or more, 16 of which 32-bit byte offsets do not
    reach: chosen lanes against the oracle, the totals against the lane losses."""
    log_case(f"far rows T={T} B={B} A={A} bf16={bf16} {variant}")
    g = torch.Generator(device="cuda").manual_seed(9300 + A)
    f = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    log_probs = variant.get("behaviour") == "log_probs"
    x = dict(target_logits=f(T, B, A), behaviour_logits=-f(T, B).abs() - 0.5 if log_probs else f(T, B, A),
             actions=torch.randint(0, A, (T, B), generator=g, device="cuda", dtype=torch.int32), rewards=f(T, B),
             discounts=torch.where(f(T, B) > 1.5, 0.0, 0.99), values=f(T, B), bootstrap_value=f(B))
    if bf16:
        x.update(target_logits=x["target_logits"].bfloat16(), behaviour_logits=x["behaviour_logits"].bfloat16())
    lanes = sorted({0, 1, 15, 16, B // 2, B // 3, *range(B - 20, B)})
    at = torch.tensor(lanes, device="cuda")
    p = call_params(Params(1.0, 1.0, 0.9))
    out = run_loss_grad(x, p, **variant)
    vs, pg = vt.vtrace_targets(**x, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam,
                               **{k: v for k, v in variant.items() if k != "grad_dtype"})
    pick = lambda t: t.index_select(0 if t.dim() == 1 else 1, at).cpu()  # noqa: E731
    args = [pick(t).float().numpy() if t.is_floating_point() else pick(t).numpy() for t in x.values()]
    o = oracle.loss_and_grads(*args, p.rho_bar, p.c_bar, p.lam, p.baseline_cost, p.entropy_cost,
                              **{k: v for k, v in variant.items() if k != "grad_dtype"})
    rel = 2.0 ** -8 if "grad_dtype" in variant else 1e-4
    for name, t, e in (("vs", out.vs, o.vs), ("pg_advantages", out.pg_advantages, o.pg_advantages),
                       ("d_values", out.d_values, o.d_values), ("targets.vs", vs, o.vs),
                       ("targets.pg_advantages", pg, o.pg_advantages)):
        assert_close(name, pick(t).numpy(), e)
    assert_close("d_logits", pick(out.d_logits).float().numpy(), o.d_logits, rtol=rel)
    assert_close("lane_losses", out.lane_losses[at].cpu().numpy(), o.lane_losses)
    sums = out.lane_losses.double().sum(0).cpu().numpy()
    rss = out.lane_losses.double().square().sum(0).sqrt().cpu().numpy()
    assert np.all(np.abs(np_out(out.losses)[1:] - sums) <= 1e-5 * rss + 1e-4 * np.abs(sums))
