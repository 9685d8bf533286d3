"""The binding's native marshalling (csrc/fast_call.cpp) against its Python path:
the same results bit for bit, the same errors, and everything unusual left to the
Python path."""

import warnings

import numpy as np
import pytest
import torch
from torch.overrides import TorchFunctionMode

import paper_1802_01561_amd as vt
from paper_1802_01561_amd import binding


def _loss_args(device, T=5, B=6, A=9, dtype=torch.float32):
    g = torch.Generator().manual_seed(1)
    f = lambda *s: torch.randn(*s, generator=g).to(device)  # noqa: E731
    x = dict(target_logits=f(T, B, A).to(dtype), behaviour_logits=f(T, B, A).to(dtype),
             actions=torch.randint(0, A, (T, B), generator=g, dtype=torch.int32).to(device), rewards=f(T, B),
             discounts=torch.full((T, B), 0.99).to(device), values=f(T, B), bootstrap_value=f(B))
    e = dict(dtype=torch.float32, device=device)
    out = vt.LossGrad(torch.empty(4, **e), torch.empty((T, B, A), **e), torch.empty((T, B), **e),
                      torch.empty((T, B), **e), None, torch.empty((B, 3), **e))
    return x, out


class _NoWorkspace(vt.Workspace):
    def __init__(self):
        self.tensor, self.nbytes = torch.empty(4096, dtype=torch.uint8), 4096


def test_host_tensors_are_declined():
    x, out = _loss_args("cpu")
    assert binding._fast_call(x["target_logits"]) is None
    ws = _NoWorkspace()
    with pytest.raises(ValueError, match="GPU"):
        vt.vtrace_loss_grad(**x, out=out, workspace=ws)


def _gpu_stand_in(monkeypatch):
    """Stands in for a GPU tensor, which this machine may not have."""
    x = type("Tensor", (), {"is_cuda": True})()
    monkeypatch.setattr(binding.torch, "Tensor", type(x))
    return x


def test_without_the_extension_calls_take_the_python_path(monkeypatch):
    """A tree with the library alone (or an extension built against another torch)
    still runs every call; the loader's reason is told once."""
    def fails(self):
        raise ImportError("undefined symbol: of another torch")
    x = _gpu_stand_in(monkeypatch)
    monkeypatch.setattr(binding, "_fast", None)
    monkeypatch.setattr(binding._FastCall, "__init__", fails)
    with pytest.warns(RuntimeWarning, match="undefined symbol"):
        assert binding._fast_call(x) is None
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert binding._fast_call(x) is None


def test_variant_settings_are_bounded_and_exact():
    binding._variants.clear()
    key = ("epsilon", "vtrace", 1e-3, "log_probs", "clip", torch.bfloat16)
    v, address, log_probs, bf16 = binding._fast_variant(*key)
    assert (v.correction, v.behaviour_input, v.reward_transform, v.grad_dtype) == (2, 1, 1, 1)
    assert np.float32(v.epsilon) == np.float32(1e-3) and log_probs and bf16 and address
    assert binding._fast_variant(*key)[1] == address
    assert binding._fast_variant("epsilon", "vtrace", torch.tensor(1e-3), "logits", None, torch.float32) is None
    assert binding._fast_variant("epsilon", "vtrace", np.array(1e-3), "logits", None, torch.float32) is None
    with pytest.raises(ValueError):
        binding._fast_variant("nonsense", "vtrace", 1e-6, "logits", None, torch.float32)
    for i in range(3 * binding._MOST_VARIANTS):
        binding._fast_variant("epsilon", "vtrace", 1.0 + i, "logits", None, torch.float32)
    assert len(binding._variants) <= binding._MOST_VARIANTS


class _Subclass(torch.Tensor):
    pass


class _Mode(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def _count(monkeypatch):
    """Counts the native calls that launched, and those that declined."""
    fast = binding._fast_call(torch.empty(1, device="cuda"))
    seen = {"ran": 0, "declined": 0}
    for name in ("call_loss", "call_targets", "call_head"):
        def counted(*args, _f=getattr(fast, name)):
            status = _f(*args)
            seen["declined" if status is None else "ran"] += 1
            return status
        monkeypatch.setattr(fast, name, counted)
    return seen


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_same_results_as_the_python_path(dtype, monkeypatch):
    print(f"[case] fast call {dtype}", flush=True)
    x, out = _loss_args("cuda", 20, 7, 9, dtype)
    ws = vt.Workspace(20, 7, 9)
    seen = _count(monkeypatch)
    assert vt.vtrace_loss_grad(**x, c_bar=0.5, lam=0.95, out=out, workspace=ws) is out
    fast = [None if t is None else t.clone() for t in out]
    vs, pg = torch.empty_like(x["values"]), torch.empty_like(x["values"])
    vt.vtrace_targets(**x, vs=vs, pg_advantages=pg)
    fast += [vs.clone(), pg.clone()]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        vt.vtrace_targets(**x, vs=vs, pg_advantages=pg, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(vs, fast[-2]) and seen == {"ran": 3, "declined": 0}
    monkeypatch.setattr(binding, "_fast_call", lambda first: None)
    vt.vtrace_loss_grad(**x, c_bar=0.5, lam=0.95, out=out, workspace=ws)
    vt.vtrace_targets(**x, vs=vs, pg_advantages=pg)
    torch.cuda.synchronize()
    assert seen["ran"] == 3
    for a, b in zip(fast, [*out, vs, pg]):
        assert (a is None and b is None) or torch.equal(a, b)


VARIANTS = [
    dict(behaviour="log_probs", reward_transform="clip"),
    dict(grad_dtype=torch.bfloat16, reward_transform="asymmetric"),
    dict(behaviour="log_probs", grad_dtype=torch.bfloat16, correction="one_step_is", q_estimate="baseline"),
    dict(correction="epsilon", epsilon=1e-2)]
SCALARS = dict(rho_bar=1.5, c_bar=0.75, lam=0.9)
COSTS = dict(baseline_cost=0.7, entropy_cost=0.03)


def _both_paths(monkeypatch, calls):
    """Each call's outputs by the native marshalling (which must take all of them)
    and by the Python path, in the same buffers."""
    seen = _count(monkeypatch)
    results = []
    for path in ("native", "python"):
        if path == "python":
            monkeypatch.setattr(binding, "_fast_call", lambda first: None)
        got = []
        for call in calls:
            out = call()
            torch.cuda.synchronize()
            got += [None if t is None else t.clone() for t in out]
            for t in out:
                if t is not None:
                    t.fill_(-7.0)
        results.append(got)
    assert seen == {"ran": len(calls), "declined": 0}
    for i, (a, b) in enumerate(zip(*results)):
        assert (a is None and b is None) or torch.equal(a, b), i


@pytest.mark.gpu
@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("optional", [False, True])
def test_variants_as_the_python_path(variant, dtype, optional, monkeypatch):
    print(f"[case] fast call {variant} {dtype} optional outputs={optional}", flush=True)
    T, B, A = 20, 7, 9
    x, out = _loss_args("cuda", T, B, A, dtype)
    if variant.get("behaviour") == "log_probs":
        x["behaviour_logits"] = -x["rewards"].abs() - 0.5
    out = out._replace(d_logits=out.d_logits.to(variant.get("grad_dtype", torch.float32)),
                       vs=torch.empty_like(x["values"]) if optional else None,
                       pg_advantages=torch.empty_like(x["values"]) if optional else None,
                       lane_losses=out.lane_losses if optional else None)
    ws = vt.Workspace(T, B, A)
    vs, pg = torch.empty_like(x["values"]), torch.empty_like(x["values"])
    of_targets = {k: v for k, v in variant.items() if k != "grad_dtype"}
    _both_paths(monkeypatch, [
        lambda: vt.vtrace_loss_grad(**x, **SCALARS, **COSTS, **variant, out=out, workspace=ws),
        lambda: vt.vtrace_targets(**x, **SCALARS, **of_targets, vs=vs, pg_advantages=pg, workspace=ws)])


@pytest.mark.gpu
@pytest.mark.parametrize("variant", [{}, *VARIANTS])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("optional", [False, True])
def test_output_layer_as_the_python_path(variant, dtype, optional, monkeypatch):
    print(f"[case] fast call, output layer {variant} {dtype} optional outputs={optional}", flush=True)
    T, B, A, H = 20, 7, 9, 64
    x, _ = _loss_args("cuda", T, B, A, dtype)
    g = torch.Generator().manual_seed(2)
    f = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    args = dict(hidden=f(T, B, H).tanh().bfloat16(), head_weight=(f(H, A + 1) / 8).bfloat16(), head_bias=f(A + 1),
                behaviour_logits=x["behaviour_logits"], actions=x["actions"], rewards=x["rewards"],
                discounts=x["discounts"], bootstrap_value=x["bootstrap_value"])
    if variant.get("behaviour") == "log_probs":
        args["behaviour_logits"] = -x["rewards"].abs() - 0.5
    e = dict(dtype=torch.float32, device="cuda")
    more = (torch.empty((T, B), **e), torch.empty((T, B), **e), torch.empty((B, 3), **e),
            torch.empty((T, B, A + 1), **e)) if optional else (None,) * 4
    out = vt.HeadLossGrad(torch.empty(4, **e), torch.empty((T, B, H), **e).to(variant.get("grad_dtype", torch.float32)),
                          torch.empty((H, A + 1), **e), torch.empty(A + 1, **e), *more)
    ws = vt.Workspace(T, B, A, H=H)
    _both_paths(monkeypatch, [
        lambda: vt.vtrace_head_loss_grad(**args, **SCALARS, **COSTS, **variant, out=out, workspace=ws)])


@pytest.mark.gpu
@pytest.mark.parametrize("name,change,error", [
    ("actions", lambda t: t.long(), TypeError), ("rewards", lambda t: t.cpu(), ValueError),
    ("values", lambda t: t[:, :-1], ValueError), ("discounts", lambda t: t.t().contiguous().t(), ValueError),
    ("behaviour_logits", lambda t: t.bfloat16(), TypeError), ("bootstrap_value", lambda t: t.tolist(), TypeError)])
def test_same_errors_as_the_python_path(name, change, error, monkeypatch):
    print(f"[case] fast call, bad {name}", flush=True)
    x, out = _loss_args("cuda")
    ws = vt.Workspace(5, 6, 9)
    seen = _count(monkeypatch)
    with pytest.raises(error):
        vt.vtrace_loss_grad(**dict(x, **{name: change(x[name])}), out=out, workspace=ws)
    with pytest.raises(vt.VtraceError, match="PARAM"):
        vt.vtrace_loss_grad(**x, lam=1.5, out=out, workspace=ws)
    assert seen == {"ran": 1, "declined": 1}


@pytest.mark.gpu
def test_unusual_calls_take_the_python_path(monkeypatch):
    print("[case] fast call, unusual calls", flush=True)
    x, out = _loss_args("cuda")
    ws = vt.Workspace(5, 6, 9)
    seen = _count(monkeypatch)
    vt.vtrace_loss_grad(**x, out=out, workspace=ws)
    ref = out.losses.clone()
    vt.vtrace_loss_grad(**x, rho_bar=1, out=out, workspace=ws)  # an int
    vt.vtrace_loss_grad(**dict(x, rewards=x["rewards"].as_subclass(_Subclass)), out=out, workspace=ws)
    with _Mode():
        vt.vtrace_loss_grad(**x, out=out, workspace=ws)
    vt.vtrace_loss_grad(**x, out=out)  # a workspace of its own: not offered at all
    assert seen == {"ran": 1, "declined": 3}
    torch.cuda.synchronize()
    assert torch.equal(out.losses, ref)
