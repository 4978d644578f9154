"""Forms that the rules of a launch choose: problems on which each form is taken (shown by
the names of the kernels that ran), against the float64 oracle; and what calls on two
routes to one quantity may differ by.

Tolerances: float64 1e-9 relative, the library's bar.  Mixed 1e-5: the factor updates are
rounded to float32 (6e-8) in chains of 144 products, and these problems are conditioned at
most about 1e2; a sum that misses or repeats one step of 16 of its few thousand products is
off by more than 1e-3."""
import re

import numpy as np
import pytest

import synth
from oracle import lma as olma

pytestmark = pytest.mark.gpu

BARS = {"fp64": 1e-9, "mixed": 1e-5}


def kernels_of(call):
    """The result of a call and the library's kernels in the order in which they ran."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as pf:
        result = call()
        torch.cuda.synchronize()
    ran = sorted((e.time_range.start, e.name) for e in pf.events() if e.device_type == torch.autograd.DeviceType.CUDA)
    found = (re.match(r"(?:void )?lma::(\w+(?:<[^(]*>)?)\(", name) for _, name in ran)
    names = [m[1] for m in found if m]
    if not names:
        pytest.skip("the profiler records no kernels here")
    return result, names


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


_REF = {}


def reference(p, key):
    if key not in _REF:
        _REF[key] = olma.fit_predict(p)
    return _REF[key]


# Products split along k.  13 windows that reach to the end: up to 286 tiles a step (a full
# turn of the 256 CUs whole, the rest in parts, more and fewer than 32 of them); three
# windows of 21 tiles: every tile of a step in parts.
SPLIT = {"rest of a turn": (dict(n=5200, M=13, B=12, s=200, n_u=300), True),
         "all tiles": (dict(n=7000, M=5, B=2, s=400, n_u=200), False)}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(SPLIT))
def test_products_in_parts_along_k(lib, name, precision):
    size, whole = SPLIT[name]
    b = size["n"] // size["M"]
    p = synth.make_random(seed=11, d=3, uneven=(b - 12, b + 12), sn2=0.05, **size)
    ref = reference(p, name)

    def call():
        state = lib.fit_problem(p, precision=precision)
        return state, state.predict(p.U, p.u_block_ptr)

    (state, (mean, var)), names = kernels_of(call)
    lml = state.lml()
    state.free()
    form = "double, false" if precision == "fp64" else "float, true"
    part, few, more = f"k_update_part<{form}>", f"k_update<{form}, 1, true>", f"k_update<{form}, 2, true>"
    steps = [i for i, k in enumerate(names) if k == part]
    sums = [names[i + 1] for i in steps]           # each is followed by the sums of its parts
    assert steps and set(sums) <= {few, more}
    print(f"  {len(steps)} steps in parts, {sums.count(few)} of at most 32 tiles", flush=True)
    if whole:
        assert any(names[i - 1] == f"k_update<{form}, 4, false>" for i in steps) and set(sums) == {few, more}
    bar = BARS[precision]
    assert rel(mean.cpu().numpy(), ref["mean"]) < bar and rel(var.cpu().numpy(), ref["var"]) < bar
    assert abs(lml - ref["lml"]) < bar * abs(ref["lml"])


# Tiles of few rows and launches of few tiles, mixed, with factors of 1 to 24 column tiles:
# the shares of the waves end where a float32 sum is folded, the last of 16 k with the one before
@pytest.mark.parametrize("n,M,B", [(130, 1, 0), (1300, 1, 0), (3000, 1, 0), (2900, 3, 2), (9000, 30, 2)])
def test_mixed_sums_shared_by_waves(lib, n, M, B):
    p = synth.make_random(seed=n + 5, n=n, d=3, M=M, s=61, n_u=3 * M, B=B, uneven=(max(1, n // M - 9), n // M + 9), sn2=0.05)
    ref = olma.fit_predict(p)

    def call():
        state = lib.fit_problem(p, precision="mixed")
        return state, state.predict(p.U, p.u_block_ptr)

    (state, (mean, var)), names = kernels_of(call)
    lml = state.lml()
    state.free()
    assert any(k.startswith("k_update_slim<float, true") for k in names)
    bar = BARS["mixed"]
    assert rel(mean.cpu().numpy(), ref["mean"]) < bar and rel(var.cpu().numpy(), ref["var"]) < bar
    assert abs(lml - ref["lml"]) < bar * abs(ref["lml"])


# A likelihood asked for with its gradient is formed in one order of sums, alone (or by a
# fit) in the order that is fastest at its size: the values agree to rounding, also where
# points lie dense on a line and the factors are conditioned worst
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-9), ("mixed", 1e-8)])
@pytest.mark.parametrize("n,d,M,B,s", [(600, 3, 5, 2, 40), (1399, 1, 7, 2, 200), (4507, 1, 30, 2, 703), (2500, 5, 4, 3, 130)])
def test_likelihood_with_and_without_its_gradient(lib, n, d, M, B, s, precision, bar):
    p = synth.make_random(seed=n, n=n, d=d, M=M, s=s, n_u=5, B=B, uneven=(n // M - 20, n // M + 20), sn2=0.05)
    problem = lib.LmlProblem.from_problem(p, precision=precision)
    value = problem(p.log_hyp, grad=False)
    with_grad, _ = problem(p.log_hyp, grad=True)
    state = lib.fit_problem(p, precision=precision)
    fitted = state.lml()
    state.free()
    print(f"  value {value!r} with gradient {with_grad!r} fit {fitted!r}", flush=True)
    assert abs(value - with_grad) < bar * abs(with_grad) and fitted == value


# The mean and variance of a point, asked for alone and among 300 others: a request's size
# decides the order of the sums, so the last bits may differ, no more
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-9), ("mixed", 1e-5)])
def test_one_point_alone_and_in_a_request(lib, precision, bar):
    p = synth.make_random(seed=9, n=5000, d=3, M=8, s=150, n_u=301, B=3, uneven=(610, 640), sn2=0.05)
    state = lib.fit_problem(p, precision=precision)
    mean, var = (t.clone() for t in state.predict(p.U, p.u_block_ptr))
    for u in (0, 150, 300):
        ptr = np.where(np.asarray(p.u_block_ptr) > u, 1, 0).astype(np.int64)
        m1, v1 = state.predict(p.U[u:u + 1], ptr)
        assert abs(float(m1[0] - mean[u])) < bar * float(mean.abs().max())
        assert abs(float(v1[0] - var[u])) < bar * float(var.abs().max())
    state.free()


# The backward pass forms the encoder's activations again from the weights of its own
# forward pass, whatever parameter updates lie between (the head's and the second layer's
# transposed weights are the current ones).  Tolerance: that of the network's oracle test.
@pytest.mark.parametrize("between", ["one update", "two updates", "other parameters", "other parameters and an update"])
def test_backward_after_a_parameter_change(lib, between):
    import torch
    from oracle import deepsets as ods
    from paper_1411_4510_amd import warmstart as ws
    sizes = [63, 300, 128]
    rng = np.random.default_rng(21)
    ptr, sn = ws.aligned_layout(sizes)
    feats = rng.standard_normal((int(ptr[-1]), ws.NFEAT)).astype(np.float32)
    labels, masks = rng.standard_normal((3, ws.NOUT)), np.ones((3, ws.NOUT))
    before = ws.he_init(4)
    net = ws.Network(max_rows=int(ptr[-1]), max_sets=3)
    net.set_params(before)
    net.forward(torch.as_tensor(feats, device="cuda"), ptr, sn)
    net.backward(labels, masks)
    if "other parameters" in between:
        net.set_params(ws.he_init(5))
    for _ in range({"one update": 1, "two updates": 2, "other parameters": 0}.get(between, 1)):
        net.adam(0.05)
    _, grad = net.backward(labels, masks, want_grad=True)
    sets = [feats[int(ptr[b]):int(ptr[b]) + n].astype(np.float64) for b, n in enumerate(sizes)]
    old = {k: v.astype(np.float64) for k, v in ws.unpack(before).items()}
    new = {k: v.astype(np.float64) for k, v in ws.unpack(net.get_params()).items()}
    outs, cache = ods.forward(old, sets)
    _, fresh = ods.forward(new, sets)
    cache["W"] = fresh["W"]                        # the current weights
    want = ods.backward(new, cache, outs, labels, masks)
    for b in range(3):                             # what the current activations would give
        for k in ("H1b", "H2b"):
            cache["sets"][b][k] = fresh["sets"][b][k]
    wrong = ods.backward(new, cache, outs, labels, masks)
    got = ws.unpack(grad.cpu().numpy())
    for k in ods.ORDER:
        assert rel(got[k], want[k]) <= 5e-3, k
        if k in ("W1", "b1", "W2", "b2"):
            assert rel(got[k], wrong[k]) > 5e-2, k
