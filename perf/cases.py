"""Performance cases of the LMA library: what its users run, through its public entry points.

A case is a dict of plain values.  Its "kind" names the work of one pass:

  fit        fit, then predict mean and variance, then the likelihood of the state
             (the regression itself; both precisions)
  lml        log marginal likelihood, with its gradient or alone, on data uploaded once
             (one step of a hyperparameter search)
  predict    mean and variance from a state that is kept (serving)
  cov        mean and full covariance of a small test set from a state that is kept
  partition  the block partition of training and test points that precedes a fit
  train      one training step of the warm-start network (forward, backward, Adam)

Sizes follow the repository's workloads (n=600 smoke run, n=2048, n=16384 sweep, n=65536,
n=131072 gradient, the d=21 mixture of the benchmark, the n=4096 warm-start sets) and ragged
neighbours of them.  Inputs are made on the GPU from the seed: points in the unit cube (d <= 8)
or a mixture of 32 Gaussians (d = 21), outputs a random-feature draw from the prior plus noise,
blocks by sorting on the first coordinate.
"""
import math

import numpy as np
import torch

import paper_1411_4510_amd as lma
from paper_1411_4510_amd import warmstart

F64 = torch.float64


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # the smoke run's problem: latency of a whole fit and prediction, ragged blocks
        dict(name="fit_600", kind="fit", precision="fp64", n=600, d=3, M=5, B=2, s=40, n_u=80, uneven=True),
        # a small regression: eight equal blocks, support set below one tile
        dict(name="fit_2048", kind="fit", precision="fp64", n=2048, d=4, M=8, B=1, s=64, n_u=256, uneven=False),
        # the middle workload: 64 blocks of 1024
        dict(name="fit_65536", kind="fit", precision="fp64", n=65536, d=8, M=64, B=2, s=512, n_u=8192, uneven=False),
        # the benchmark's problem (d = 21 mixture, uneven blocks, B = 3, |S| = 1024) at half its size
        dict(name="fit_262144", kind="fit", precision="fp64", n=262144, d=21, M=128, B=3, s=1024, n_u=32768,
             uneven=True),
        # mixed precision on sizes that are multiples of nothing
        dict(name="fit_mixed_50021", kind="fit", precision="mixed", n=50021, d=7, M=41, B=3, s=333, n_u=5003,
             uneven=True),
        # the wide end of the |S| x B sweep: B = M - 1, every window reaches to the last block (full GP)
        dict(name="fit_fullgp_16384", kind="fit", precision="fp64", n=16384, d=8, M=16, B=15, s=256, n_u=4096,
             uneven=False),
        # the likelihood and gradient of a warm-start training set (labels: 30 of these for each of 20000 sets)
        dict(name="lml_4096", kind="lml", precision="fp64", n=4096, d=5, M=16, B=2, s=256, grad=True, uneven=False),
        # the gradient workload, in mixed precision
        dict(name="lml_mixed_131072", kind="lml", precision="mixed", n=131072, d=8, M=128, B=2, s=512, grad=True,
             uneven=False),
        # serving: a request of 100 points against a fitted state
        dict(name="predict_100", kind="predict", precision="fp64", n=65536, d=8, M=64, B=2, s=512, n_u=100,
             uneven=False),
        # the joint covariance of a small test set
        dict(name="cov_512", kind="cov", precision="fp64", n=16384, d=5, M=16, B=2, s=256, n_u=512, uneven=True),
        # blocks for a 65536-point problem
        dict(name="partition_65536", kind="partition", n=65536, d=8, M=64, n_u=8192, iters=10),
        # a minibatch of the warm-start network's training
        dict(name="train_64x4096", kind="train", sets=64, n=4096, uneven=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_problem(rng, n_hi, block_hi):
    """Sizes of a regression: block sizes from a tenth of a tile to block_hi, B from PIC upwards."""
    n = _log_int(rng, 500, n_hi)
    block = _log_int(rng, 100, min(block_hi, n // 3))
    M = max(3, n // block)
    B = min(rng.choice([0, 1, 1, 2, 2, 3, 3, 4]), M - 1)
    if n <= 20000 and rng.random() < 0.15:
        B = M - 1
    d = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 21])
    return dict(n=n, d=d, M=M, B=B, s=_log_int(rng, 16, min(1024, n // 2)), uneven=rng.random() < 0.6)


def draw(rng):
    cap = 0.8 * work(listed()[3])["flops"]
    while True:
        kind = rng.choice(["fit"] * 5 + ["lml"] * 4 + ["predict", "cov", "partition", "train"])
        precision = rng.choice(["fp64", "fp64", "mixed"])
        if kind == "fit":
            c = dict(kind=kind, precision=precision, **_draw_problem(rng, 200000, 2048))
            c["n_u"] = _log_int(rng, 50, max(60, c["n"] // 4))
        elif kind == "lml":
            c = dict(kind=kind, precision=precision, **_draw_problem(rng, 131072, 1024), grad=rng.random() < 0.8)
        elif kind == "predict":
            c = dict(kind=kind, precision=precision, **_draw_problem(rng, 65536, 1024), n_u=_log_int(rng, 1, 4000))
        elif kind == "cov":
            c = dict(kind=kind, precision=precision, **_draw_problem(rng, 30000, 1024), n_u=_log_int(rng, 10, 1000))
        elif kind == "partition":
            n = _log_int(rng, 2000, 262144)
            c = dict(kind=kind, n=n, d=rng.choice([1, 2, 4, 5, 8, 21]), M=_log_int(rng, 4, max(5, min(256, n // 200))),
                     n_u=_log_int(rng, 100, max(200, n // 8)), iters=rng.choice([5, 10, 20]))
        else:
            c = dict(kind=kind, sets=_log_int(rng, 1, 64), n=_log_int(rng, 100, 4096), uneven=rng.random() < 0.5)
        if work(c)["flops"] <= cap:
            return c


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _block_ptr(n, M, uneven, rng):
    """M non-empty blocks; uneven sizes spread over about a factor of three."""
    w = rng.uniform(0.5, 1.5, size=M) if uneven else np.ones(M)
    cuts = np.round(np.cumsum(w) / w.sum() * n).astype(np.int64)
    bp = np.concatenate([[0], cuts])
    bp[-1] = n
    for m in range(1, M):                      # at least one point each
        bp[m] = min(max(bp[m], bp[m - 1] + 1), n - (M - m))
    return bp


def _points(n, d, gen, centres=None):
    if d <= 8:
        return torch.rand((n, d), generator=gen, device="cuda", dtype=F64)
    which = torch.randint(centres.shape[0], (n,), generator=gen, device="cuda")
    return centres[which] + 0.2 * torch.randn((n, d), generator=gen, device="cuda", dtype=F64)


def _outputs(sets, ell, sf2, gen, features=256):
    """Joint random-feature draw from the squared-exponential prior at several point sets."""
    d = sets[0].shape[1]
    W = torch.randn((d, features), generator=gen, device="cuda", dtype=F64) / ell[:, None]
    phase = 2 * math.pi * torch.rand((features,), generator=gen, device="cuda", dtype=F64)
    amp = math.sqrt(2.0 * sf2 / features)
    return [torch.cat([amp * torch.cos(P @ W + phase).sum(1) for P in S.split(65536)]) for S in sets]


def _regression(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    n, d, M, s = case["n"], case["d"], case["M"], case["s"]
    n_u = case.get("n_u", 0)
    centres = torch.rand((32, d), generator=gen, device="cuda", dtype=F64)
    if case["kind"] == "lml":                   # the ranges that hyperparameter searches meet
        ell = np.exp(rng.uniform(math.log(0.1), math.log(2.0), size=d))
        sf2, sn2 = math.exp(rng.uniform(math.log(0.3), math.log(3.0))), math.exp(rng.uniform(math.log(0.01), math.log(0.5)))
    elif d <= 8:
        ell, sf2, sn2 = np.exp(rng.uniform(math.log(0.1), 0.0, size=d)), 1.0, 0.05
    else:
        ell, sf2, sn2 = np.ones(d), 1.0, 0.01
    X, U = _points(n, d, gen, centres), _points(n_u, d, gen, centres)
    X = X[torch.argsort(X[:, 0])].contiguous()
    U = U[torch.argsort(U[:, 0])].contiguous()
    bp = _block_ptr(n, M, case["uneven"], rng)
    ell_t = torch.tensor(ell, device="cuda")
    y = _outputs([X], ell_t, sf2, gen)[0]
    y = y + math.sqrt(sn2) * torch.randn((n,), generator=gen, device="cuda", dtype=F64)
    S = X[torch.sort(torch.randperm(n, generator=gen, device="cuda")[:s]).values].contiguous()
    st = dict(kind=case["kind"], X=X, y=y, S=S, block_ptr=bp, B=case["B"], precision=case["precision"],
              log_hyp=np.concatenate([np.log(ell), [math.log(sf2), math.log(sn2)]]))
    if n_u:
        at = torch.as_tensor(bp[1:-1], device="cuda")
        cuts = 0.5 * (X[at - 1, 0] + X[at, 0])
        ub = torch.searchsorted(U[:, 0].contiguous(), cuts).cpu().numpy()
        st["U"] = U
        st["u_block_ptr"] = np.concatenate([[0], ub, [n_u]]).astype(np.int64)
    return st


def _sets(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    k, n = case["sets"], case["n"]
    sizes = rng.integers(max(2, n // 2), n + 1, size=k) if case["uneven"] else np.full(k, n)
    ptr, set_n = warmstart.aligned_layout(sizes)
    feats = torch.zeros((int(ptr[-1]), warmstart.NFEAT), device="cuda")
    labels, masks = np.zeros((k, warmstart.NOUT), np.float32), np.zeros((k, warmstart.NOUT), np.float32)
    for i in range(k):
        d, m = int(rng.integers(1, 9)), int(sizes[i])
        rows = feats[int(ptr[i]):int(ptr[i]) + m]
        rows[:, :d] = torch.rand((m, d), generator=gen, device="cuda")
        rows[:, 8] = torch.randn((m,), generator=gen, device="cuda")
        rows[:, 9:9 + d] = 1.0
        masks[i] = warmstart.valid_mask(d)
        labels[i] = masks[i] * rng.normal(-1.0, 1.0, size=warmstart.NOUT)
    return dict(kind="train", ptr=ptr, set_n=set_n, feats=feats, labels=torch.tensor(labels, device="cuda"),
                masks=torch.tensor(masks, device="cuda"), params=warmstart.he_init(seed))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        st = _sets(case, seed)
        st["net"] = warmstart.Network(max_rows=int(st["ptr"][-1]), max_sets=len(st["set_n"]))
        st["net"].set_params(st["params"])
        return st
    if kind == "partition":
        gen = torch.Generator(device="cuda").manual_seed(seed)
        rng = np.random.default_rng(seed)
        n, d, M = case["n"], case["d"], case["M"]
        centres = torch.rand((32, d), generator=gen, device="cuda", dtype=F64)
        return dict(kind=kind, X=_points(n, d, gen, centres), U=_points(case["n_u"], d, gen, centres), M=M,
                    lo=n // M // 2, hi=max(n // M * 3 // 2, -(-n // M)), iters=case["iters"],
                    rand=rng.integers(0, 2 ** 32, size=M, dtype=np.uint64).astype(np.uint32))
    st = _regression(case, seed)
    if kind == "lml":
        st["problem"] = lma.LmlProblem(st["X"], st["y"], st["block_ptr"], st["S"], st["B"], precision=st["precision"])
        st["grad"] = case["grad"]
    elif kind in ("predict", "cov"):
        st["state"] = lma.fit(st["X"], st["y"], st["block_ptr"], st["S"], st["B"], st["log_hyp"],
                              precision=st["precision"])
    return st


def run(st):
    kind = st["kind"]
    if kind == "fit":
        state = lma.fit(st["X"], st["y"], st["block_ptr"], st["S"], st["B"], st["log_hyp"], precision=st["precision"])
        mean, var = state.predict(st["U"], st["u_block_ptr"])
        lml = state.lml()
        state.free()
        return {"mean": mean, "var": var, "lml": lml}
    if kind == "lml":
        out = st["problem"](st["log_hyp"], grad=st["grad"])
        return {"lml": out[0], "grad": out[1]} if st["grad"] else {"lml": out}
    if kind == "predict":
        mean, var = st["state"].predict(st["U"], st["u_block_ptr"])
        return {"mean": mean, "var": var}
    if kind == "cov":
        mean, cov = st["state"].predict_cov(st["U"], st["u_block_ptr"])
        return {"mean": mean, "cov": cov}
    if kind == "partition":
        return lma.partition(st["X"], st["M"], st["lo"], st["hi"], st["iters"], st["rand"], U=st["U"])
    out = st["net"].forward(st["feats"], st["ptr"], st["set_n"])
    _, grad = st["net"].backward(st["labels"], st["masks"], want_grad=True, want_loss=False)
    st["net"].adam(1e-3)
    return {"out": out, "grad": grad}


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "train":
        rows, w = case["sets"] * case["n"] * (0.75 if case["uneven"] else 1.0), warmstart.WIDTH
        per_row = 2.0 * (warmstart.NFEAT * w + w * w)
        # forward, both weight gradients, and the gradient that reaches the first layer
        return {"bytes": rows * warmstart.NFEAT * 4 + 5 * warmstart.NPARAM * 4,
                "flops": rows * (2 * per_row + 2.0 * w * w)}
    n, d, M = case["n"], case["d"], case["M"]
    n_u = case.get("n_u", 0)
    if kind == "partition":
        # seeding, the rounds, the bounded assignment and the test points: 3 operations per coordinate and pair
        return {"bytes": 8.0 * (n + n_u) * (d + 1), "flops": 3.0 * d * M * (n * (2 + case["iters"]) + n_u)}
    s, B, b = float(case["s"]), min(case["B"], M - 1), n / M
    J = [b * (min(m + B, M - 1) - m + 1) for m in range(M)]
    W = [j - b for j in J]
    pairs = sum(b * j for j in J) - 0.5 * n * b                 # entries of the residual band
    support = s ** 3 / 3 + n * s * s
    assemble = 2 * s * pairs + (3 * d + 10) * (pairs + n * s)
    factor = sum(j ** 3 / 3 + j * j * (s + 1) for j in J)
    reduce = sum(b * (s + 1) ** 2 for _ in J) + s ** 3 / 3
    fit = support + assemble + factor + reduce
    u = n_u / M
    test = n_u * s * s * 2 + sum(u * (2 * s * min(b * (2 * B + 1), n) + 2 * s * j) + u * j * j * 1.0 for j in J)
    test += sum(u * sum(J[q] ** 2 for q in range(max(0, m - B), m)) for m in range(M))
    inputs = 8.0 * (n * (d + 1) + s * d)
    if kind == "fit":
        return {"bytes": inputs + 8.0 * n_u * (d + 2), "flops": fit + test}
    if kind == "lml":
        if not case["grad"]:
            return {"bytes": inputs, "flops": fit}
        back = sum(j ** 3 / 3 + j * j * s + 2 * j * s * s + j * j * (b + s) for j in J)
        back += sum(w * w * s for w in W) + 4 * s ** 3 + 2 * d * (pairs * (B + 1) + 2 * n * s)
        return {"bytes": inputs + 8.0 * (d + 2), "flops": fit + back}
    if kind == "predict":
        # the factors of the windows are the state: a request reads each once
        return {"bytes": 8.0 * n_u * (d + 2) + sum(4.0 * j * (j + 2 * s) for j in J) + 8.0 * n * s, "flops": test}
    return {"bytes": 8.0 * n_u * (d + 1 + n_u) + sum(4.0 * j * (j + 2 * s) for j in J) + 8.0 * n * s,
            "flops": test + n_u * n_u * s + n_u * n_u * (2 * B + 1) / M * (2 * s + sum(J) / M)}


# ----------------------------------------------------------------------------
# the same results in plain torch, float64
# ----------------------------------------------------------------------------

def _cov(A, C, log_hyp, d, same=False):
    sq = torch.zeros((A.shape[0], C.shape[0]), device=A.device, dtype=F64)
    for t in range(d):
        sq = sq + ((A[:, t, None] - C[None, :, t]) / torch.exp(log_hyp[t])) ** 2
    K = torch.exp(log_hyp[d]) * torch.exp(-0.5 * sq)
    if same:
        K = K + torch.exp(log_hyp[d + 1]) * torch.eye(A.shape[0], device=A.device, dtype=F64)
    return K


def _solve(L, R):
    return torch.linalg.solve_triangular(L, R, upper=False)


def _reference(st, log_hyp, cov=False, test=True):
    """The windows' definition (Definitions 1-2, Theorem 2 in whitened form), one window at a time."""
    X, S, c, bp, B = st["X"], st["S"], st["y"], st["block_ptr"], st["B"]
    d, M, s = X.shape[1], len(bp) - 1, S.shape[0]
    B = min(B, M - 1)
    test = test and "U" in st
    Sig = _cov(S, S, log_hyp, d, same=True)
    Ls = torch.linalg.cholesky(Sig)
    if test:
        U, ubp = st["U"], st["u_block_ptr"]
        n_u = U.shape[0]
        Ku = _cov(S, U, log_hyp, d)
        Vu = _solve(Ls, Ku)
        G, lu, xi = torch.zeros((n_u, s), device="cuda", dtype=F64), torch.zeros(n_u, device="cuda", dtype=F64), torch.zeros(n_u, device="cuda", dtype=F64)
        cols = {}
    Sdd, ydd, q, ld = Sig, torch.zeros(s, device="cuda", dtype=F64), 0.0, 0.0
    for m in range(M):
        hi = min(m + B, M - 1)
        J = torch.cat([X[bp[m + 1]:bp[hi + 1]], X[bp[m]:bp[m + 1]]])
        cJ = torch.cat([c[bp[m + 1]:bp[hi + 1]], c[bp[m]:bp[m + 1]]])
        w = J.shape[0] - int(bp[m + 1] - bp[m])
        K = _cov(J, S, log_hyp, d)
        V = _solve(Ls, K.T)
        L = torch.linalg.cholesky(_cov(J, J, log_hyp, d, same=True) - V.T @ V)
        rhs = [K, cJ[:, None]]
        if test:
            u0, u1 = int(ubp[m]), int(ubp[hi + 1])
            rhs.append(_cov(J, U[u0:u1], log_hyp, d) - V.T @ Vu[:, u0:u1])
        sol = _solve(L, torch.cat(rhs, 1))
        Z, z = sol[w:, :s], sol[w:, s]
        Sdd, ydd, q = Sdd + Z.T @ Z, ydd + Z.T @ z, q + z @ z
        ld = ld + 2.0 * torch.log(torch.diagonal(L)[w:]).sum()
        if test and u1 > u0:
            T = sol[:, s + 1:]
            x = T[w:]
            G[u0:u1] += x.T @ Z
            lu[u0:u1] += x.T @ z
            xi[u0:u1] += (x * x).sum(0)
            own = int(ubp[m + 1]) - u0
            if w > 0 and own > 0:
                p = T[:w, :own]
                G[u0:u0 + own] += p.T @ sol[:w, :s]
                lu[u0:u0 + own] += p.T @ sol[:w, s]
                xi[u0:u0 + own] += (p * p).sum(0)
            if cov:
                cols[m] = (T.clone(), w, u0)
    Ld = torch.linalg.cholesky(Sdd)
    g = torch.cholesky_solve(ydd[:, None], Ld)[:, 0]
    lml = -0.5 * (q - ydd @ g + ld + 2.0 * torch.log(torch.diagonal(Ld)).sum()
                  - 2.0 * torch.log(torch.diagonal(Ls)).sum() + c.shape[0] * math.log(2 * math.pi))
    if not test:
        return {"lml": lml}
    E = Ku.T - G
    T = _solve(Ld, E.T)
    out = {"lml": lml, "mean": E @ g + lu}
    sf2, sn2 = torch.exp(log_hyp[d]), torch.exp(log_hyp[d + 1])
    out["var"] = sf2 + sn2 - (Vu * Vu).sum(0) - xi + (T * T).sum(0)
    if cov:
        C = T.T @ T
        for a in range(M):
            for b in range(a, min(a + B, M - 1) + 1):
                ua, ub = slice(int(ubp[a]), int(ubp[a + 1])), slice(int(ubp[b]), int(ubp[b + 1]))
                if ua.stop == ua.start or ub.stop == ub.start:
                    continue
                R = _cov(U[ua], U[ub], log_hyp, d, same=a == b) - Vu[:, ua].T @ Vu[:, ub]
                for m in range(max(0, b - B), a + 1):
                    t, w, u0 = cols[m]
                    t = t if m == a else t[w:]
                    R = R - t[:, ua.start - u0:ua.stop - u0].T @ t[:, ub.start - u0:ub.stop - u0]
                C[ua, ub] += R
                if b != a:
                    C[ub, ua] += R.T
        out["cov"] = C
    return out


def _network(st):
    """The warm-start network in float64 without the kernels' bfloat16 roundings: outputs and loss gradient."""
    p = {k: torch.tensor(v, device="cuda", dtype=F64, requires_grad=True) for k, v in warmstart.unpack(st["params"]).items()}
    outs = []
    for i, m in enumerate(st["set_n"]):
        x = st["feats"][int(st["ptr"][i]):int(st["ptr"][i]) + int(m)].to(F64)
        h = torch.relu(x @ p["W1"].T + p["b1"])
        h = torch.relu(h @ p["W2"].T + p["b2"]).mean(0)
        outs.append(torch.relu(p["W3"] @ h + p["b3"]) @ p["W4"].T + p["b4"])
    out = torch.stack(outs)
    lab, msk = st["labels"].to(F64), st["masks"].to(F64)
    loss = (((out - lab) ** 2 * msk).sum(1) / msk.sum(1)).mean()
    loss.backward()
    return {"out": out.detach(), "grad": torch.cat([p[k].grad.reshape(-1) for k, _ in warmstart.LAYOUT])}


def exact(case, seed):
    kind = case["kind"]
    if kind == "partition":       # permutations and sizes are whole numbers; the centres follow from them
        return None
    if kind == "train":
        return _network(_sets(case, seed))
    b, B = case["n"] / case["M"], min(case["B"], case["M"] - 1)
    cubes = sum((b * (min(m + B, case["M"] - 1) - m + 1)) ** 3 for m in range(case["M"]))
    if cubes > 2.5e13:
        return None
    st = _regression(case, seed)
    log_hyp = torch.tensor(st["log_hyp"], device="cuda")
    if kind == "lml":
        if not case["grad"]:
            with torch.no_grad():
                return {"lml": _reference(st, log_hyp)["lml"].item()}
        if cubes > 3e11 or case["M"] > 400:
            with torch.no_grad():
                return {"lml": _reference(st, log_hyp)["lml"].item(), "grad": None}
        log_hyp.requires_grad_(True)
        v = _reference(st, log_hyp)["lml"]
        v.backward()
        return {"lml": v.item(), "grad": log_hyp.grad.cpu().numpy()}
    with torch.no_grad():
        out = _reference(st, log_hyp, cov=kind == "cov")
    if kind == "fit":
        return {"mean": out["mean"], "var": out["var"], "lml": out["lml"].item()}
    return {"mean": out["mean"], "cov": out["cov"]} if kind == "cov" else {"mean": out["mean"], "var": out["var"]}
