"""Calls at the edges of what the entry points take: they are refused or answered as
their plain definition is, whatever form the library gives them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# A noise variance beyond the float32 range: a mixed fit stores its windows in float32, so
# the pivots are infinite, no likelihood exists and the call is refused (block None: no
# factor failed).  In float64 the same holds beyond the float64 range.
@pytest.mark.parametrize("precision,log_sn2", [("mixed", 89.0), ("mixed", 100.0), ("mixed", 708.0), ("mixed", 800.0),
                                               ("fp64", 709.9), ("fp64", 800.0)])
@pytest.mark.parametrize("B", [0, 2])
def test_variance_beyond_the_storage_type_is_refused(lib, precision, log_sn2, B):
    p = synth.make_random(seed=7, n=600, d=3, M=5, s=40, n_u=5, B=B, uneven=(60, 180), sn2=0.05)
    p.log_hyp = p.log_hyp.copy()
    p.log_hyp[-1] = log_sn2
    problem = lib.LmlProblem.from_problem(p, precision=precision)
    for call in (lambda: lib.fit_problem(p, precision=precision).free(), lambda: problem(p.log_hyp, grad=False),
                 lambda: problem(p.log_hyp, grad=True)):
        with pytest.raises(lib.LmaError) as e:
            call()
        assert e.value.status == lib.LMA_E_NOT_PD and e.value.block is None


# 2^30 points (a launch holds fewer than 2^32 threads) and one more: every count and label
def test_bounded_assignment_of_two_to_the_thirty_points(lib):
    import torch
    n = 2 ** 30 + 1
    P = torch.rand((n, 1), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    C = torch.tensor([[0.25], [0.75]], dtype=torch.float64, device="cuda")
    label, count, rounds = lib.bounded_assign(P, C, 0, n)
    nearer = (P[:, 0] - 0.25) ** 2 <= (P[:, 0] - 0.75) ** 2   # ties to the lower index
    assert rounds == 1 and bool(torch.equal(label == 0, nearer))
    assert count.tolist() == [int(nearer.sum()), n - int(nearer.sum())]
    del P, label, nearer
    lib.release_cache()
    torch.cuda.empty_cache()


# seeding with its draw in every workgroup (up to 2048 blocks of 256 points) and in one:
# the same indices as the oracle on both sides of the edge, no points, one round, several
@pytest.mark.parametrize("n,k", [(2048 * 256, 5), (2048 * 256 + 1, 1), (2048 * 256 + 1, 2), (2048 * 256 + 1, 3), (700001, 6)])
def test_seeding_on_both_sides_of_the_scan_limit(lib, n, k):
    from oracle import partition as opart
    rng = np.random.default_rng(n + k)
    P = np.round(rng.uniform(size=(n, 2)), 2)     # points on chosen centres: weights of 0
    rand = rng.integers(0, 2 ** 32, size=k, dtype=np.uint64).astype(np.uint32)
    C, idx = lib.kmeans_seed(P, k, rand)
    Co, io = opart.seed(P, k, rand)
    assert np.array_equal(idx.cpu().numpy(), io) and np.array_equal(C.cpu().numpy(), Co)


# the time of a round grows as the points do: fourfold points take about four times as long
# (17 times where every workgroup scanned every block)
def test_seeding_time_is_linear_in_the_points(lib):
    import time
    import torch
    rand = np.random.default_rng(1).integers(0, 2 ** 32, size=33, dtype=np.uint64).astype(np.uint32)
    t = []
    for n in (2 ** 22, 2 ** 24):
        P = torch.rand((n, 4), dtype=torch.float64, device="cuda")
        lib.kmeans_seed(P, 33, rand)
        runs = []
        for _ in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            lib.kmeans_seed(P, 33, rand)
            torch.cuda.synchronize()
            runs.append(time.perf_counter() - t0)
        t.append(min(runs))
    print(f"  33 centres: {t[0] * 1e3:.2f} ms at 2^22 points, {t[1] * 1e3:.2f} ms at 2^24", flush=True)
    assert t[1] < 8 * t[0]


def settled_free_memory():
    """Free device memory once the driver has taken back what was freed."""
    import time
    import torch
    torch.cuda.synchronize()
    last = -1
    for _ in range(40):
        now = torch.cuda.mem_get_info()[0]
        if now == last:
            break
        last = now
        time.sleep(0.25)
    return last


# A prediction with 24 MiB more than it cannot do without: the 64 MiB for sums of split
# products are an extra that it leaves out (the order of its sums differs then, no more)
def test_prediction_without_room_for_its_extra_workspace(lib):
    import torch
    p = synth.make_random(seed=3, n=6000, d=4, M=5, s=60, n_u=100, B=2, uneven=(1180, 1220), sn2=0.05)
    state = lib.fit_problem(p)
    U = torch.as_tensor(p.U, device="cuda")
    mean, var = (t.clone() for t in state.predict(U, p.u_block_ptr))
    lib.release_cache()
    torch.cuda.empty_cache()
    before = settled_free_memory()
    state.predict(U, p.u_block_ptr)
    workspace = before - settled_free_memory()  # the library keeps it for the next call
    lib.release_cache()
    torch.cuda.empty_cache()
    fill = [torch.empty(settled_free_memory() - (2 << 30), dtype=torch.uint8, device="cuda")]
    for piece in (256 << 20, 12 << 20):  # until the device is full
        try:
            while True:
                fill.append(torch.empty(piece, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            if piece == 256 << 20:
                fill.pop()  # room for small pieces
                torch.cuda.empty_cache()
    room = 0
    while room < workspace - (40 << 20):
        room += fill.pop().numel()
    torch.cuda.empty_cache()
    print(f"  workspace {workspace >> 20} MiB, room {room >> 20} MiB", flush=True)
    mean2, var2 = state.predict(U, p.u_block_ptr)
    del fill
    state.free()
    lib.release_cache()
    torch.cuda.empty_cache()
    assert workspace > (64 << 20)
    assert float((mean2 - mean).norm() / mean.norm()) < 1e-9 and float((var2 - var).norm() / var.norm()) < 1e-9


CACHE_SCRIPT = """
import sys
import numpy as np
import paper_1411_4510_amd as lma
import synth

def problem(n, M, s, seed):
    return synth.make_random(seed=seed, n=n, d=3, M=M, s=s, n_u=50, B=2, uneven=(n // M - 20, n // M + 20), sn2=0.05)

def mark(text):
    print("== " + text, file=sys.stderr, flush=True)

a, b = problem(6000, 3, 1000, 1), problem(1500, 3, 200, 2)
for i in range(4):
    mark("cycle %d" % i)
    for p in (a, b):
        st = lma.fit_problem(p)
        st.predict(p.U, p.u_block_ptr)
        st.free()
        lma.LmlProblem.from_problem(p)(p.log_hyp, grad=True)
mark("many")
states = [lma.fit_problem(problem(6000 + 300 * i, 3, 400, i)) for i in range(16)]
for st in states:
    st.free()
mark("released")
lma.release_cache()
mark("end")
"""


# The device cache, by its own trace: two problems of different sizes taken in turn allocate
# nothing once both have run, and what is kept is at most twelve blocks and 4 GiB of those
# up to 1 GiB, all of it handed back by lma_release_cache
def test_device_cache_keeps_two_problems_and_is_bounded(lib):
    import os
    import re
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CACHE_SCRIPT], cwd=root, env={**os.environ, "LMA_CACHE_TRACE": "1"},
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    where, kept, mallocs, most = "", [], {}, (0, 0.0)
    for line in r.stderr.splitlines():
        if line.startswith("== "):
            where = line[3:]
        elif "hipMalloc" in line:
            mallocs[where] = mallocs.get(where, 0) + 1
        elif m := re.search(r"put ([\d.]+) GB", line):
            kept.append(float(m[1]))
        elif m := re.search(r"cached block of ([\d.]+) GB|evict ([\d.]+) GB", line):
            kept.remove(float(m[1] or m[2]))
        elif m := re.search(r"free all: ([\d.]+) GB", line):
            assert abs(float(m[1]) - sum(kept)) < 0.01 * (len(kept) + 1)
            kept = []
        if "put" not in line:      # a block is put once its predecessor is evicted
            most = max(most, (len([k for k in kept if k <= 1.08]), sum(k for k in kept if k <= 1.08)))
    print(f"  hipMalloc calls {mallocs}, most blocks kept {most}", flush=True)
    assert mallocs["cycle 0"] > 0 and mallocs.get("cycle 2", 0) == mallocs.get("cycle 3", 0) == 0
    assert most[0] <= 12 and most[1] <= 4.3 + 0.12 and kept == []


# 540000 windows of one point, a test point each.  The support rows and the output row of the
# windows, and the products of the test rows, are 1080000 tiles of few rows: more than one
# launch holds (2^32 threads, 4096 per tile; of a larger one only the remainder would run).
# With one point per window the definition has a closed form; tolerance: the mixed bar.
def test_half_a_million_windows(lib):
    M, s, ell, sn2 = 540000, 64, 0.5, 1.0
    rng = np.random.default_rng(5)
    X = np.sort(rng.uniform(0, 100.0, size=M))
    y = np.sin(X) + 0.1 * rng.standard_normal(M)
    U = X + 1e-3
    S = X[::M // s][:s]
    ptr = np.arange(M + 1, dtype=np.int64)
    state = lib.fit(X[:, None], y, ptr, S[:, None], 0, np.log([ell, 1.0, sn2]), precision="mixed")
    mean, var = (t.cpu().numpy() for t in state.predict(U[:, None], ptr))
    lml = state.lml()
    state.free()
    lib.release_cache()

    def kernel(a, b):
        return np.exp(-0.5 * ((a[:, None] - b[None]) / ell) ** 2)

    Sig = kernel(S, S) + sn2 * np.eye(s)
    Li = np.linalg.inv(np.linalg.cholesky(Sig)).T
    K, Ku = kernel(X, S), kernel(U, S)
    V, Vu = K @ Li, Ku @ Li
    R = 1.0 + sn2 - (V ** 2).sum(1)
    Z, z = K / np.sqrt(R)[:, None], y / np.sqrt(R)
    Sdd, ydd = Sig + Z.T @ Z, Z.T @ z
    g = np.linalg.solve(Sdd, ydd)
    x = (np.exp(-0.5 * ((U - X) / ell) ** 2) - (Vu * V).sum(1)) / np.sqrt(R)
    E = Ku - x[:, None] * Z
    want_mean = E @ g + x * z
    want_var = 1.0 + sn2 - (Vu ** 2).sum(1) - x ** 2 + (E * np.linalg.solve(Sdd, E.T).T).sum(1)
    want = -0.5 * (z @ z - ydd @ g + np.log(R).sum() + np.linalg.slogdet(Sdd)[1] - np.linalg.slogdet(Sig)[1]
                   + M * np.log(2 * np.pi))
    for got, ref in ((mean, want_mean), (var, want_var)):
        assert np.abs(got - ref).max() < 1e-4 * np.abs(ref).max()
    assert abs(lml - want) < 1e-4 * abs(want)


# Window solves of very unequal windows: launches that hold the windows with a tile in
# them.  Windows of 1 to 14 tiles in several classes against the oracle, and 20000 windows
# of two points beside one of 8000: what the launches take (85 ms with every window in each)
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-9), ("mixed", 1e-5)])
@pytest.mark.parametrize("B", [0, 1, 3])
def test_windows_of_very_unequal_sizes(lib, B, precision, bar):
    from oracle import lma as olma
    sizes = [5, 3, 400, 7, 1300, 2, 130, 129, 900, 4, 4, 260, 1, 1]
    p = synth.make_random(seed=8, n=sum(sizes), d=3, M=len(sizes), s=70, n_u=60, B=B, uneven=(1, 1300), sn2=0.05)
    p.block_ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    ref = olma.fit_predict(p)
    for budget in (0, 1):
        state = lib.fit_problem(p, precision=precision)
        if budget:  # chunks of windows, each with an order of its own
            full = state.nbytes()
            state.free()
            state = lib.fit_problem(p, precision=precision, mem_budget=int(0.75 * full))
            assert state.chunks() > 1
        mean, var = state.predict(p.U, p.u_block_ptr)
        lml = state.lml()
        state.free()
        for got, want in ((mean.cpu().numpy(), ref["mean"]), (var.cpu().numpy(), ref["var"])):
            assert np.linalg.norm(got - want) < bar * np.linalg.norm(want)
        assert abs(lml - ref["lml"]) < bar * abs(ref["lml"])


def test_solves_of_one_large_among_many_small_windows(lib):
    import torch
    from torch.profiler import ProfilerActivity, profile
    sizes = np.full(20000, 2)
    sizes[6000] = 8000
    rng = np.random.default_rng(2)
    n = int(sizes.sum())
    X = np.sort(rng.uniform(size=n))[:, None]
    y = np.sin(9 * X[:, 0]) + 0.1 * rng.standard_normal(n)
    bp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as pf:
        lib.fit(X, y, bp, X[::500], 0, np.log([0.3, 1.0, 0.05]), precision="mixed").free()
        torch.cuda.synchronize()
    ran = [e.time_range.elapsed_us() for e in pf.events()
           if e.device_type == torch.autograd.DeviceType.CUDA and "k_solve_step" in e.name]
    if not ran:
        pytest.skip("the profiler records no kernels here")
    print(f"  {len(ran)} launches, {sum(ran) / 1e3:.2f} ms", flush=True)
    assert sum(ran) < 20e3


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-9), ("mixed", 1e-5)])
@pytest.mark.parametrize("sizes", [[2] * 1500 + [1500] + [2] * 1500 + [300], [129] * 8400 + [300]], ids=["12", "3"])
def test_solves_of_launches_that_are_cut(lib, sizes, precision, bar):
    # B = 0: PIC in closed form; launches with and without the small windows
    rng = np.random.default_rng(3)
    sizes = np.array(sizes)
    n, ell, sf2, sn2 = int(sizes.sum()), 0.4, 1.3, 0.3
    bp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    X = np.sort(rng.uniform(0, 10, size=(n, 1)), axis=0)
    y = np.sin(2 * X[:, 0]) + np.sqrt(sn2) * rng.standard_normal(n)
    S = np.linspace(0, 10, 30)[:, None]
    U = X[bp[:-1]] + 0.01  # one point in each block
    up = np.arange(len(sizes) + 1, dtype=np.int64)

    def k(a, b):
        return sf2 * np.exp(-0.5 * (a - np.swapaxes(b, -1, -2)) ** 2 / ell ** 2)

    # Sigma_SS and the blocks' covariances hold the noise, as the fit's do
    L = np.linalg.cholesky(k(S, S) + sn2 * np.eye(len(S)))
    dot, rhs, kept = k(S, S) + sn2 * np.eye(len(S)), np.zeros(len(S)), []
    for nb in np.unique(sizes):
        ms = np.flatnonzero(sizes == nb)
        rows = bp[ms][:, None] + np.arange(nb)
        Xm, KmS = X[rows], k(X[rows], S)
        V = np.linalg.solve(L, np.swapaxes(KmS, 1, 2))
        R = k(Xm, Xm) + sn2 * np.eye(nb) - np.swapaxes(V, 1, 2) @ V
        KuS = k(U[ms][:, None], S)
        Rum = k(U[ms][:, None], Xm) - np.swapaxes(np.linalg.solve(L, np.swapaxes(KuS, 1, 2)), 1, 2) @ V
        sol = np.linalg.solve(R, np.concatenate([KmS, y[rows][..., None]], axis=2))
        G = np.swapaxes(KmS, 1, 2) @ sol
        dot, rhs = dot + G[:, :, :-1].sum(0), rhs + G[:, :, -1].sum(0)
        kept.append((ms, KuS[:, 0], (Rum @ sol)[:, 0]))
    g = np.linalg.solve(dot, rhs)
    want = np.empty(len(sizes))
    for ms, KuS, r in kept:
        want[ms] = KuS @ g + r[:, -1] - r[:, :-1] @ g
    state = lib.fit(X, y, bp, S, 0, np.log([ell, sf2, sn2]), precision=precision)
    mean = state.predict(U, up)[0].cpu().numpy()
    alone = state.predict(U[:1], np.minimum(up, 1))[0].cpu().numpy()
    state.free()
    assert np.linalg.norm(mean - want) < bar * np.linalg.norm(want)
    assert abs(alone[0] - want[0]) < bar * np.linalg.norm(want)


def pic_lml(torch, sizes, X, y, S, log_hyp):
    """Log likelihood of PIC (B = 0, equal sizes together) as a differentiable expression."""
    ell, sf2, sn2 = log_hyp.exp()

    def k(a, b):
        return sf2 * torch.exp(-0.5 * (a - b.transpose(-1, -2)) ** 2 / ell ** 2)

    eye = torch.eye(len(S), dtype=X.dtype)
    Sig = k(S, S) + sn2 * eye
    L = torch.linalg.cholesky(Sig)
    start = np.concatenate([[0], np.cumsum(sizes)])
    dot, rhs, out = Sig, 0.0, -0.5 * len(y) * np.log(2 * np.pi) + L.diagonal().log().sum()
    for nb in np.unique(sizes):
        rows = torch.tensor(start[np.flatnonzero(sizes == nb)][:, None] + np.arange(nb))
        K = k(X[rows], S)
        V = torch.linalg.solve_triangular(L, K.transpose(1, 2).contiguous(), upper=False)
        R = k(X[rows], X[rows]) + sn2 * torch.eye(int(nb), dtype=X.dtype)
        LR = torch.linalg.cholesky(R - V.transpose(1, 2).contiguous() @ V)
        h = torch.linalg.solve_triangular(LR, torch.cat([K, y[rows][..., None]], 2), upper=False)
        flat = h.reshape(-1, h.shape[2])
        G = flat.T.contiguous() @ flat
        dot, rhs = dot + G[:-1, :-1], rhs + G[:-1, -1]
        out = out - 0.5 * G[-1, -1] - LR.diagonal(dim1=1, dim2=2).log().sum()
    Ld = torch.linalg.cholesky(dot)
    z = torch.linalg.solve_triangular(Ld, rhs[:, None], upper=False)
    return out + 0.5 * (z * z).sum() - Ld.diagonal().log().sum()


def test_gradient_of_one_large_among_many_small_windows(lib):
    import torch
    sizes = np.full(20000, 2)
    sizes[6000] = 8000
    rng = np.random.default_rng(4)
    n = int(sizes.sum())
    bp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    X = np.sort(rng.uniform(0, 10, size=(n, 1)), axis=0)
    y = np.sin(2 * X[:, 0]) + 0.5 * rng.standard_normal(n)
    S = np.linspace(0, 10, 30)[:, None]
    hyp = np.log([0.4, 1.3, 0.3])
    h = torch.tensor(hyp, requires_grad=True)
    want = pic_lml(torch, sizes, *[torch.tensor(a) for a in (X, y, S)], h)
    want.backward()
    value, grad = lib.lml(X, y, bp, S, 0, hyp, grad=True)
    ref = h.grad.numpy()
    print(f"  {abs(value - want.item()) / abs(want.item()):.1e}, "
          f"{np.linalg.norm(grad - ref) / np.linalg.norm(ref):.1e}", flush=True)
    assert abs(value - want.item()) < 1e-9 * abs(want.item())
    # sums over n points with terms of either sign: 100 times the bar of a value
    assert np.linalg.norm(grad - ref) < 1e-7 * np.linalg.norm(ref)


def test_centre_update_of_more_workgroups_than_a_launch_holds(lib, monkeypatch):
    # all partial sums at once: 262145 chunks of 4096 points x 64 groups of 8 centres, 2^24 + 64
    # workgroups of 256 threads.  Whole coordinates: the sums are exact in any order.
    import torch
    n, k = 2 ** 30 + 4096, 512
    monkeypatch.setenv("LMA_KMEANS_PART_BYTES", str(4 << 30))
    gen = torch.Generator(device="cuda").manual_seed(1)
    label = torch.randint(0, k, (n,), dtype=torch.int32, device="cuda", generator=gen)
    P = torch.randint(0, 64, (n, 1), dtype=torch.int32, device="cuda", generator=gen).double()
    C, count = lib.kmeans_update(P, label, torch.zeros(k, 1, dtype=torch.float64, device="cuda"))
    want = torch.zeros(k, dtype=torch.int64, device="cuda")
    total = torch.zeros(k, dtype=torch.float64, device="cuda")
    for i in range(0, n, 2 ** 26):
        want += torch.bincount(label[i:i + 2 ** 26], minlength=k)
        total += torch.bincount(label[i:i + 2 ** 26], weights=P[i:i + 2 ** 26, 0], minlength=k)
    assert torch.equal(count.long(), want)
    assert torch.equal(C[:, 0], total / want)
    del P, label
    torch.cuda.empty_cache()
