"""Kernel variants at the sizes where they can go wrong (edges of tiles and
blocks, remainders, smallest sizes), against the float64 oracle.

Tolerance: the library's float64 bar, 1e-9 relative (2-norm of a vector, |.| of
the log marginal likelihood); the problems are conditioned at most about 1e4, so
float64 rounding leaves four orders of margin."""
import numpy as np
import pytest

import synth
from oracle import lma as olma

pytestmark = pytest.mark.gpu

BAR = 1e-9


@pytest.fixture(scope="module")
def lib():
    import paper_1411_4510_amd as lma
    lma.load()
    return lma


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


def check_fit(lib, p, bar=BAR, precision="fp64"):
    ref = olma.fit_predict(p)
    st = lib.fit_problem(p, precision=precision)
    mean, var = st.predict(p.U, p.u_block_ptr)
    lml = st.lml()
    st.free()
    assert rel(mean.cpu().numpy(), ref["mean"]) < bar
    assert rel(var.cpu().numpy(), ref["var"]) < bar
    assert abs(lml - ref["lml"]) < bar * abs(ref["lml"])


# one window of n points: its last diagonal tile has n mod 128 real rows
@pytest.mark.parametrize("n,s", [(16, 1), (17, 15), (31, 16), (33, 17), (112, 5), (113, 127), (127, 128), (129, 129),
                                 (255, 40), (257, 143)])
def test_diagonal_tile_block_edges(lib, n, s):
    s = min(s, n)
    p = synth.make_random(seed=100 + n, n=n, d=2, M=1, s=s, n_u=9, B=0, uneven=(n, n), sn2=0.05)
    check_fit(lib, p)


# windows from one to a dozen tiles in one launch of the vector solves, some with an
# empty separator; forward and backward (the mixed path runs both; its bar is 1e-4)
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("B", [0, 1, 4])
def test_vector_solves_of_unequal_windows(lib, B, precision, bar):
    p = synth.make_random(seed=61, n=1500, d=3, M=5, s=70, n_u=60, B=B, uneven=(20, 700), sn2=0.05)
    check_fit(lib, p, bar=bar, precision=precision)


# launches of few tiles run in pieces of 64 x 64 and 32 x 32: windows of 1 to 16 tiles
# (16 and fewer tiles per launch, up to 128, more), pieces of padding only (blocks of
# 130 and 33 points), test tiles of a few rows
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("n,M,B,s,n_u", [(33, 1, 0, 7, 3), (130, 1, 0, 33, 200), (520, 4, 3, 130, 70),
                                         (1600, 8, 2, 260, 333), (4200, 25, 4, 97, 31)])
def test_pieces_of_tiles(lib, n, M, B, s, n_u, precision, bar):
    p = synth.make_random(seed=n, n=n, d=4, M=M, s=s, n_u=n_u, B=B, uneven=(max(1, n // M - 15), n // M + 15), sn2=0.05)
    check_fit(lib, p, bar=bar, precision=precision)


# test tiles of 1 to 65 rows (16, 32 and 64 rows have forms of their own, 65 none), alone
# and beside whole tiles in one launch (blocks without and with many test points), with
# the output row of windows of 1 to 20 tiles; full covariance over such tiles; a memory
# budget, which forms the test rows without a band and the windows chunk by chunk
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("n,M,B,counts", [(700, 3, 1, (1, 0, 16)), (2700, 3, 2, (17, 32, 33)), (2600, 4, 3, (64, 1, 0, 65)),
                                          (2560, 1, 0, (5,)), (9000, 30, 2, (3,) * 29 + (140,))])
def test_tiles_of_few_rows(lib, n, M, B, counts, precision, bar):
    rng = np.random.default_rng(n)
    p = synth.make_random(seed=n + 2, n=n, d=3, M=M, s=61, n_u=sum(counts), B=B, uneven=(n // M - 9, n // M + 9), sn2=0.05)
    p.u_block_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    p.U = rng.uniform(size=(sum(counts), 3))
    ref = olma.fit_predict(p)
    cov_ref = olma.predict_cov(p)[1]
    full = 0
    for share in (1.0, 0.6) if M > 3 else (1.0,):  # three windows do not fit a smaller budget one by one
        st = lib.fit_problem(p, precision=precision, mem_budget=int(share * full) if share < 1 else 0)
        full = st.nbytes()
        mean, var = st.predict(p.U, p.u_block_ptr)
        mean2, cov = st.predict_cov(p.U, p.u_block_ptr)
        st.free()
        assert rel(mean.cpu().numpy(), ref["mean"]) < bar and rel(mean2.cpu().numpy(), ref["mean"]) < bar
        assert rel(var.cpu().numpy(), ref["var"]) < bar
        assert rel(cov.cpu().numpy(), cov_ref) < bar


# mean and residual sums in parts of the column list: row tiles of 1 to 128 points (waves
# share columns up to 64 rows), lists shorter and longer than the parts, 1024 and more
# row tiles (no parts), windows at both ends of the overlap
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("n,M,B,n_u", [(90, 1, 0, 1), (300, 2, 1, 33), (500, 3, 0, 3 * 17), (900, 4, 3, 4 * 65),
                                       (1300, 3, 1, 3 * 129), (2600, 1040, 1, 2080)])
def test_kernel_sums_in_parts(lib, n, M, B, n_u, precision, bar):
    p = synth.make_random(seed=n + 1, n=n, d=5, M=M, s=50, n_u=n_u, B=B, uneven=(max(1, n // M - 9), n // M + 9), sn2=0.05)
    check_fit(lib, p, bar=bar, precision=precision)


# partition kernels: sums in the documented order bit for bit (chunks of 4096 points,
# groups of eight centres), counts in LDS up to 2048 centres and global beyond, the
# sort's ranks over chunk and wave edges
@pytest.mark.parametrize("n,k,d", [(1, 1, 1), (63, 7, 3), (65, 8, 2), (4096, 9, 64), (4097, 17, 1), (12300, 300, 5),
                                   (262145, 33, 2)])
def test_centre_update_bit_for_bit(lib, n, k, d):
    rng = np.random.default_rng(n + k)
    P, C = rng.standard_normal((n, d)), rng.standard_normal((k, d))
    label = rng.integers(-1, k + 1, size=n).astype(np.int32)  # labels outside 0..k-1 count for no centre
    label[label == k // 2] = (k // 2 + 1) % k                 # a centre without points
    sums, count = np.zeros((k, d)), np.zeros(k, dtype=np.int64)
    for a in range(0, n, 4096):
        lab, Q = label[a:a + 4096], P[a:a + 4096]
        ok = (lab >= 0) & (lab < k)
        count += np.bincount(lab[ok], minlength=k)
        sums += np.stack([np.bincount(lab[ok], weights=Q[ok, t], minlength=k) for t in range(d)], axis=1)
    want = np.where(count[:, None] > 0, sums / np.maximum(count, 1)[:, None], C)
    got, cnt = lib.kmeans_update(P, label, C)
    assert np.array_equal(cnt.cpu().numpy(), count) and np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n,k,d,lo,hi", [(64, 3, 2, 0, 64), (1025, 40, 3, 10, 40), (4700, 2100, 2, 1, 3),
                                         (70000, 20, 2, 3000, 4000)])
def test_partition_steps_equal_the_oracle(lib, n, k, d, lo, hi):
    from oracle import kmeans as okm
    from oracle import partition as opart
    rng = np.random.default_rng(n + k)
    P = np.round(rng.uniform(size=(n, d)), 3)     # ties among distances
    C = P[rng.choice(n, size=k, replace=False)]
    lab, dist = lib.kmeans_assign(P, C)
    lo_, do = okm.assign(P, C)
    assert np.array_equal(lab.cpu().numpy(), lo_) and np.array_equal(dist.cpu().numpy(), do)
    lab, cnt, _ = lib.bounded_assign(P, C, lo, hi)
    want = opart.bounded_assign(P, C, lo, hi)
    want = want[0] if isinstance(want, tuple) else want
    assert np.array_equal(lab.cpu().numpy(), want)


# encoder kernels: sets that end inside a 64-point piece, a 128-point tile with an empty
# half, one point, and more pieces than workgroups; tolerances of the network's oracle
# test (float32 accumulation and bfloat16 rounding flips); a backward pass that follows
# a parameter update uses the activations of its own forward pass
@pytest.mark.parametrize("sizes", [[1], [63, 64, 65], [128, 129, 1, 191], [4096] * 5 + [77]])
def test_network_piece_edges(sizes):
    import torch
    from paper_1411_4510_amd import warmstart as ws
    rng = np.random.default_rng(sum(sizes))
    ptr, sn = ws.aligned_layout(sizes)
    feats = rng.standard_normal((int(ptr[-1]), ws.NFEAT)).astype(np.float32)  # padding rows hold values too
    params = ws.he_init(3)
    labels = rng.standard_normal((len(sizes), ws.NOUT)).astype(np.float32)
    masks = np.ones_like(labels)
    net = ws.Network(max_rows=int(ptr[-1]), max_sets=len(sizes))
    net.set_params(params)
    out = net.forward(torch.as_tensor(feats, device="cuda"), ptr, sn).cpu().numpy()
    _, grad = net.backward(labels, masks, want_grad=True)
    net.adam(0.1)
    net.adam(0.1)
    _, after = net.backward(labels, masks, want_grad=True)
    p = ws.unpack(params)
    X = torch.as_tensor(feats, dtype=torch.float64)
    w = {k: torch.tensor(v, dtype=torch.float64, requires_grad=True) for k, v in p.items()}
    outs = []
    for b, n in enumerate(sizes):
        x = X[int(ptr[b]):int(ptr[b]) + n]
        h = torch.relu(torch.relu(x @ w["W1"].T + w["b1"]) @ w["W2"].T + w["b2"]).mean(0)
        outs.append(torch.relu(w["W3"] @ h + w["b3"]) @ w["W4"].T + w["b4"])
    ref = torch.stack(outs)
    ((ref - torch.as_tensor(labels)) ** 2).mean(1).mean().backward()
    # against the network without bfloat16 roundings: 2^-9 per operand, five operands deep
    assert rel(out, ref.detach().numpy()) < 5 * 2.0 ** -8
    g = ws.unpack(grad.cpu().numpy())
    for k in g:
        assert rel(g[k], w[k].grad.numpy()) < 10 * 2.0 ** -8, k
    assert np.all(np.isfinite(after.cpu().numpy()))


# products split along k: one window of 24 column tiles (few tiles per launch), eight of 9
# with a ragged test set, tiles left over from full turns of the CUs
@pytest.mark.parametrize("precision,bar", [("fp64", BAR), ("mixed", 1e-4)])
@pytest.mark.parametrize("n,M,B,s,n_u", [(3000, 1, 0, 60, 100), (3000, 2, 1, 60, 100), (3400, 9, 8, 140, 500)])
def test_products_split_along_k(lib, n, M, B, s, n_u, precision, bar):
    p = synth.make_random(seed=n + M, n=n, d=3, M=M, s=s, n_u=n_u, B=B, uneven=(n // M - 30, n // M + 30), sn2=0.05)
    check_fit(lib, p, bar=bar, precision=precision)
