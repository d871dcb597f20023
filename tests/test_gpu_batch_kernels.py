"""The kernels that go over all variables of a batch in tiles of 1024: features,
initial draws and chain means, at the tiles' edges and odd row starts."""
import ctypes as ct

import numpy as np
import pytest

from oracle import learned as M
from paper_2311_02101_amd import workload as wl
from tests.parity import say

pytestmark = pytest.mark.gpu


def _plan(tables, ns, chains, seed=3, precision="f32"):
    from paper_2311_02101_amd import hp
    K = tables[0].shape[0]
    W, b = wl.gaussian_rbm(2, K, wl.hidden_units_for(K), seed)
    return hp.Plan(tables, ns, W, b, chains=chains, precision=precision, seed=seed)


# exact: the features are small dyadic numbers, rounded once to bfloat16
@pytest.mark.parametrize("sizes,skew", [([7, 1023, 1024, 1025, 9], 0), ([2049, 8], 1)])
def test_features_at_tile_edges(hip, sizes, skew):
    import torch
    from paper_2311_02101_amd import learned as Lr
    tables = [wl.random_formula(n, 31, tag=f) for f, n in enumerate(sizes)]
    plan = _plan(tables, sizes, 2)
    buf = torch.zeros(sum(sizes) * M.F_IN + 8, dtype=torch.int16, device="cuda")
    x = buf[skew:skew + sum(sizes) * M.F_IN]           # skew 1: rows at two-byte alignment only
    say(f"[features] sizes={sizes} skew={skew}")
    assert Lr._lib().hp_features(plan._h, ct.c_void_p(x.data_ptr()), Lr._stream()) == 0
    torch.cuda.synchronize()
    got = (x.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    want = np.concatenate([M.bf16_round(M.features(t, n)) for t, n in zip(tables, sizes)])
    assert np.array_equal(got.reshape(-1, M.F_IN), want)
    assert not buf[:skew].any() and not buf[skew + sum(sizes) * M.F_IN:].any()
    plan.free()


# exact: the draws are integers, the means a sum of bytes divided once
@pytest.mark.parametrize("sizes,chains,lo,hi", [([7, 1023, 1024, 1025, 9], 5, 1, 5), ([2049, 8, 10], 67, 0, 66)])
def test_initial_draws_and_means_at_tile_edges(hip, sizes, chains, lo, hi):
    import torch
    from paper_2311_02101_amd import learned as Lr
    tables = [wl.random_formula(n, 32, tag=f) for f, n in enumerate(sizes)]
    plan = _plan(tables, sizes, chains, seed=6)
    v0 = [wl.initial_state(chains, n, 6, tag=f) for f, n in enumerate(sizes)]
    st = plan.new_state(v0)
    q = torch.tensor(np.random.default_rng(1).uniform(0, 1, sum(sizes)).astype(np.float32), device="cuda")
    say(f"[init chains] sizes={sizes} chains {lo}..{hi} of {chains}")
    Lr.init_chains(plan, q, st, lo, hi)
    mean = Lr.chain_mean(plan, st.v)
    torch.cuda.synchronize()
    qh = q.cpu().numpy().astype(np.float64)
    off = np.concatenate([[0], np.cumsum(sizes)])
    for f, n in enumerate(sizes):
        v = st.formula(f)[0]
        assert np.array_equal(v[lo:hi], M.init_assignment(qh[off[f]:off[f + 1]], 6, f, np.arange(lo, hi)))
        assert np.array_equal(v[:lo], v0[f][:lo]) and np.array_equal(v[hi:], v0[f][hi:])
        want = v.sum(axis=0, dtype=np.int64).astype(np.float32) / np.float32(chains)
        assert np.array_equal(mean.cpu().numpy()[off[f]:off[f + 1]], want)
    plan.free()


# exact: counts are integers and kept rows are copies.  Chains at the edges of
# the 32-chain words and of the in-place permutation (256), columns at the edges
# of its 64-column slabs, clauses at the edge of a tile of 8192
@pytest.mark.parametrize("sizes,B,precision,alias", [([63, 64, 65], 1, "f64", False), ([1025, 9], 33, "f32", False),
                                                     ([1366, 70], 64, "f64", True), ([100, 30], 256, "f32", False),
                                                     ([40, 100], 257, "f64", False)])
def test_merge_at_tile_edges(hip, sizes, B, precision, alias):
    import torch
    from oracle import up as U
    tables = [wl.random_formula(n, 41, tag=f) for f, n in enumerate(sizes)]
    plan = _plan(tables, sizes, B, seed=4, precision=precision)
    st = plan.new_state([wl.initial_state(B, n, 4, tag=f) for f, n in enumerate(sizes)])
    plan.run(st, 2)
    torch.cuda.synchronize()
    rng = np.random.default_rng(B)
    before = [st.formula(f) for f in range(len(sizes))]
    parts = [rng.integers(0, 2, (B, n)).astype(np.uint8) for n in sizes]
    for f in range(len(sizes)):
        parts[f][B // 2] = before[f][0][B // 3]          # equal counts
    if alias:
        parts = [x[0] for x in before]
    cand = st.v if alias else torch.tensor(np.concatenate([c.ravel() for c in parts]), device="cuda")
    say(f"[merge] sizes={sizes} B={B} {precision} alias={alias}")
    plan.merge_candidates(st, cand)
    torch.cuda.synchronize()
    for f, n in enumerate(sizes):
        want_v, want_nu = U.merge_topb(tables[f], n, before[f][0], before[f][1], parts[f])
        v, nu, s_max, best = st.formula(f)
        assert np.array_equal(v, want_v) and np.array_equal(nu, want_nu)
        assert np.array_equal(s_max, before[f][2]) and np.array_equal(best, before[f][3])
    plan.free()


# rows at the edges of a tile of 32, a step of 128 and the 512 workgroups; the
# bounds are those of the initializer's parity tests (FP32 sums of 256 products)
@pytest.mark.parametrize("rows", [1, 31, 32, 127, 128, 129, 512 * 128, 512 * 128 + 1])
def test_perceptron_rows_at_step_edges(hip, rows):
    import torch
    from paper_2311_02101_amd import learned as Lr
    net = Lr.MLP(seed=17)
    rng = np.random.default_rng(rows)
    xf = M.bf16_round(rng.standard_normal((rows, M.F_IN)))
    y = rng.uniform(0, 1, rows).astype(np.float32)
    bits = torch.tensor((xf.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).view(np.int16), device="cuda")
    p = net.host_params()
    n1 = M.F_IN * M.HIDDEN
    params = (p[:n1].reshape(M.F_IN, M.HIDDEN), p[n1:n1 + M.HIDDEN], p[n1 + M.HIDDEN:n1 + 2 * M.HIDDEN], p[-1])
    say(f"[mlp] rows={rows}")
    q = net.forward(bits)
    loss = net.backward(bits, torch.tensor(y, device="cuda"))
    torch.cuda.synchronize()
    want, _ = M.forward(xf, *params)
    assert np.max(np.abs(q.cpu().numpy() - want)) < 2e-6
    g = M.gradients(xf, y.astype(np.float64), *params)
    got = net.grad.cpu().numpy().astype(np.float64)
    parts = dict(W1=got[:n1].reshape(M.F_IN, M.HIDDEN), b1=got[n1:n1 + M.HIDDEN],
                 w2=got[n1 + M.HIDDEN:n1 + 2 * M.HIDDEN], b2=got[-1:])
    for k, v in parts.items():
        assert np.max(np.abs(v - g[k])) < 1e-4 * max(np.max(np.abs(g[k])), 1e-30), k
    want_loss = M.loss(xf, y.astype(np.float64), *params) * rows
    assert abs(float(loss.item()) - want_loss) < 1e-5 * abs(want_loss)
