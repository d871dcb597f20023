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
