"""Batches of many small formulas: the exchange and the merge take smaller launches
there, the same results (more than 512 chains: counts ranked without staging)."""
import numpy as np
import pytest

from oracle import up as U
from paper_2311_02101_amd import hp, workload as wl
from tests.parity import say
from tests.test_gpu_temper import _check_round

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,B,precision", [([12] * 70 + [5, 16], 8, "f64"), ([64, 11, 85], 33, "f32"),
                                               ([20], 600, "f64")])
def test_merge_of_small_formulas(hip, sizes, B, precision):
    import torch
    tables = [wl.random_formula(n, 71, k=3, lengths=[1, 2, 3], probs=[0.2, 0.5, 0.3], tag=f)
              for f, n in enumerate(sizes)]
    W, b, _ = wl.pretrained_rbm(3, wl.FSTAR_PAIR)
    plan = hp.Plan(tables, sizes, W, b, chains=B, temps=wl.default_temperatures(B, 2), precision=precision, seed=7)
    st = plan.new_state([wl.initial_state(B, n, 7, tag=f) for f, n in enumerate(sizes)])
    plan.run(st, 2)
    rng = np.random.default_rng(B)
    parts = [rng.integers(0, 2, (B, n)).astype(np.uint8) for n in sizes]
    before = [st.formula(f) for f in range(len(sizes))]
    say(f"[tiny merge] {len(sizes)} formulas, B={B} {precision}")
    plan.merge_candidates(st, torch.tensor(np.concatenate([c.ravel() for c in parts]), device="cuda"))
    torch.cuda.synchronize()
    for f, n in enumerate(sizes):
        want_v, want_nu = U.merge_topb(tables[f], n, before[f][0], before[f][1], parts[f])
        v, nu, _, _ = st.formula(f)
        assert np.array_equal(v, want_v) and np.array_equal(nu, want_nu)
    plan.free()


# one, two and four waves a chain
@pytest.mark.parametrize("sizes", [[5, 10], [10, 21], [40, 7]])
def test_exchange_of_small_formulas(hip, sizes):
    import torch
    tables = [wl.random_formula(n, 72, k=5, lengths=[1, 2, 3, 4, 5], probs=[0.2] * 5, tag=f)
              for f, n in enumerate(sizes)]
    W, b, _ = wl.pretrained_rbm(5, wl.FSTAR_PAIR)
    temps = np.array([0, 1, 1, 0, 1, 0, 0], np.int32)
    plan = hp.Plan(tables, sizes, W, b, chains=7, temps=temps, precision="f64", seed=9)
    st = plan.new_state([wl.initial_state(7, n, 9, tag=f) for f, n in enumerate(sizes)])
    say(f"[tiny exchange] {sizes}")
    for r in range(4):
        plan.run(st, 1)
        torch.cuda.synchronize()
        _check_round(plan, st, tables, sizes, W, b, 0, 9)
    plan.free()
