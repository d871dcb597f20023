"""Pull formulas with variables of far more clauses than their neighbours, whose
lists are summed by a wave: lengths on either side of the limit of 16 and of the 64
entries taken at a time, several in one slice, averages in registers and in global
memory."""
import numpy as np
import pytest

from oracle import rbmsat as R
from paper_2311_02101_amd import hp, workload as wl
from tests.parity import compare_state, say, teacher_forced_sweep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,threads,hubs,precision", [
    (320, 64, {1: 16, 2: 17, 70: 63}, "f64"), (320, 128, {64: 64, 65: 65, 320: 220}, "f32"),
    (321, 64, {3: 128, 4: 129, 60: 17, 321: 200}, "f32"), (257, 512, {257: 219, 128: 191}, "f64")])
def test_long_lists(hip, n, threads, hubs, precision):
    rng = np.random.default_rng(n)
    C, k = 220, 5
    T = np.stack([rng.permutation(n)[:k] + 1 for _ in range(C)], axis=1).astype(np.int32)
    row = np.zeros(C, dtype=int)                     # hubs take a clause's slots from the first on
    T[np.isin(T, list(hubs))] = next(v for v in range(1, n + 1) if v not in hubs)
    for v, d in hubs.items():
        on = rng.permutation(np.flatnonzero(row < k - 1))[:d]
        T[row[on], on] = v
        row[on] += 1
    T *= rng.choice([-1, 1], T.shape).astype(np.int32)
    for i in range(C):                               # distinct literals only: no padding copies
        while len(set(T[:, i])) < k:
            T[k - 1, i] = rng.integers(1, n + 1) * rng.choice([-1, 1])
    W, b, _ = wl.pretrained_rbm(k, wl.FSTAR_PAIR)
    chains = 3
    temps = wl.default_temperatures(chains, 2)
    v0 = wl.initial_state(chains, n, 52)
    plan = hp.Plan([T], [n], W, b, chains=chains, temps=temps, precision=precision, seed=52, threads=threads,
                   kernel="pull")
    st = plan.new_state([v0])
    op, ost = R.plan(T, n, W, b), R.initial(v0)
    say(f"[pull lists] n={n} threads={threads} hubs={hubs} {precision}")
    if precision == "f32":
        for _ in range(4):
            teacher_forced_sweep(plan, st, 0, ost, op, temps, alpha=1e-3, seed=52, prec="f32")
    else:
        for S in (4, 0, 6):
            plan.run(st, S)
            if S:
                ost = R.run(ost, op, temps, S, alpha=1e-3, seed=52)
        compare_state(st.formula(0), (ost.v, ost.nu, ost.s_max, ost.best), "f64", f"n={n}", 1e-13)
    plan.free()
