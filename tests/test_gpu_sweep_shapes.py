"""Launch shapes of the sweep kernels where they can go wrong: one variable per
thread (formulas up to the workgroup's size, on either side of the edge), and
clause phases of few steps for many waves (waves with no step, an odd last one)."""
import numpy as np
import pytest

from oracle import rbmsat as R
from paper_2311_02101_amd import hp, workload as wl
from tests.parity import compare_state, f64_bounds, say, teacher_forced_sweep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,chains,threads,precision", [
    (7, 7, 2, 1024, "f64"), (63, 7, 1, 64, "f64"), (64, 7, 3, 64, "f32"), (65, 7, 3, 64, "f64"),
    (255, 3, 2, 256, "f32"), (1024, 7, 1, 1024, "f32"), (1024, 3, 2, 1024, "f64"), (1025, 7, 1, 1024, "f64"),
    (130, 7, 300, 256, "f64")])
def test_small_formulas_on_many_threads(hip, n, k, chains, threads, precision):
    T = wl.random_formula(n, 51, k=k, lengths=[1, 2, 3] if k == 3 else wl.LENGTHS,
                          probs=[0.2, 0.5, 0.3] if k == 3 else wl.LENGTH_PROBS)
    W, b, _ = wl.pretrained_rbm(k, wl.FSTAR_PAIR)
    temps = wl.default_temperatures(chains, 2)
    v0 = wl.initial_state(chains, n, 51)
    plan = hp.Plan([T], [n], W, b, chains=chains, temps=temps, precision=precision, seed=51, threads=threads, split=1)
    st = plan.new_state([v0])
    op, ost = R.plan(T, n, W, b), R.initial(v0)
    say(f"[shapes] n={n} k={k} chains={chains} threads={threads} {precision}")
    if precision == "f32":
        for _ in range(4):
            teacher_forced_sweep(plan, st, 0, ost, op, temps, alpha=1e-3, seed=51, prec="f32")
    else:
        for S in (5, 0, 7):                      # the pipe restarts with every run
            plan.run(st, S)
            if S:
                ost = R.run(ost, op, temps, S, alpha=1e-3, seed=51)
        compare_state(st.formula(0), (ost.v, ost.nu, ost.s_max, ost.best), "f64", f"n={n}",
                      f64_bounds(plan, [T])[1])
    plan.free()


# pull: slices of 64 variables and their edges, more than four variables per
# thread (averages in global memory), one Philox block per clause, and a variable
# that sits in most clauses (its slice's lists padded to its length)
@pytest.mark.parametrize("n,k,threads,hub,precision", [
    (63, 7, 64, False, "f64"), (65, 7, 64, False, "f32"), (300, 7, 64, False, "f64"), (257, 3, 64, False, "f32"),
    (513, 7, 256, True, "f64"), (130, 3, 128, True, "f32")])
def test_pull_slices(hip, n, k, threads, hub, precision):
    T = wl.random_formula(n, 52, k=k, lengths=[1, 2, 3] if k == 3 else wl.LENGTHS,
                          probs=[0.2, 0.5, 0.3] if k == 3 else wl.LENGTH_PROBS)
    if hub:
        T[:, ::2] = np.where(T[:, ::2] == T[:1, ::2], np.sign(T[:1, ::2]) * (n - 1), T[:, ::2])
    W, b, _ = wl.pretrained_rbm(k, wl.FSTAR_PAIR)
    chains = 3
    temps = wl.default_temperatures(chains, 2)
    v0 = wl.initial_state(chains, n, 52)
    plan = hp.Plan([T], [n], W, b, chains=chains, temps=temps, precision=precision, seed=52, threads=threads,
                   kernel="pull")
    st = plan.new_state([v0])
    op, ost = R.plan(T, n, W, b), R.initial(v0)
    say(f"[pull] n={n} k={k} threads={threads} hub={hub} {precision}")
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


# formulas whose tables do not fit in LDS beside them (above 13 600 variables) split
# as far as hp_run_noalloc's scratch goes, and no call of theirs is refused
@pytest.mark.parametrize("n,chains,precision", [(14000, 2, "f64"), (16384, 9, "f32"), (16500, 64, "f64")])
def test_large_formulas_split_like_one_workgroup(hip, n, chains, precision):
    T = wl.random_formula(n, 53)
    W, b, _ = wl.pretrained_rbm(7, wl.FSTAR_PAIR)
    temps = wl.default_temperatures(chains, 2)
    v0 = [wl.initial_state(chains, n, 53)]
    out = []
    for split, noalloc in ((1, False), (0, False), (0, True)):
        plan = hp.Plan([T], [n], W, b, chains=chains, temps=temps, precision=precision, seed=53, split=split)
        say(f"[large split] n={n} chains={chains} {precision} split={plan.split} noalloc={noalloc}")
        st = plan.new_state(v0)
        (plan.run_noalloc if noalloc else plan.run)(st, 3)
        plan.check()
        out.append(st.formula(0) + (plan.split,))
        plan.free()
    assert out[0][4] == 1 and (out[1][4] > 1 or chains == 64)
    for got in out[1:]:
        for a, c in zip(out[0][:4], got[:4]):
            assert np.array_equal(a, c)
