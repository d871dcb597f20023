"""The push kernels with every table in LDS (what a tuned plan may take) against
those that read the contribution rows through the caches: the same bits, over the
forms of the visible phase, both precisions and the edges of steps and
workgroups."""
import numpy as np
import pytest

from paper_2311_02101_amd import hp, workload as wl
from tests.parity import say

pytestmark = pytest.mark.gpu


# one variable per thread, then 1, 2 and (FP32) 4 groups of four in registers, then
# averages in global memory; the chains (or 1024 threads) make the automatic choice
# the wide layout
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("n,k,chains,threads", [
    (63, 7, 2, 1024), (64, 3, 3, 1024), (1024, 7, 1, 1024),                      # one variable per thread
    (65, 7, 800, 64), (256, 3, 800, 64), (64, 7, 4000, 64), (1025, 7, 1, 1024),  # one group
    (257, 7, 800, 64), (512, 3, 800, 64),                                        # two groups
    (513, 7, 800, 64), (1024, 3, 800, 64), (1025, 7, 800, 64), (4097, 3, 600, 256)])   # four or none
def test_layouts_agree(hip, n, k, chains, threads, precision):
    T = wl.random_formula(n, 61, k=k, lengths=[1, 2, 3] if k == 3 else wl.LENGTHS,
                          probs=[0.2, 0.5, 0.3] if k == 3 else wl.LENGTH_PROBS)
    W, b, _ = wl.pretrained_rbm(k, wl.FSTAR_PAIR)
    v0 = [wl.initial_state(chains, n, 61)]
    got = []
    for kernel, kind in (("auto", 1), ("push", 0)):
        plan = hp.Plan([T], [n], W, b, chains=chains, temps=wl.default_temperatures(chains, 2), precision=precision,
                       seed=61, threads=threads, kernel=kernel, split=1)
        info = plan.info()
        say(f"[layouts] n={n} k={k} chains={chains} threads={threads} {precision} kind={info['bucket_kind']}")
        assert info["bucket_kind"] == [kind] and info["bucket_threads"] == [threads]
        st = plan.new_state(v0)
        for S in (3, 0, 4):
            plan.run(st, S)
        got.append(st.formula(0))
        plan.free()
    for a, c in zip(*got):
        assert np.array_equal(a, c)


# the steps of a clause phase from the counter, several sweeps a run: an odd number
# of steps, more waves than pairs of steps (the size-clustered model counts for any
# number on 1024 threads), against one wave
@pytest.mark.parametrize("n", [10, 33, 75, 350, 1500])
def test_counted_steps(hip, n):
    T = wl.random_formula(n, 62)
    W, b, _ = wl.pretrained_rbm(7, wl.FSTAR_PAIR)
    rbms = wl.pretrained_size_rbms(wl.FSTAR_PAIR, 7)
    lens = np.array([len(set(c)) for c in T.T])
    steps = sum(-(-int((lens == v).sum()) // 64) for v in set(lens))
    got = []
    for t in (64, 1024):
        plan = hp.Plan([T], [n], W, b, chains=3, temps=wl.default_temperatures(3, 2), seed=62, threads=t, split=1,
                       size_rbms=rbms)
        say(f"[steps] n={n} threads={t} steps={steps} dyn={plan.info()['bucket_dyn']}")
        assert plan.info()["bucket_dyn"] == [int(t == 1024)]
        st = plan.new_state([wl.initial_state(3, n, 62)])
        for S in (5, 1, 6):
            plan.run(st, S)
        got.append(st.formula(0))
        plan.free()
    for a, c in zip(*got):
        assert np.array_equal(a, c)


# split members of fewer than 1024 threads keep their rows in LDS and take their
# steps round-robin: against one workgroup of the same size
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("n,k,chains,threads,split", [(65, 7, 3, 64, 2), (257, 7, 2, 128, 16), (300, 3, 40, 64, 4),
                                                      (1027, 7, 2, 64, 2), (2100, 3, 3, 512, 4), (451, 7, 2, 256, 0)])
def test_split_members_of_few_waves(hip, n, k, chains, threads, split, precision):
    T = wl.random_formula(n, 63, k=k, lengths=[1, 2, 3] if k == 3 else wl.LENGTHS,
                          probs=[0.2, 0.5, 0.3] if k == 3 else wl.LENGTH_PROBS)
    W, b, _ = wl.pretrained_rbm(k, wl.FSTAR_PAIR)
    got = []
    for sp in (1, split):
        plan = hp.Plan([T], [n], W, b, chains=chains, temps=wl.default_temperatures(chains, 2), precision=precision,
                       seed=63, threads=threads, split=sp)
        say(f"[few waves] n={n} k={k} chains={chains} threads={threads} {precision} split={plan.split}")
        assert (plan.split > 1) == (sp != 1)
        st = plan.new_state([wl.initial_state(chains, n, 63)])
        for S in (3, 0, 4):
            plan.run(st, S)
        plan.check()
        got.append(st.formula(0))
        plan.free()
    for a, c in zip(*got):
        assert np.array_equal(a, c)
