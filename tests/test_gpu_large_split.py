"""Formulas above 13 600 variables split by default, and may share the device all
the same: the workgroups of a chain join before its first sweep, and a chain that
does not get together runs in one workgroup with the same bits."""
import numpy as np
import pytest

from paper_2311_02101_amd import hp, workload as wl
from tests.parity import say

pytestmark = pytest.mark.gpu


def _plan(T, n, chains, precision, **kw):
    W, b, _ = wl.pretrained_rbm(7, wl.FSTAR_PAIR)
    return hp.Plan([T], [n], W, b, chains=chains, temps=wl.default_temperatures(chains, 2), precision=precision,
                   seed=53, **kw)


def _states_equal(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


# limit 1: members wait for two reloads, so chains are left to one workgroup;
# the run is not void and hp_check has nothing to report
@pytest.mark.parametrize("n,chains,precision,members", [(14000, 2, "f64", 16), (14001, 31, "f32", 4),
                                                        (16384, 9, "f32", 8), (17000, 1, "f64", 16)])
def test_members_that_do_not_join(hip, n, chains, precision, members):
    T = wl.random_formula(n, 53)
    v0 = [wl.initial_state(chains, n, 53)]
    one = _plan(T, n, chains, precision, split=1)
    st = one.new_state(v0)
    for S in (2, 0, 1):
        one.run(st, S)
    want, t = st.formula(0), st.get_t()
    one.free()
    for limit in (1, 0):
        for noalloc in (False, True):
            plan = _plan(T, n, chains, precision, split_wait_limit=limit)
            say(f"[large split] n={n} chains={chains} {precision} split={plan.split} limit={limit} noalloc={noalloc}")
            assert plan.split == members
            st = plan.new_state(v0)
            for S in (2, 0, 1):
                (plan.run_noalloc if noalloc else plan.run)(st, S)
            plan.check()
            assert st.get_t() == t and _states_equal(want, st.formula(0))
            plan.free()


# a device whose compute units are taken by another stream's run
def test_large_split_beside_other_work(hip):
    import torch
    n, chains = 14000, 16
    T = wl.random_formula(n, 53)
    v0 = [wl.initial_state(chains, n, 53)]
    other = _plan(T, n, 256, "f32", split=1)
    busy = other.new_state([wl.initial_state(256, n, 54)])
    one, plan = _plan(T, n, chains, "f32", split=1), _plan(T, n, chains, "f32")
    assert plan.split > 1
    st1, st = one.new_state(v0), plan.new_state(v0)
    one.run(st1, 4)
    torch.cuda.synchronize()
    say(f"[large split] beside another run, split={plan.split}")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    other.run(busy, 100, stream=side)
    plan.run(st, 4)
    plan.check()
    assert _states_equal(st1.formula(0), st.formula(0))
    for p in (other, one, plan):
        p.free()


# 64 chains of 16384 variables: the mailboxes of two members would exceed the
# scratch of the allocation-free entry, which took these chains unsplit
def test_split_bounded_by_scratch(hip):
    T = wl.random_formula(16384, 53)
    plan = _plan(T, 16384, 64, "f32")
    assert plan.split == 1
    plan.free()


def test_explicit_split_of_large_formulas_is_refused(hip):
    T = wl.random_formula(14000, 53)
    with pytest.raises(hp.HpError, match="tables fit in LDS") as e:
        _plan(T, 14000, 2, "f64", split=2)
    assert e.value.status == hp.HP_EUNSUPPORTED
