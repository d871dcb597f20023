"""Returned assignments that lie in the same memory as the state's: a history buffer
of which the state is one window."""
import numpy as np
import pytest

from oracle import up as U
from paper_2311_02101_amd import hp, workload as wl
from tests.parity import say

pytestmark = pytest.mark.gpu


# shifts by columns, by a row and by the other direction; 1024 workgroups of
# columns, more than run at once
@pytest.mark.parametrize("shift", [64, -64, 1, 16384, -16384])
def test_candidates_overlapping_the_state(hip, shift):
    import torch
    n, B, F = 16384, 256, 2
    rng = np.random.default_rng(abs(shift))
    tables = [(rng.integers(1, n + 1, (3, 400)) * rng.choice([-1, 1], (3, 400))).astype(np.int32) for _ in range(F)]
    W, b, _ = wl.pretrained_rbm(3, wl.FSTAR_PAIR)
    plan = hp.Plan(tables, [n] * F, W, b, chains=B, temps=wl.default_temperatures(B, 2), precision="f32", seed=3)
    st = plan.new_state([np.zeros((B, n), np.uint8)] * F)
    size = F * B * n
    buf = torch.from_numpy(rng.integers(0, 2, size + abs(shift)).astype(np.uint8)).cuda()
    st.v = buf[max(shift, 0):max(shift, 0) + size]
    cand = buf[max(-shift, 0):max(-shift, 0) + size]
    st.nu.copy_(torch.from_numpy(rng.random(size).astype(np.float32)))
    before = [st.formula(f) for f in range(F)]
    rows = cand.cpu().numpy().reshape(F, B, n)
    say(f"[merge overlap] shift={shift}")
    plan.merge_candidates(st, cand)
    torch.cuda.synchronize()
    for f in range(F):
        want_v, want_nu = U.merge_topb(tables[f], n, before[f][0], before[f][1], rows[f])
        v, nu, _, _ = st.formula(f)
        assert np.array_equal(v, want_v) and np.array_equal(nu, want_nu)
    plan.free()
