"""The library's host path on a stub of the HIP runtime (no GPU)."""
import pytest

from tests.host_path import run


# A run that needs counters or mailboxes notes and advances the sweep counter
# first; if a launch behind that fails, no sweep ran and the counter is as before
@pytest.mark.parametrize("kwargs,n,chains,failing", [
    ("dict()", 4096, 8, "sweep_split_kernel"),                       # split
    ("dict(split=1)", 300, 4000, "sweep_push_kernel"),               # persistent grid
    ("dict()", 14000, 4, "sweep_push_kernel"),                       # joined split, the launch behind it
    ("dict(split=1)", 300, 2, "sweep_push_kernel")])                 # neither: the counter goes last
def test_counter_of_a_failed_run(tmp_path, kwargs, n, chains, failing):
    got = run(tmp_path, f"""
T = wl.random_formula({n}, 5)
W, b, _ = wl.pretrained_rbm(7, wl.FSTAR_PAIR)
p = Plan([T], [{n}], W, b, chains={chains}, **{kwargs})
st = p.state()
kernels()
out = dict(ok=p.call("hp_run", ct.byref(st), ct.c_int64(7)), t=int(p.t[0]), names=kernels())
for name in ("hp_run", "hp_run_noalloc"):
    stub.stub_fail({failing!r}.encode())
    out[name] = [p.call(name, ct.byref(st), ct.c_int64(5)), int(p.t[0])]
    stub.stub_fail(b"")
    out[name] += [p.call(name, ct.byref(st), ct.c_int64(1)), int(p.t[0])]
""")
    assert any(failing in k for k in got["names"]), got["names"]
    assert got["ok"] == 0 and got["t"] == 7
    assert got["hp_run"] == [-3, 7, 0, 8]
    assert got["hp_run_noalloc"] == [-3, 8, 0, 9]


# A variable in every clause must not pad its neighbours' lists to its own
# length: pull formulas with such variables cost the device memory of their
# occurrences (four times at most, here with one in every slice of 64 variables)
@pytest.mark.parametrize("every", [0, 1, 64])
def test_device_memory_of_pull_lists(tmp_path, every):
    got = run(tmp_path, f"""
n, c, k = 4096, 20000, 3
rng = np.random.default_rng(1)
T = rng.integers(1, n + 1, (k, c)).astype(np.int32)
hubs = 1 if {every} == 1 else n // 64
if {every}:
    T[1] = rng.integers(0, hubs, c) * 64 + 1
W, b, _ = wl.pretrained_rbm(k, wl.FSTAR_PAIR)
free = stub.stub_bytes()
p = Plan([T], [n], W, b, chains=2, kernel="pull")
pull = stub.stub_bytes() - free
q = Plan([T], [n], W, b, chains=2, kernel="push", split=1)
out = dict(pull=pull, push=stub.stub_bytes() - free - pull, occurrences=k * c, n=n)
""")
    lists = got["pull"] - got["push"]
    assert lists <= 4 * (4 * got["occurrences"] + 20 * got["n"])
