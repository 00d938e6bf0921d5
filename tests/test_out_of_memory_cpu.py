"""Set-up calls whose GPU scratch does not fit: the host builder needs none, so a host CSR is built there.
The library runs against a device of host memory (fake_hip) in a process of its own; no GPU calls."""
import pathlib
import subprocess
import sys

import pytest

ROOT = pathlib.Path(__file__).resolve().parent.parent

SCRIPT = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the library looks its symbols up
import numpy as np
import paper_2605_15695_amd as pc
from paper_2605_15695_amd import binding

n, deg = 30000, 8                                          # past the size the GPU is used from
assert n * deg >= 200000
rng = np.random.default_rng(5)
rows = [np.sort(rng.choice(n, deg, replace=False)) for _ in range(n)]
rows[1:n // 2:2] = rows[0:n // 2:2]                        # half of the row pairs share their columns
colidx = np.concatenate(rows).astype(np.int32)
rowptr = np.arange(0, n * deg + 1, deg, dtype=np.int32)
vals = rng.random(n * deg).astype(np.float32)
kw = dict(V=2, S=1, SG=4)


def same(h, ref):
    e, r = pc.pcsr_export(h), pc.pcsr_export(ref)
    return all(np.array_equal(e[k], r[k]) for k in r)


host = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(flags=pc.PCSR_FLAG_HOST_ONLY, **kw))
row = np.repeat(np.arange(n, dtype=np.int32), deg)
at = np.lexsort((row, colidx))
t = np.concatenate([[0], np.cumsum(np.bincount(colidx, minlength=n))]).astype(np.int32), row[at], vals[at]
host_t = pc.pcsr_build(n, n, *t, pc.make_params(flags=pc.PCSR_FLAG_HOST_ONLY, **kw))
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    lib = tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so"
    subprocess.run(["g++", "-O1", "-fPIC", "-shared", "-o", str(lib), str(ROOT / "tests/fake_hip/fake_hip.cpp")], check=True)
    return lib


def _run(fake, body):
    r = subprocess.run([sys.executable, "-c", SCRIPT + body, str(fake)], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]


# the upload's three arrays, then the first of the build's own
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_build_falls_back_to_the_host(fake, k):
    _run(fake, f"""
fake.fake_hip_fail({k}, {k})
h = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(**kw))
assert fake.fake_hip_allocations() > {k} and same(h, host)
h.close()
""")


def test_build_reports_what_fits_nowhere(fake):
    _run(fake, """
fake.fake_hip_fail(1, 1 << 30)                             # the product's own arrays neither
for flags in (0, pc.PCSR_FLAG_GPU_BUILD):
    try:
        pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(flags=flags, **kw))
        assert False
    except pc.PcsrError as e:
        assert e.code == binding.PCSR_E_OOM
assert fake.fake_hip_live() == 0
""")


def test_build_on_the_gpu_is_not_replaced_where_it_was_asked_for(fake):
    _run(fake, """
fake.fake_hip_fail(2, 2)
try:
    pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(flags=pc.PCSR_FLAG_GPU_BUILD, **kw))
    assert False
except pc.PcsrError as e:
    assert e.code == binding.PCSR_E_OOM
""")


# refused: what the upload of rowptr asks for, not the product's arrays
@pytest.mark.parametrize("transpose", [True, False])
def test_operator_falls_back_to_the_host(fake, transpose):
    _run(fake, f"""
fake.fake_hip_refuse(n * 4, n * 4 + 4096)
a, b = binding.pcsr_operator_build(n, n, rowptr, colidx, vals, pc.make_params(**kw), 64, {transpose})
assert same(a, host) and (same(b, host_t) if {transpose} else b is None)
""")


def test_operator_picks_the_same_parameters_there(fake):
    _run(fake, """
p = pc.pcsr_select(pc.pcsr_features(n, n, rowptr, colidx), 64)
p.flags |= pc.PCSR_FLAG_HOST_ONLY
ref = pc.pcsr_build(n, n, rowptr, colidx, vals, p)
fake.fake_hip_refuse(n * 4, n * 4 + 4096)
picked, _ = binding.pcsr_operator_build(n, n, rowptr, colidx, vals, None, 64, False)
assert same(picked, ref)
""")


def test_kept_memory_goes_back_when_asked_for_and_when_the_device_is_low(fake):
    _run(fake, """
lib = binding._lib()
small = slice(0, 1000 * deg)


def build_and_close():
    pc.pcsr_build(1000, n, rowptr[:1001], colidx[small], vals[small]).close()
    assert fake.fake_hip_live() > 0


build_and_close()
assert pc.pcsr_release_cached() >= 1000 * deg * 8 and fake.fake_hip_live() == 0
assert pc.pcsr_release_cached() == 0
build_and_close()
fake.fake_hip_memory(13, 100)
assert lib.pcsr_release_cached_if_low(None) == 0 and fake.fake_hip_live() > 0      # more than an eighth is free
fake.fake_hip_memory(11, 100)
fake.fake_hip_capture(1)
assert lib.pcsr_release_cached_if_low(None) == 0 and fake.fake_hip_live() > 0
fake.fake_hip_capture(0)
assert lib.pcsr_release_cached_if_low(None) > 0 and fake.fake_hip_live() == 0
""")


def test_no_exception_leaves_the_library(fake):
    """Each of the library's own allocations on the host fails once: a call returns a code, and nothing leaks."""
    _run(fake, """
lib = binding._lib()
small = slice(0, 1000 * deg)
arrays = rowptr[:1001], colidx[small], vals[small]
ptrs = [a.ctypes.data for a in arrays]


def call(params):                                          # without Python's own allocations in between
    p, h = pc.make_params(**params), ctypes.c_void_p()
    def run(bad):
        fake.fake_new_fail(bad)
        rc = lib.pcsr_build(1000, n, 1000 * deg, *ptrs, ctypes.byref(p), ctypes.byref(h))
        if rc == 0:
            rc = lib.pcsr_reserve_workspace(h, 64)
            free = lib.pcsr_free(h)
            assert free == 0
        lib.pcsr_release_cached(None)
        used = fake.fake_new_calls()
        fake.fake_new_fail(0)
        return rc, used
    return run


for params in (dict(V=1), dict(V=2, S=1, SG=4), dict(V=1, S=1, SG=4, flags=pc.PCSR_FLAG_COLUMN_ORDER)):
    run = call(params)
    assert run(0)[0] == 0
    rc, used = run(1 << 30)
    assert rc == 0 and used >= 8 and fake.fake_hip_live() == 0
    for bad in range(1, used + 1):
        rc, _ = run(bad)
        assert rc in (0, binding.PCSR_E_OOM), (params, bad, rc)
        assert fake.fake_hip_live() == 0, (params, bad)
""")


# large enough for the values to follow on threads of their own: the build gives up, or ends, while they do
@pytest.mark.parametrize("k", [0, 2, 3, 4, 5])
def test_values_still_under_way_when_the_build_ends(fake, k):
    _run(fake, f"""
n = 150_000
colidx = np.tile(colidx, n // 30000)
rowptr = np.arange(0, n * deg + 1, deg, dtype=np.int32)
vals = rng.random(n * deg).astype(np.float32)              # 4.8 MB
assert vals.nbytes >= 4 << 20
host = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(flags=pc.PCSR_FLAG_HOST_ONLY, **kw))
if {k}:
    fake.fake_hip_fail({k}, {k})
    h = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(**kw))
    assert same(h, host)
    h.close()
else:
    bad = rowptr.copy()
    bad[7] = bad[8] + 1
    try:
        pc.pcsr_build(n, n, bad, colidx, vals, pc.make_params(**kw))
        assert False
    except pc.PcsrError as e:
        assert e.code == binding.PCSR_E_BAD_CSR
""")


# the upload's three arrays, the columns and values, the check's two; then what the search for communities asks for
@pytest.mark.parametrize("k", range(8, 13))
@pytest.mark.parametrize("S", [0, 1])
def test_without_scratch_for_communities_the_build_goes_on(fake, k, S):
    """Rows that look like communities, by what the library is told that the probe and the rounds found: out of memory in the
    search leaves the format asked for, out of memory for the windows the order without them."""
    _run(fake, f"""
checked = np.zeros(10, np.int32)                           # bad, first, last, longest, nonempty, -, two sums of 64 bits
checked[[2, 3, 4, 6]] = n * deg, deg, n, 1 << 20
found = np.array([n * 16, n * 16, (1 << 17) // 100], np.uint64)  # same, sampled, pairs with one label
for slot, a in enumerate((checked, found)):
    fake.fake_hip_answer(slot, ctypes.c_size_t(a.nbytes), a.ctypes.data_as(ctypes.c_void_p))
flags = pc.PCSR_FLAG_CLUSTER_IF_USEFUL | pc.PCSR_FLAG_CLUSTER_WINDOWS | pc.PCSR_FLAG_GPU_BUILD | ({S} and pc.PCSR_FLAG_COLUMN_ORDER)
fake.fake_hip_fail({k}, {k} + ({k} == 12))                 # (there once more after the blocks kept for reuse have gone back)
h = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(V=1, S={S}, SG=32 * {S}, flags=flags, vec=2, lanes_per_row=16))
assert fake.fake_hip_allocations() >= {k}
f, launch = pc.pcsr_format(h), pc.pcsr_query_launch(h, 64)
assert launch["lds_bytes"] == 0                            # no windows
if {k} < 12:
    assert f["S"] == {S} and (not {S} or f["SG"] == 32) and (launch["lanes_per_row"], launch["vec"]) == (16, 2)
else:
    assert f["S"] == 1 and f["SG"] == 1024 and (launch["lanes_per_row"], launch["vec"]) == (16, 4)
h.close()
pc.pcsr_release_cached()
assert fake.fake_hip_live() == 0
""")


def test_without_memory_for_the_bands_products_go_without(fake):
    _run(fake, """
checked = np.zeros(10, np.int32)                           # bad, first, last, longest, nonempty
checked[[2, 3, 4]] = n * deg, deg, n
flags = pc.PCSR_FLAG_GPU_BUILD | pc.PCSR_FLAG_COLUMN_BANDS


def built():
    fake.fake_hip_fail(0, 0)
    fake.fake_hip_answer(0, ctypes.c_size_t(checked.nbytes), checked.ctypes.data_as(ctypes.c_void_p))
    h = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(V=1, flags=flags))
    left = fake.fake_hip_live()
    h.close()
    pc.pcsr_release_cached()
    assert fake.fake_hip_live() == 0
    return left, fake.fake_hip_allocations()


whole = built()
fake.fake_hip_refuse(2 << 20, 2 << 20)                     # the table of the bands, in whole MiB
less = built()
assert less[0] < whole[0] and less[1] >= whole[1]
""")


# how often the bands of a direction do not fit: beside the other direction's scratch, or whenever they are asked for
@pytest.mark.parametrize("times", [0, 1, 2, 1 << 30])
def test_operators_are_built_again_where_the_other_direction_took_the_room(fake, times):
    """What a handle goes without does not depend on what the other direction, built at the same time, had allocated just then."""
    _run(fake, f"""
rowptr, colidx = np.arange(0, n * 100 + 1, 100, dtype=np.int32), np.tile(np.arange(100, dtype=np.int32) * 300, n)
checked, xcds = np.zeros(10, np.int32), np.arange(9, dtype=np.int32) * (n // 8)
checked[[2, 3, 4]] = n * 100, 100, n                       # bad, first, last, longest, nonempty
for slot, a in enumerate((checked, xcds)):
    fake.fake_hip_answer(slot, ctypes.c_size_t(a.nbytes), a.ctypes.data_as(ctypes.c_void_p))
fake.fake_hip_streams(1)
vals = np.ones(n * 100, np.float32)
args = n, n, rowptr, colidx, vals, pc.make_params(V=1, flags=pc.PCSR_FLAG_COLUMN_BANDS), 256, True


def bands(h):                                              # several launches, if the handle has them
    before = fake.fake_hip_launches()
    assert binding._lib().pcsr_spmm(h.raw, ctypes.c_void_p(1 << 33), ctypes.c_void_p(1 << 40), 256, None) == 0
    return fake.fake_hip_launches() - before > 1


fake.fake_hip_refuse(2 << 20, 2 << 20)                     # the table of the bands, in whole MiB
fake.fake_hip_refuse_times({times})
a, b = binding.pcsr_operator_build(*args)
assert fake.fake_hip_streams_made() > 0                    # both directions at once, the first time
assert bands(a) == bands(b) == ({times} < 1 << 30), (bands(a), bands(b))
a.close()
b.close()
pc.pcsr_release_cached()
assert fake.fake_hip_live() == 0
""")
