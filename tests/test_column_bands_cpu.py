"""How many launches a product in bands of columns takes, on a device of host memory (fake_hip).  No GPU calls."""
import pytest

from tests.test_out_of_memory_cpu import _run, fake  # noqa: F401  (a fixture)

HANDLE = """
m, deg, n_cols = 20000, 134, 300_000                       # B of 20 MB and more from K = 16 on
f = np.array(pc.pcsr_features(n, n, rowptr, colidx), dtype=np.float64)
f[:2], f[2], f[4:7], f[7:9], f[15], f[16] = 300_000, 300_000 * deg, deg, 0.1, 0.5, 0.0
cols = np.tile(np.arange(deg, dtype=np.int32) * (n_cols // deg), m)
ptr = np.arange(0, m * deg + 1, deg, dtype=np.int32)
checked = np.zeros(10, np.int32)                           # bad, first, last, longest, nonempty
checked[[2, 3, 4]] = m * deg, deg, m
xcds = np.arange(9, dtype=np.int32) * (m // 8)             # the rows of each XCD
for slot, a in enumerate((checked, xcds)):
    fake.fake_hip_answer(slot, ctypes.c_size_t(a.nbytes), a.ctypes.data_as(ctypes.c_void_p))
B, C = 1 << 33, 1 << 40                                    # not looked at


def handle(**kw):
    return pc.pcsr_build(m, n_cols, ptr, cols, np.ones(m * deg, np.float32), pc.make_params(**kw))


def launches(h, K):
    before = fake.fake_hip_launches()
    assert binding._lib().pcsr_spmm(h.raw, ctypes.c_void_p(B), ctypes.c_void_p(C), K, None) == 0
    return fake.fake_hip_launches() - before
"""


SELECTED = """
p = pc.pcsr_select(f, {hint})
assert p.S == 0 and p.V == 1 and p.flags & pc.PCSR_FLAG_COLUMN_BANDS
p.flags = (p.flags & ~(pc.PCSR_FLAG_CLUSTER_IF_USEFUL | pc.PCSR_FLAG_CLUSTER_WINDOWS)) | pc.PCSR_FLAG_GPU_BUILD
h = handle(**{{k: getattr(p, k) for k, _ in p._fields_ if k != "reserved"}})
q = pc.pcsr_query_kernel(h, {K})
"""


# selected for one width and used at another, which the shape that stands in covers in slices: the last lane of a row computes
# columns of the slice before, so that a band added to C would be added twice
@pytest.mark.parametrize("hint,K", [(33, 65), (33, 67), (42, 70), (49, 66), (50, 66), (50, 74), (62, 126), (66, 130), (75, 131), (126, 134),
                                    (33, 257), (66, 302)])
def test_bands_only_where_no_two_slices_share_columns(fake, hint, K):  # noqa: F811
    _run(fake, HANDLE + SELECTED.format(hint=hint, K=K) + f"""
assert q["grid_y"] == 1 and q["lanes_per_row"] * q["vec"] * q["rep"] >= {K}
assert launches(h, {hint}) > 1 and launches(h, 128) > 1
assert {K} > 256 or launches(h, {K}) > 1
h.close()
""")


@pytest.mark.parametrize("hint,K", [(50, 514), (75, 519), (75, 1030)])
def test_one_band_where_slices_share_columns(fake, hint, K):  # noqa: F811
    _run(fake, HANDLE + SELECTED.format(hint=hint, K=K) + f"""
assert {K} % q["vec"] and q["grid_y"] > 1
assert launches(h, {K}) == 1
h.close()
""")


def test_auto_shapes_are_those_of_the_band_kernel(fake):  # noqa: F811
    """Wide rows left to the library, as an operator's are: slices of 64 columns, or a tile of up to 512."""
    _run(fake, HANDLE + """
h = handle(flags=pc.PCSR_FLAG_GPU_BUILD | pc.PCSR_FLAG_COLUMN_BANDS)
shape = lambda K: (lambda q: (q["lanes_per_row"], q["vec"], q["rep"], q["grid_y"]))(pc.pcsr_query_kernel(h, K))  # noqa: E731
for K in (64, 96, 128, 256, 512, 1024):
    assert shape(K) == (16, 4, 1, (K + 63) // 64) and launches(h, K) > 1, K
    assert pc.pcsr_query_launch(h, K) == pc.pcsr_query_kernel(h, K)
for K, s in ((72, (32, 4, 1, 1)), (200, (64, 4, 1, 1)), (260, (64, 4, 2, 1)), (515, (64, 4, 2, 2)), (1000, (64, 4, 2, 2))):
    assert shape(K) == s, K
assert shape(1 << 20)[2:] == (1, 1 << 14) and shape(8_000_000) == (64, 4, 2, 15625)  # as wide as a grid takes
h.close()
""")


def test_wide_tiles_keep_parts_of_20_at_every_width(fake):  # noqa: F811
    """A handle whose tile is a whole row of 75 to 256 columns, at other widths: its sums were of 8, and shorter parts are less exact."""
    _run(fake, HANDLE.replace("m, deg, n_cols = 20000, 134, 300_000", "m, deg, n_cols = 100_000, 90, 100_000") + """
parts = {}
for lanes in (16, 32, 64):
    h = handle(flags=pc.PCSR_FLAG_GPU_BUILD | pc.PCSR_FLAG_COLUMN_BANDS, lanes_per_row=lanes, vec=4, rep=1)
    parts[lanes] = [launches(h, K) for K in (48, 64, 96, 128)]
    h.close()
assert max(parts[16]) == 6 and max(parts[32] + parts[64]) == 90 // 20, parts
""")


def test_tiles_of_512_columns_are_walked_in_bands_where_much_is_saved(fake):  # noqa: F811
    _run(fake, HANDLE.replace("m, deg, n_cols = 20000, 134, 300_000", "m, deg, n_cols = 100_000, 90, 200_000") + """
h = handle(flags=pc.PCSR_FLAG_GPU_BUILD | pc.PCSR_FLAG_COLUMN_BANDS)
for K, several in ((130, True), (256, True), (260, False), (300, False), (340, False)):
    assert (launches(h, K) > 1) == several, K
h.close()
""")
    _run(fake, HANDLE.replace("n_cols = 20000, 134, 300_000", "n_cols = 20000, 134, 100_000") + """
h = handle(flags=pc.PCSR_FLAG_GPU_BUILD | pc.PCSR_FLAG_COLUMN_BANDS)
assert launches(h, 260) > 1 and launches(h, 300) > 1
h.close()
""")
