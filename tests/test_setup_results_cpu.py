"""How results of set-up kernels come to the host through pinned memory, on a device of host memory (fake_hip).  No GPU calls."""
from tests.test_out_of_memory_cpu import _run, fake  # noqa: F401  (a fixture)

FEATURES = """
lib = binding._lib()
fake.fake_hip_pinned(1)
dev = np.zeros(16, np.int32).ctypes.data                   # kernels do not run: not looked at


def features(n_hat):
    counted = np.zeros(11, np.int64)                       # the first of them: non-empty rows
    counted[0] = n_hat
    fake.fake_hip_answer(0, ctypes.c_size_t(counted.nbytes), counted.ctypes.data_as(ctypes.c_void_p))
    out = (ctypes.c_double * 17)()
    rc = lib.pcsr_features_device(1000, 1000, 5000, ctypes.c_void_p(dev), ctypes.c_void_p(dev), 0, out, 17)
    return rc, out[1]
"""


def test_results_come_through_coherent_memory(fake):  # noqa: F811
    """The host looks for them while the kernel is there: hipHostMallocCoherent, whatever the default is."""
    _run(fake, FEATURES + """
assert features(77) == (0, 77.0) and features(78) == (0, 78.0)
fake.fake_hip_pinned_flags.restype = ctypes.c_uint
assert fake.fake_hip_pinned_flags() & 0x40000000
""")


def test_results_that_arrive_late_are_not_taken_for_the_next_ones(fake):  # noqa: F811
    _run(fake, FEATURES + """
assert features(77) == (0, 77.0)
fake.fake_hip_keep_back()
assert features(111)[0] == binding.PCSR_E_HIP              # the wait for them fails
assert features(222) == (0, 222.0)                         # and they arrive while the next call waits for its own
assert features(333) == (0, 333.0)
""")


def test_refused_while_a_stream_is_captured(fake):  # noqa: F811
    """As a copy on the null stream is, however the results come: what the capture is yet to make would be counted."""
    _run(fake, FEATURES + """
assert features(77) == (0, 77.0)
fake.fake_hip_capture(1)
assert features(78)[0] == binding.PCSR_E_HIP
fake.fake_hip_capture(0)
assert features(79) == (0, 79.0)
""")
