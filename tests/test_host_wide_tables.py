"""CPU-only: the tables that the kernels of contexts with m_max > 13 decode with, run on the host against the oracle."""
import ctypes

import numpy as np
import pytest

from test_host_logic import emul, oracle19, wide19  # noqa: F401


@pytest.fixture(scope="module")
def tables19(wide19):  # noqa: F811
    lib = wide19.lib
    lib.emul_wide_tab_decode_i8.restype = ctypes.c_uint64
    lib.emul_wide_tab_decode_i8.argtypes = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_void_p]

    def decode(idx):
        idx = np.ascontiguousarray(idx, dtype=np.uint64)
        out = np.empty((idx.size, 24), dtype=np.int8)
        return out, int(lib.emul_wide_tab_decode_i8(idx.ctypes.data, idx.size, out.ctypes.data))

    return decode


def test_wide_tables_decode_every_class(tables19, oracle19):  # noqa: F811
    rng = np.random.default_rng(193)
    idx = [rng.integers(0, oracle19.num_points, size=100000, dtype=np.uint64)]
    for c in oracle19.classes():
        off, size = int(c["offset"]), int(c["size"])
        idx.append(np.array([off, off + size - 1] + [off + int(v) for v in rng.integers(0, size, size=40, dtype=np.uint64)], dtype=np.uint64))
    idx = np.concatenate(idx)
    got, bad = tables19(idx)
    assert bad == 0 and np.array_equal(got, oracle19.decode(idx)[0])


def test_wide_tables_out_of_range(tables19, oracle19):  # noqa: F811
    got, bad = tables19(np.array([oracle19.num_points, 2 ** 56 - 1], dtype=np.uint64))
    assert bad == 2 and not got.any()
