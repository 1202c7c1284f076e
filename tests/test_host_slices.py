"""CPU-only: where slice_kernel reads its words, walked lane by lane over whole matrices."""
import ctypes

import pytest

from test_host_logic import emul  # noqa: F401


@pytest.fixture(scope="module")
def pairs_wrong(emul):  # noqa: F811
    fn = emul.lib.emul_slice_pairs_wrong
    fn.restype = ctypes.c_uint64
    fn.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return fn


@pytest.mark.parametrize("strip_rows", [64, 128])
def test_word_pairs_lie_inside_the_matrix(pairs_wrong, strip_rows):
    """Every N up to three strips and every KB up to 9: strips that end in one row, rows of one block, odd block counts"""
    bad = [(N, KB) for KB in range(1, 10) for N in range(1, 3 * strip_rows + 3) if N * KB >= 2 and pairs_wrong(N, KB, strip_rows)]
    assert not bad, bad


@pytest.mark.parametrize("strip_rows", [64, 128])
@pytest.mark.parametrize("N,KB", [(129, (1 << 24) - 1), (255, (1 << 24) - 1), (256, (1 << 24) - 1), (1 << 16, 171), (65537, 1), (4097, 171)])
def test_word_pairs_of_large_matrices(pairs_wrong, N, KB, strip_rows):
    """Up to 2^32 blocks: offsets of a strip near 2^31, more blocks left than 32 bits hold"""
    assert pairs_wrong(N, KB, strip_rows) == 0
