"""CPU-only: how slice_kernel cuts a product, and where it reads its words, walked lane by lane over whole matrices."""
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


@pytest.fixture(scope="module")
def plan(emul):  # noqa: F811
    def f(M, KB, *Ns, num_cu=256, bf16=False):
        out = (ctypes.c_int * 6)()
        emul.lib.emul_slice_plan(num_cu, M, KB, int(bf16), (ctypes.c_int * len(Ns))(*Ns), len(Ns), out)
        return tuple(out)
    return f


def test_plan_covers_the_tokens(plan):
    for M in range(33, 1025):
        tiles, passes, strip_rows, ksplit = plan(M, 171, 4096)[:4]
        assert tiles in (2, 3, 4) and strip_rows == (64 if tiles == 2 else 128)
        assert 32 * tiles * (passes - 1) < M <= 32 * tiles * passes and ksplit >= 1


def _promised(M, N, num_cu=256):
    """llvq.h: more strips of 256 rows x 256 tokens (128 x 512 from M = 384 on) than half the compute units"""
    rows, tokens = (256, 256) if M < 384 else (128, 512)
    return M > 64 and -(-N // rows) * -(-M // tokens) * 2 > num_cu


def test_k_is_not_split_where_reproducible_sums_are_promised(plan):
    Ns = (8192, 8193, 16129, 16384, 16385, 32513, 32768, 32769, 33024, 40000, 65536, 65537, 128256)
    seen = 0
    for N in Ns:
        for M in (65, 96, 97, 128, 129, 160, 250, 256, 257, 320, 383, 384, 513, 1024):
            for KB in (1, 2, 16, 42, 171, 342, 598, 1195):
                if _promised(M, N):
                    for bf16 in (False, True):
                        seen += 1
                        p = plan(M, KB, N, bf16=bf16)
                        assert p[3] == 1 and (p[4] == 1 or not p[5]), (N, M, KB)
                        assert plan(M, KB, 1024, N, bf16=bf16)[3] == 1, (N, M, KB)        # beside a small matrix as well
    assert seen > 800
    assert plan(64, 171, 40000)[0] == 2 and plan(128, 171, 1024)[3] > 1      # small products still share their rows


def test_products_that_take_the_strip_kernel(plan):
    """65 <= M < 384 on large products, measured on either side (see strip_faster); never elsewhere"""
    def strip(N, KB, M, bf16):
        return bool(plan(M, KB, N, bf16=bf16)[5])

    from test_gpu_slice_kernel import STRIP_SIZES
    for N, KB, M, xd in STRIP_SIZES:
        assert strip(N, KB, M, xd == "bf16"), (N, KB, M)
    for N, KB, M, bf16 in ((14336, 598, 250, False), (14336, 598, 256, True), (11008, 342, 129, False), (65536, 171, 256, True), (65536, 20, 300, True)):
        assert strip(N, KB, M, bf16), (N, KB, M)
        assert not strip(N, KB, 64, bf16) and not strip(N, KB, 384, bf16)
    for N, KB, M, bf16 in ((14336, 171, 250, False), (4096, 171, 256, True), (1024, 598, 200, False), (65536, 171, 128, True), (64, 1, 129, True)):
        assert not strip(N, KB, M, bf16), (N, KB, M)
