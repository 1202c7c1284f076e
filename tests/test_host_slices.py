"""CPU-only: which kernel a product of 33 or more activation rows takes, how it is cut, and where slice_kernel reads its words, walked
lane by lane over whole matrices."""
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


class Plan:
    def __init__(self, lib, M, KB, Ns, bf16, num_cu):
        out = (ctypes.c_int * 8)()
        lib.emul_plan(num_cu, M, KB, int(bf16), (ctypes.c_int * len(Ns))(*Ns), len(Ns), out)
        self.token_tiles, self.passes, self.strip_rows, self.slice_split, self.strip_split, self.panel_split = out[:6]
        self.route = ("slice", "strip", "panel")[out[6]]
        self.multi = ("slice", "panel", "apart")[out[7]]


@pytest.fixture(scope="module")
def plan(emul):  # noqa: F811
    return lambda M, KB, *Ns, bf16=False, num_cu=256: Plan(emul.lib, M, KB, Ns, bf16, num_cu)


def test_plan_covers_the_tokens(plan):
    for M in range(33, 1025):
        p = plan(M, 171, 4096)
        assert p.token_tiles in (2, 3, 4) and p.strip_rows == (64 if p.token_tiles == 2 else 128)
        assert 32 * p.token_tiles * (p.passes - 1) < M <= 32 * p.token_tiles * p.passes and p.slice_split >= 1


def _promised(M, N, num_cu):
    """llvq.h: more strips of 256 rows x 256 tokens (128 x 512 from M = 384 on) than half the compute units"""
    rows, tokens = (256, 256) if M < 384 else (128, 512)
    return M > 64 and -(-N // rows) * -(-M // tokens) * 2 > num_cu


@pytest.mark.parametrize("num_cu", [32, 64, 128, 256])
def test_k_is_not_split_where_reproducible_sums_are_promised(plan, num_cu):
    Ns = (1025, 2048, 4097, 8192, 8193, 16129, 16384, 16385, 32513, 32768, 32769, 33024, 40000, 65536, 65537, 128256)
    seen = 0
    for N in Ns:
        for M in (65, 96, 97, 128, 129, 160, 250, 256, 257, 320, 383, 384, 513, 1024):
            for KB in (1, 2, 16, 42, 171, 342, 598, 1195):
                if not _promised(M, N, num_cu):
                    continue
                for bf16 in (False, True):
                    seen += 1
                    p = plan(M, KB, N, bf16=bf16, num_cu=num_cu)
                    assert {"slice": p.slice_split, "strip": p.strip_split, "panel": p.panel_split}[p.route] == 1, (N, M, KB)
                    p = plan(M, KB, 1024, N, bf16=bf16, num_cu=num_cu)                     # beside a small matrix as well
                    assert {"slice": p.slice_split, "panel": p.panel_split, "apart": 1}[p.multi] == 1, (N, M, KB)
    assert seen > 1000
    assert plan(128, 171, 1024).slice_split > 1                                          # small products still share their rows


def test_routes(plan):
    """The kernel that measured faster, on either side of the lines (see best_route and multi_route)"""
    for N, KB, M, bf16, route in ((4096, 171, 256, True, "slice"), (14336, 171, 250, False, "slice"), (65536, 171, 128, True, "slice"),
                                  (14336, 598, 250, False, "strip"), (14336, 598, 256, True, "strip"), (65536, 171, 256, True, "strip"),
                                  (65536, 20, 256, True, "strip"), (65536, 20, 257, True, "panel"),
                                  (11008, 342, 129, False, "strip"), (64, 1, 129, True, "slice"),
                                  (4096, 171, 320, False, "slice"), (4096, 171, 512, False, "slice"), (1024, 171, 1024, True, "slice"),
                                  (4096, 60, 1024, True, "slice"), (8192, 60, 512, True, "slice"), (4096, 598, 512, True, "panel"),
                                  (14336, 171, 320, True, "panel"), (14336, 171, 1024, False, "panel"), (28672, 60, 320, False, "panel"),
                                  (8192, 171, 513, False, "panel"), (2, 1, 33, False, "slice"), (14336, 598, 64, False, "slice")):
        assert plan(M, KB, N, bf16=bf16).route == route, (N, KB, M, bf16)
    for Ns, KB, M, bf16, route in (((4096, 1024, 1024), 171, 250, False, "slice"), ((14336, 14336), 171, 250, False, "slice"),
                                   ((28672, 28672), 171, 256, True, "apart"), ((65536, 1024), 171, 256, True, "apart"),
                                   ((14336, 14336), 171, 512, False, "panel"), ((14336, 14336), 171, 1024, True, "apart"),
                                   ((4096, 1024, 1024), 171, 1024, True, "panel")):
        assert plan(M, KB, *Ns, bf16=bf16).multi == route, (Ns, KB, M, bf16)


def test_sizes_of_the_device_tests_reach_their_kernels(plan):
    from test_gpu_slice_kernel import MULTI_PANEL_SIZES, PANEL_SIZES, SLICE_SIZES, STRIP_SIZES
    for sizes, route in ((SLICE_SIZES, "slice"), (STRIP_SIZES, "strip"), (PANEL_SIZES, "panel")):
        for N, KB, M, *xd in sizes:
            for bf16 in ((xd[0] == "bf16",) if xd else (False, True)):
                assert plan(M, KB, N, bf16=bf16).route == route, (N, KB, M)
    for Ns, KB, M, xd in MULTI_PANEL_SIZES:
        assert plan(M, KB, *Ns, bf16=xd == "bf16").multi == "panel", (Ns, KB, M)


def test_panel_reaches_as_far_as_its_offsets(plan):
    assert plan(1024, 87381, 1000, bf16=True).route == "panel"                          # 1024 x 87381 x 48 bytes just fit 32 bits
    assert plan(1024, 87382, 1000, bf16=True).route == "slice"
