"""llvq_matmul and llvq_matmul_multi at M >= 33, kernel by kernel.  Slices of K that share activation tiles and are added in LDS, at
the edges of token tiles (32 per tile, up to four per pass), row tiles (64 and 128 rows per workgroup) and slices (block pairs
dealt to four or eight slices of one or more workgroups: fewer pairs than slices, an odd block count, a row of one block); strips
of 256 rows x 256 tokens; panels of 128 rows x 512 tokens."""
import numpy as np
import pytest

from paper_2603_11021_amd import LLVQ_IDX_U24, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_11021_amd import LLVQ
    return LLVQ(13, 0)


# sizes that the choice of kernels gives to slice_kernel, panel_kernel, panel_kernel with several matrices in one launch, and
# strip_kernel (checked in tests/test_host_slices.py)
SLICE_SIZES = [(1, 2, 33), (31, 1, 64), (33, 3, 64), (64, 2, 65), (65, 7, 96), (127, 8, 97), (129, 16, 128), (128, 17, 129), (63, 33, 192), (130, 5, 193),
               (97, 9, 256), (96, 10, 383), (40, 171, 160), (257, 40, 34), (300, 40, 1024), (1100, 33, 1000), (2051, 21, 513), (65, 1, 385)]
PANEL_SIZES = [(14000, 171, 513, "f16"), (28600, 60, 257, "bf16"), (8200, 33, 385, "bf16")]
MULTI_PANEL_SIZES = [((4100, 1000, 130, 3000), 81, 400, "bf16"), ((5000, 7000), 9, 513, "f16"), ((2050, 1), 342, 1024, "f16")]
STRIP_SIZES = [(65601, 3, 129, "bf16"), (65537, 1, 255, "f16"), (40001, 5, 161, "f16"), (65300, 9, 256, "bf16"), (8003, 598, 129, "f16"), (11001, 301, 250, "bf16")]


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _bound(xd):
    # fp16 weights carry 2^-11 per weight (a single block, M * N draws: below 2^-11 * 4); bf16 weights enter as two terms (2^-16)
    return 2e-3 if xd == "f16" else 1e-4


def _activations(x, xd):
    import torch
    return _dev(x).to(torch.float16 if xd == "f16" else torch.bfloat16)


@pytest.mark.parametrize("xd", ["f16", "bf16"])
@pytest.mark.parametrize("N,KB,M", SLICE_SIZES)
def test_slices_match_the_oracle(gpu, oracle13, N, KB, M, xd):
    idx, gain, x = synth.layer(8, 5000 + N + 7 * KB + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16")
    import torch
    y = torch.full((M, N), float("nan"), device="cuda:0")                 # every element has to be written
    gpu.llvq_matmul(_activations(x, xd), _dev(synth.pack_u48(idx).reshape(-1)), _dev(gain.reshape(-1)), N, KB, out=y)
    ref = oracle13.matmul(x, idx, gain)
    err = np.abs(y.cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max()
    assert err <= _bound(xd), err


@pytest.mark.parametrize("N,KB,M,xd", [(12801, 164, 257, "bf16"), (12801, 164, 320, "f16"), (4000, 512, 383, "bf16"), (12801, 164, 256, "f16")])
def test_long_layers_on_either_side_of_a_third_pass(gpu, oracle13, N, KB, M, xd):
    """257 <= M < 384 on layers with many steps: the panel kernel with up to half of its waves' tokens past M"""
    import torch
    idx, gain, x = synth.layer(8, 7000 + N + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16")
    y = torch.full((M, N), float("nan"), device="cuda:0")
    gpu.llvq_matmul(_activations(x, xd), _dev(synth.pack_u48(idx).reshape(-1)), _dev(gain.reshape(-1)), N, KB, out=y)
    assert not torch.isnan(y).any()
    rows = np.concatenate([np.arange(8), np.arange(N - 8, N), np.random.default_rng(N + M).choice(N, 24, replace=False)])
    ref = oracle13.matmul(x, idx[rows], gain[rows])
    err = np.abs(y.cpu().numpy().astype(np.float64)[:, rows] - ref).max() / np.abs(ref).max()
    assert err <= _bound(xd), err


@pytest.mark.parametrize("Ns,KB,M,xd", [((64, 1, 130, 65), 6, 33, "f16"), ((129, 128), 11, 100, "bf16"), ((5, 300, 33), 2, 383, "bf16")])
def test_slices_of_several_matrices(gpu, oracle13, Ns, KB, M, xd):
    import torch
    parts = [synth.layer(8, 6000 + i + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16") for i, N in enumerate(Ns)]
    x = parts[0][2]
    outs = [torch.full((M, N), float("nan"), device="cuda:0") for N in Ns]
    gpu.llvq_matmul_multi(_activations(x, xd), [_dev(synth.pack_u48(p[0]).reshape(-1)) for p in parts], [_dev(p[1].reshape(-1)) for p in parts], list(Ns), KB,
                          outs=outs)
    for p, y in zip(parts, outs):
        ref = oracle13.matmul(x, p[0], p[1])
        err = np.abs(y.cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max()
        assert err <= _bound(xd), err


@pytest.mark.parametrize("M,xd", [(33, "f16"), (100, "bf16")])
@pytest.mark.parametrize("N", [65, 129, 193])
def test_last_strip_of_a_single_block(gpu, oracle13, N, M, xd):
    """One block per row and one row in the last strip: its word is read as the second of a pair, in every word format"""
    import torch
    idx, gain, x = synth.layer(8, 8000 + N + M, N, 24, M, x_dtype=np.float16 if xd == "f16" else "bf16")
    d_x, d_gain = _activations(x, xd), _dev(gain.reshape(-1))
    ref = oracle13.matmul(x, idx, gain)
    base = gpu.llvq_shell_offset(3)
    words3 = idx % np.uint64(gpu.llvq_shell_offset(4) - base)                 # 24-bit words address shell 3
    ref3 = oracle13.matmul(x, words3 + np.uint64(base), gain)

    def out():
        return torch.full((M, N), float("nan"), device="cuda:0")

    d48, d64, d24 = _dev(synth.pack_u48(idx).reshape(-1)), _dev(idx.view(np.int64).reshape(-1)), _dev(synth.pack_u24(words3).reshape(-1))
    for y, want in ((gpu.llvq_matmul(d_x, d48, d_gain, N, 1, out=out()), ref), (gpu.llvq_matmul(d_x, d64, d_gain, N, 1, out=out()), ref),
                    (gpu.llvq_matmul_coded(d_x, d24, N, 1, 24, base, gain=d_gain, fmt=LLVQ_IDX_U24, out=out()), ref3),
                    (gpu.llvq_matmul_multi(d_x, [d48, d48], [d_gain, d_gain], [N, N], 1, outs=[out(), out()])[1], ref)):
        err = np.abs(y.cpu().numpy().astype(np.float64) - want).max() / np.abs(want).max()
        assert err <= _bound(xd), err


@pytest.mark.parametrize("M,xd", [(65, "bf16"), (256, "f16")])
def test_many_rows_give_the_same_bits(gpu, oracle13, M, xd):
    """More strips of 256 rows x 256 tokens than half the compute units: K is not split, also beside a small matrix"""
    import torch
    N, KB = 33024, 40
    idx, gain, x = synth.layer(8, 9000 + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16")
    d_x, d_idx, d_gain = _activations(x, xd), _dev(synth.pack_u48(idx).reshape(-1)), _dev(gain.reshape(-1))
    n = 100                                                                   # the first rows as a matrix of their own

    def single():
        return gpu.llvq_matmul(d_x, d_idx, d_gain, N, KB)

    def multi():
        return gpu.llvq_matmul_multi(d_x, [d_idx[:6 * KB * n], d_idx], [d_gain[:KB * n], d_gain], [n, N], KB)[1]

    rows = np.concatenate([np.arange(4), np.arange(N - 4, N), np.random.default_rng(M).choice(N, 24, replace=False)])
    ref = oracle13.matmul(x, idx[rows], gain[rows])
    for product in (single, multi):
        y = product()
        for _ in range(3):
            assert torch.equal(product(), y)
        err = np.abs(y.cpu().numpy().astype(np.float64)[:, rows] - ref).max() / np.abs(ref).max()
        assert err <= _bound(xd), err


@pytest.mark.parametrize("N,KB,M,xd", STRIP_SIZES)
def test_strips_match_the_oracle(gpu, oracle13, N, KB, M, xd):
    """256 rows x up to 256 tokens: partial strips, partial and whole token tiles, odd block counts, single blocks, K split and whole"""
    import torch
    idx, gain, x = synth.layer(8, 9500 + N + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16")
    d_x, d_gain = _activations(x, xd), _dev(gain.reshape(-1))
    rows = np.unique(np.concatenate([np.arange(8), np.arange(N - 8, N), np.random.default_rng(N + M).choice(N, 40, replace=False)]))
    d_rows = _dev(rows)
    base = gpu.llvq_shell_offset(3)
    words3 = idx % np.uint64(gpu.llvq_shell_offset(4) - base)                 # 24-bit words address shell 3
    refs = [oracle13.matmul(x, idx[rows], gain[rows]), oracle13.matmul(x, words3[rows] + np.uint64(base), gain[rows])]

    def out():
        return torch.full((M, N), float("nan"), device="cuda:0")              # every element has to be written

    for y, ref in ((gpu.llvq_matmul(d_x, _dev(synth.pack_u48(idx).reshape(-1)), d_gain, N, KB, out=out()), refs[0]),
                   (gpu.llvq_matmul(d_x, _dev(idx.view(np.int64).reshape(-1)), d_gain, N, KB, out=out()), refs[0]),
                   (gpu.llvq_matmul_coded(d_x, _dev(synth.pack_u24(words3).reshape(-1)), N, KB, 24, base, gain=d_gain, fmt=LLVQ_IDX_U24, out=out()), refs[1])):
        assert not torch.isnan(y).any()
        err = np.abs(y[:, d_rows].cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max()
        assert err <= _bound(xd), err


def test_strips_of_several_matrices_one_after_the_other(gpu, oracle13):
    import torch
    Ns, KB, M = (65001, 700, 65001), 21, 250
    parts = [synth.layer(8, 9700 + i, N, 24 * KB, M) for i, N in enumerate(Ns)]
    x = parts[0][2]
    d_x, d_idx, d_gain = _activations(x, "f16"), [_dev(synth.pack_u48(p[0]).reshape(-1)) for p in parts], [_dev(p[1].reshape(-1)) for p in parts]
    outs = [torch.full((M, N), float("nan"), device="cuda:0") for N in Ns]
    gpu.llvq_matmul_multi(d_x, d_idx, d_gain, list(Ns), KB, outs=outs)
    for (idx, gain, _), y, N in zip(parts, outs, Ns):
        rows = np.unique(np.concatenate([np.arange(4), np.arange(N - 4, N), np.random.default_rng(N).choice(N, 24, replace=False)]))
        ref = oracle13.matmul(x, idx[rows], gain[rows])
        assert not torch.isnan(y).any()
        err = np.abs(y.cpu().numpy().astype(np.float64)[:, rows] - ref).max() / np.abs(ref).max()
        assert err <= _bound("f16"), err


@pytest.mark.parametrize("N,KB,M,xd", PANEL_SIZES)
def test_panels_match_the_oracle(gpu, oracle13, N, KB, M, xd):
    """one token in the last pass or in the last wave's share, partial panels, K split and whole"""
    import torch
    idx, gain, x = synth.layer(8, 9900 + N + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16")
    y = torch.full((M, N), float("nan"), device="cuda:0")
    gpu.llvq_matmul(_activations(x, xd), _dev(synth.pack_u48(idx).reshape(-1)), _dev(gain.reshape(-1)), N, KB, out=y)
    assert not torch.isnan(y).any()
    rows = np.unique(np.concatenate([np.arange(4), np.arange(N - 4, N), np.random.default_rng(N + M).choice(N, 32, replace=False)]))
    ref = oracle13.matmul(x, idx[rows], gain[rows])
    err = np.abs(y.cpu().numpy().astype(np.float64)[:, rows] - ref).max() / np.abs(ref).max()
    assert err <= _bound(xd), err


@pytest.mark.parametrize("Ns,KB,M,xd", MULTI_PANEL_SIZES)
def test_panels_of_several_matrices(gpu, oracle13, Ns, KB, M, xd):
    """ragged row counts, so that every matrix ends in a partial panel; K split and whole"""
    import torch
    parts = [synth.layer(8, 9800 + i + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16") for i, N in enumerate(Ns)]
    x = parts[0][2]
    outs = [torch.full((M, N), float("nan"), device="cuda:0") for N in Ns]
    gpu.llvq_matmul_multi(_activations(x, xd), [_dev(synth.pack_u48(p[0]).reshape(-1)) for p in parts], [_dev(p[1].reshape(-1)) for p in parts], list(Ns), KB,
                          outs=outs)
    for (idx, gain, _), y, N in zip(parts, outs, Ns):
        rows = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(N).choice(N, min(N, 40), replace=False)]))
        ref = oracle13.matmul(x, idx[rows], gain[rows])
        assert not torch.isnan(y).any()
        err = np.abs(y.cpu().numpy().astype(np.float64)[:, rows] - ref).max() / np.abs(ref).max()
        assert err <= _bound(xd), err


def test_products_that_clear_y_can_be_captured_in_a_graph(gpu, oracle13):
    """K split in each of the three kernels (y is cleared, then added to) and several matrices in one launch: every replay, with eager
    work and synchronisations in between, reproduces the eager result up to the order of the fp32 atomic adds"""
    import torch
    cases = []
    for N, KB, M, xd in ((40, 171, 160, "f16"), (11001, 301, 250, "bf16"), (4100, 131, 1000, "bf16")):
        idx, gain, x = synth.layer(8, 9950 + M, N, 24 * KB, M, x_dtype=np.float16 if xd == "f16" else "bf16")
        rows = np.unique(np.concatenate([[0, N - 1], np.random.default_rng(M).choice(N, min(N, 24), replace=False)]))
        cases.append((_activations(x, xd), _dev(synth.pack_u48(idx).reshape(-1)), _dev(gain.reshape(-1)), N, KB,
                      torch.empty((M, N), dtype=torch.float32, device="cuda:0"), rows, oracle13.matmul(x, idx[rows], gain[rows])))
    x, idx, gain, N, KB = cases[0][:5]
    several = [torch.empty((x.shape[0], n), dtype=torch.float32, device="cuda:0") for n in (N, 17)]

    def run():
        for x_, idx_, gain_, N_, KB_, y, _, _ in cases:
            gpu.llvq_matmul(x_, idx_, gain_, N_, KB_, out=y)
        gpu.llvq_matmul_multi(x, [idx, idx[:6 * KB * 17]], [gain, gain[:KB * 17]], [N, 17], KB, outs=several)

    run()
    torch.cuda.synchronize()
    ys = [c[5] for c in cases] + several
    eager = [y.clone() for y in ys]
    for (_, _, _, _, _, y, rows, ref) in cases:
        assert np.abs(y.cpu().numpy().astype(np.float64)[:, rows] - ref).max() / np.abs(ref).max() <= 2e-3
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for rep in range(4):
        for y in ys:
            y.fill_(float(rep))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for y, want in zip(ys, eager):
            # up to 16 partial sums of fp32 in another order
            assert float((y - want).abs().max()) <= 16 * 2.0 ** -23 * float(want.abs().max())
