"""The table-driven decoder of the contexts with m_max > 13: sizes at the edges of its kernels, and the two classes that are
placed step by step."""
import numpy as np
import pytest

from paper_2603_11021_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu19():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_11021_amd import LLVQ
    return LLVQ(19, 0)


@pytest.fixture(scope="module")
def oracle19():
    from oracle.llvq_oracle import Oracle
    return Oracle(19)


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _indices(oracle19, rng, n):
    """random indices, every seventh from one of the two classes that are placed step by step (4^18 0^6 and 1^19 3 5 7 9 11)"""
    idx = rng.integers(0, oracle19.num_points, size=n, dtype=np.uint64)
    classes = oracle19.classes()
    for k, cid in enumerate((972, 1438)):
        off, size = int(classes[cid]["offset"]), int(classes[cid]["size"])
        idx[3 + 7 * k::14] = off + rng.integers(0, size, size=idx[3 + 7 * k::14].shape, dtype=np.uint64)
    return idx


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1025, 70001])
def test_wide_decode_sizes(gpu19, oracle19, n):
    rng = synth.rng_for(19, 100 + n)
    idx = _indices(oracle19, rng, n)
    got = gpu19.llvq_decode_i8(_dev(idx.view(np.int64))).cpu().numpy()
    assert np.array_equal(got, oracle19.decode(idx)[0])


# rows and blocks around the tiles of 16 rows x 4 blocks and the batches of 64 blocks; the last two deal their batches as waves finish
@pytest.mark.parametrize("N,KB,M,xd", [(1, 1, 1, "f16"), (3, 1, 2, "bf16"), (17, 3, 3, "f16"), (15, 5, 15, "f16"), (33, 66, 16, "bf16"),
                                       (2048, 600, 1, "bf16"), (4096, 300, 2, "f16"), (4200, 25, 16, "f16")])
def test_wide_matmul_sizes(gpu19, oracle19, N, KB, M, xd):
    import torch
    rng = synth.rng_for(19, 200 + N + M)
    idx = _indices(oracle19, rng, N * KB).reshape(N, KB)
    gain = synth.gains(rng, (N, KB))
    x = synth.activations(rng, M, 24 * KB, "bf16" if xd == "bf16" else np.float16)
    d_x = _dev(x).to(torch.bfloat16 if xd == "bf16" else torch.float16)
    y = gpu19.llvq_matmul(d_x, _dev(idx.view(np.int64).reshape(-1)), _dev(gain.reshape(-1)), N, KB).cpu().numpy().astype(np.float64)
    rows = np.unique(np.concatenate([np.arange(min(N, 20)), np.arange(max(0, N - 20), N), rng.integers(0, N, size=30)]))
    ref = oracle19.matmul(x, idx[rows], gain[rows])
    assert np.abs(y[:, rows] - ref).max() <= 1e-5 * np.abs(ref).max()
