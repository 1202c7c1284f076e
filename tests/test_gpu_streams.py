"""Tensors that the binding makes for a call on a stream other than the current one."""
import numpy as np
import pytest

from paper_2603_11021_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_11021_amd import LLVQ
    return LLVQ(13, 0)


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("M", [1, 7, 40])
def test_activations_that_are_not_contiguous(gpu, oracle13, M):
    """columns of a wider tensor, on the current stream and on another one: the same rows as a contiguous copy"""
    import torch
    N, KB = 50, 9
    idx, gain, x = synth.layer(6, 5300 + M, N, 24 * KB, M)
    d_idx, d_gain = _dev(synth.pack_u48(idx).reshape(-1)), _dev(gain.reshape(-1))
    wide = torch.full((M, 24 * KB + 8), 7.0, dtype=torch.float16, device="cuda:0")
    wide[:, 8:] = _dev(x).half()
    ref = oracle13.matmul(x, idx, gain)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for stream in (None, side):
        y = torch.empty((M, N), dtype=torch.float32, device="cuda:0")
        torch.cuda.synchronize()
        gpu.llvq_matmul(wide[:, 8:], d_idx, d_gain, N, KB, out=y, stream=stream)
        torch.cuda.synchronize()
        assert np.abs(y.cpu().numpy().astype(np.float64) - ref).max() / np.abs(ref).max() <= 2e-3
