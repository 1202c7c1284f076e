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


def test_scratch_of_another_stream_is_not_handed_out_while_it_runs(gpu):
    import torch
    from paper_2603_11021_amd import binding
    n = 3 << 20
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    side = torch.cuda.Stream()
    ws = binding._workspace(n, "cuda:0", side)
    where = ws.data_ptr()
    del ws
    assert torch.empty(n, dtype=torch.uint8, device="cuda:0").data_ptr() != where       # the current stream's memory
    ws = binding._workspace(n, "cuda:0", None)
    where = ws.data_ptr()
    del ws
    assert torch.empty(n, dtype=torch.uint8, device="cuda:0").data_ptr() == where       # kept for the next call of a stream


def test_gptq_on_another_stream(gpu):
    """the block-wise loop and the group scales on a stream of the caller's: the results of the current stream"""
    import torch
    N, K = 64, 24 * 6
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    W = torch.randn((N, K), device="cuda:0", generator=g)
    z = torch.randn((2 * K, K), device="cuda:0", generator=g)
    H = (z.t() @ z / (2 * K) + 0.05 * torch.eye(K, device="cuda:0")).double().cpu().numpy()
    G = np.linalg.inv(H)
    U = _dev(np.linalg.cholesky((G + G.T) / 2).T.astype(np.float32))
    d_H = _dev(H.astype(np.float32))
    results = []
    for stream in (None, torch.cuda.Stream()):
        Wq = W.clone()
        torch.cuda.synchronize()
        idx, gain = gpu.llvq_gptq_quantize(Wq, U, stream=stream)
        s = gpu.llvq_gptq_group_scales(Wq, W, d_H, gain, lam=1e-3, stream=stream)
        torch.cuda.synchronize()
        results.append((idx, gain, s, Wq))
    for a, b in zip(*results):
        assert torch.equal(a, b)
