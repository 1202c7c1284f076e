"""llvq_gptq_group_scales at the sizes where its kernels change shape: rows that do not fill a wave, block columns that do not
fill a group of four, systems of one panel and of several, the largest system that is solved in LDS and one that is not."""
import numpy as np
import pytest

from paper_2603_11021_amd import synth
from oracle.gptq_oracle import group_scales

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,KB,lam", [(1, 1, 0.0), (33, 16, 0.0), (7, 17, 2e-3), (129, 31, 0.0), (300, 33, 4e-3), (3, 65, 0.0), (6, 171, 1e-3),
                                      (2, 270, 0.0), (2, 276, 0.0), (2, 301, 0.0)])
def test_group_scales_against_the_normal_equations(N, KB, lam):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_11021_amd import LLVQ
    q = LLVQ(13, 0)
    K = 24 * KB
    rng = synth.rng_for(12, 1000 * KB + N)
    X = rng.standard_normal((64, K))
    H = (X.T @ X / 64 + np.diag(np.linspace(0.5, 2.0, K))).astype(np.float32)
    gain = (0.1 * np.exp(0.2 * rng.standard_normal((N, KB)))).astype(np.float16)
    d_gain = torch.from_numpy(gain).to("cuda:0")
    idx = torch.from_numpy(synth.pack_u48(synth.indices(rng, (N, KB))).reshape(-1)).to("cuda:0")
    d_Wq = q.llvq_decode(idx, d_gain.reshape(-1), out_dtype=torch.float32).reshape(N, K)
    Wq = d_Wq.cpu().numpy()
    W0 = (Wq + 0.01 * rng.standard_normal((N, K))).astype(np.float32)
    s = q.llvq_gptq_group_scales(d_Wq, torch.from_numpy(W0).to("cuda:0"), torch.from_numpy(H).to("cuda:0"), d_gain, lam=lam).cpu().numpy()
    want = group_scales(W0.astype(np.float64), Wq.astype(np.float64), H.astype(np.float64), lam=lam)
    assert np.allclose(s, want, rtol=2e-3, atol=2e-4), np.abs(s - want).max()
    g1 = d_gain.cpu().numpy()
    assert (np.abs(g1.astype(np.float64) - gain.astype(np.float64) * s) <= 2.0 ** -10 * np.abs(gain.astype(np.float64) * s) + 6e-8).all()
    ratio = np.repeat(g1.astype(np.float64) / gain.astype(np.float64), 24, axis=1)
    assert np.allclose(d_Wq.cpu().numpy(), Wq * ratio, rtol=1e-5, atol=1e-9)


def test_group_scales_leave_a_row_without_a_definite_system_as_it_is():
    """an indefinite 'Hessian': the factorisation meets a negative pivot and the row keeps its gains"""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_11021_amd import LLVQ
    q = LLVQ(13, 0)
    N, KB = 5, 20
    K = 24 * KB
    rng = synth.rng_for(12, 7)
    Wq = rng.standard_normal((N, K)).astype(np.float32)
    gain = np.ones((N, KB), dtype=np.float16)
    d_Wq, d_gain = torch.from_numpy(Wq).to("cuda:0"), torch.from_numpy(gain).to("cuda:0")
    H = np.diag(np.where(np.arange(K) < 24 * 17, 1.0, -1.0)).astype(np.float32)
    s = q.llvq_gptq_group_scales(d_Wq, torch.from_numpy(2 * Wq).to("cuda:0"), torch.from_numpy(H).to("cuda:0"), d_gain).cpu().numpy()
    assert (s == 1.0).all() and np.array_equal(d_gain.cpu().numpy(), gain) and np.array_equal(d_Wq.cpu().numpy(), Wq)
