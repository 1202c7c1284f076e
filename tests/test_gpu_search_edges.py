"""Inputs at which the bounds of llvq_quantize's search rule out little, and the edges of the block-wise loop's step inside it."""
import numpy as np
import pytest

from paper_2603_11021_amd import synth, LLVQ_IDX_U48
from oracle.gptq_oracle import inverse_hessian_factor, spherical_gptq
from test_gpu_quantize import _check, _dev, gpu  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def _ties():
    """Vectors to which many points are equally near: one, two, four, eight or all coordinates of one magnitude"""
    rows = []
    for k in (1, 2, 4, 8, 12, 23, 24):
        v = np.zeros(24)
        v[:k] = 1.0
        rows += [v, -v, v * np.where(np.arange(24) % 2, -1.0, 1.0)]
    return np.array(rows)


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -100, 2.0 ** 60])
def test_search_among_many_equal_candidates(gpu, oracle13, scale):  # noqa: F811
    _check(gpu, oracle13, _ties() * scale, "angular", 0.0)          # any of the equals is right: only the score is compared


@pytest.mark.parametrize("norm", [0.01, 5.0, 11.0, 40.0])
def test_euclidean_search_inside_and_outside_of_the_ball(gpu, oracle13, norm):  # noqa: F811
    w = synth.rng_for(10, 77).standard_normal((40, 24))
    w *= norm / np.linalg.norm(w, axis=1, keepdims=True)
    _check(gpu, oracle13, w, "euclidean", 0.9)


@pytest.mark.parametrize("n_levels", [1, 64, 65, 130])
def test_gain_levels_more_and_fewer_than_lanes(gpu, n_levels):  # noqa: F811
    """Block column 0 sees the original rows: its gain is the nearest level, the lower one of two equally near.  2049 rows are
    one more than the waves of a launch.  Rows of norm 3 exactly lie halfway between two levels."""
    N, KB = 2049, 2
    W = synth.rng_for(11, 40 + n_levels).standard_normal((N, 24 * KB)).astype(np.float32)
    W[::100, :24] = 0.0
    W[::100, :9] = 1.0
    levels = (np.array([2.5, 3.5]) if n_levels == 64 else np.linspace(2.5, 7.5, max(n_levels, 2)))[:n_levels]
    levels = np.sort(np.concatenate([levels, np.linspace(8.0, 9.0, n_levels - levels.size)])).astype(np.float16)
    U = np.eye(24 * KB, dtype=np.float32)
    idx, gain = gpu.llvq_gptq_quantize(_dev(W.copy()), _dev(U), LLVQ_IDX_U48, gain_levels=_dev(levels))
    norm = np.linalg.norm(W[:, :24].astype(np.float64), axis=1)
    d = np.abs(norm[:, None] - levels.astype(np.float64)[None, :])
    two = np.sort(d, axis=1)[:, :2]
    exact = np.arange(N) % 100 == 0                                  # norms that fp32 holds exactly
    safe = exact | (two[:, -1] - two[:, 0] > 1e-5) | (n_levels == 1)  # elsewhere fp32 may fall on the other side of a midpoint
    want = levels[np.argmin(d, axis=1)]
    assert safe.mean() > 0.95 and np.array_equal(gain.cpu().numpy()[safe, 0], want[safe])


@pytest.mark.parametrize("N,KB", [(1, 1), (1, 3), (3, 2)])
def test_block_loop_of_few_rows(gpu, oracle13, N, KB):  # noqa: F811
    """Fewer rows than waves in a workgroup, a single block column (nothing to propagate to), strongly coupled columns"""
    rng = synth.rng_for(11, 60 + N + KB)
    X = rng.standard_normal((200, 24 * KB)) @ (np.eye(24 * KB) + 0.3 * rng.standard_normal((24 * KB, 24 * KB)))
    U = inverse_hessian_factor(X.T @ X / 200 + 0.05 * np.eye(24 * KB))
    W = (0.02 * rng.standard_normal((N, 24 * KB))).astype(np.float32)
    d_W = _dev(W.copy())
    gpu.llvq_gptq_quantize(d_W, _dev(U.astype(np.float32)), LLVQ_IDX_U48)
    ref, _, _ = spherical_gptq(oracle13, W.astype(np.float64), U)
    # gains are fp16 (2^-11 where one rounds the other way); the propagated error stays in fp32
    assert np.abs(d_W.cpu().numpy() - ref).max() <= 2.0 ** -10 * np.abs(ref).max()
