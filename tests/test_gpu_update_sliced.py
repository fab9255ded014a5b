"""The M-step by cluster slices (Section 3.1: c_k <- mean of its vectors) at the edges of its chunks and slices, on fp32
numbers of every size: the means of the fixed-point sums, bit for bit, computed with numpy's integers."""
import numpy as np
import pytest

from tests import gpu_helpers as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,per_slice", [(4, 4096), (8, 2048), (16, 1024)])
@pytest.mark.parametrize("N,slices,short", [(147 * 7168, 1, 0), (147 * 7168 + 1, 2, 0), (147 * 7168 - 1, 3, 1), (1048576 + 63, 4, 40),
                                            (1048576 + 65, 5, 1), (1048576 + 4097, 13, 5),
                                            (32768, 1, 300), (40000, 2, 3)])
def test_sums_by_slices_are_the_fixed_point_sums(d, per_slice, N, slices, short):
    K = slices * per_slice - short
    rng = np.random.default_rng(N + K + d)
    X = (rng.standard_normal((N, d)) * np.exp(4 * rng.standard_normal((N, 1)))).astype(np.float32)
    X[::1001] *= np.float32(1e-30)
    X[5:9] = -0.0
    idx = rng.integers(0, K, size=N).astype(np.uint32)
    idx[N // 2:N // 2 + 9000] = K - 1          # a chunk and more of one cluster
    idx[[0, 77, N - 1]] = K, 2**31, 2**32 - 1      # no cluster
    prev = rng.standard_normal((K, d)).astype(np.float32)
    keep = idx < K
    for bad in (False, True):
        if bad:                                # left out of the sums, flagged
            X[N // 3, d - 1], X[N - 2, 0] = np.inf, np.nan
        print(f"sums by slices N={N} d={d} K={K} non-finite={bad}", flush=True)
        got, counts, stats = g.gpu_update(X, idx, prev)
        assert stats.skipped_vectors == 3 and stats.nonfinite_inputs == int(bad)
        terms = np.rint(np.ldexp(np.where(np.isfinite(X), X, 0).astype(np.float64), stats.fixed_point_exp)).astype(np.int64)
        n = np.bincount(idx[keep], minlength=K)
        order = np.argsort(idx[keep], kind="stable")
        sums = np.zeros((K, d), np.int64)
        sums[n > 0] = np.add.reduceat(terms[keep][order], np.concatenate(([0], np.cumsum(n)))[:-1][n > 0], axis=0)
        want = np.where(n[:, None] > 0, np.ldexp(sums.astype(np.float64), -stats.fixed_point_exp) / np.maximum(n, 1)[:, None], prev)
        assert np.array_equal(counts, n) and got.tobytes() == want.astype(np.float32).tobytes()
