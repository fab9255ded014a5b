"""Fits by cells (Section 3.1: the codes are the argmin over all centroids) on data that is awkward for groups and lists, against
the direct-form kernels: cells that are empty at one grouping and not at the next, the other way round, numbers that no list
can be made for, Inf and NaN, and calls that follow on the same workspace."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N4, N8 = 1 << 22, 1 << 21   # cells of many vectors


def fits(X, C0, iters, ws, modes=(0, 1)):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    Xd, got = g.dev(X), []
    try:
        for mode in modes:
            cc.set_assign_mode(mode)
            print(f"fit N={X.shape[0]} d={X.shape[1]} K={len(C0)} iters={iters} mode {mode}", flush=True)
            got.append(g.gpu_fit(X, C0, iters, ws=ws, Xd=Xd))
    finally:
        cc.set_assign_mode(0)
    return got


def same(a, b):
    assert a[0].tobytes() == b[0].tobytes() and a[1].tobytes() == b[1].tobytes()
    assert a[2] == pytest.approx(b[2], rel=1e-12)


def small_cells(N, d, seed):
    """A bulk, 20000 vectors far from it with 8000 centroids, 200 of these twice (cells of two or three vectors, and empty ones
    that fill once the first of a pair has moved), and 64 threes of cells the middle one of which loses its two vectors to the
    others in the second E-step."""
    rng = np.random.default_rng(seed)
    out = rng.standard_normal((20000, d)) * 0.3
    out *= 2 / np.sqrt(np.linalg.norm(out, axis=1, keepdims=True))
    side = np.array([-0.5, -0.25, 0.25, 0.5])
    base = np.zeros((64, d))
    base[:, 1:4] = np.stack(np.meshgrid(side, side, side), -1).reshape(-1, 3)

    def along(*at):   # in units of 2^-10
        return (base[:, None, :] + np.pad(np.array(at)[:, None] / 1024, ((0, 0), (0, d - 1)))).reshape(-1, d)

    few = along(0, 100, -1, 106)
    bulk = rng.standard_normal((N - len(out) - len(few), d)) * 0.02
    X = np.concatenate([out, few, bulk]).astype(np.float16).astype(np.float32)
    pick = rng.permutation(20000)[:7800]
    C0 = np.concatenate([X[pick], X[pick[:200]], along(20, -21, 190), X[-2000:]]).astype(np.float32)
    return X[rng.permutation(N)], C0


@pytest.mark.parametrize("N,d,seed", [(N4, 4, 0), (N8, 8, 1)])
def test_cells_that_empty_and_fill(N, d, seed):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = small_cells(N, d, seed)
    K, iters = len(C0), 12
    ws = g.workspace(N, d, K)
    a, b = fits(X, C0, iters, ws)
    same(a, b)
    # the data is what it is meant to be: sizes of the cells at the groupings (after 1, 3 and 8 iterations)
    Xd, C, counts, size = g.dev(X), g.dev(C0), torch.empty(K, dtype=torch.uint32, device="cuda"), []
    idx = torch.empty(N, dtype=torch.uint32, device="cuda")
    for _ in range(8):
        cc.lloyd_iter(Xd, C, idx, None, counts, ws, assign_mode=1)
        torch.cuda.synchronize()
        size.append(counts.cpu().numpy().astype(np.int64))
    at = [size[0], size[2], size[7]]
    assert any(((p == 0) & (q > 0)).any() for p, q in zip(at, at[1:])) and any(((p > 0) & (q == 0)).any() for p, q in zip(at, at[1:]))


@pytest.mark.parametrize("N,d,K", [(N4 + 5, 4, 1024), (N8 + 5, 8, 1100)])
def test_numbers_too_large_for_lists(N, d, K):
    """Numbers of 2^14 and more that are no fp16 numbers: all vectors are far, and scored on the fp32 matrix cores."""
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    s = np.float32(20000.7 / np.abs(X).max())
    a, b = fits(X * s, C0 * s, 4, g.workspace(N, d, K))
    assert a[3].fp16_inputs == 0
    same(a, b)


@pytest.mark.parametrize("N,d,K", [(N4 + 5, 4, 1024), (N8 + 5, 6, 1100)])
def test_non_finite_vectors_leave_the_others_their_codes(N, d, K):
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    X = X.copy()
    odd = np.array([0, 63, 64, 1000, N // 2, N - 1])
    X[odd[::2], d - 1], X[odd[1::2], 0], X[odd[3], 1] = np.inf, np.nan, -np.inf
    ws = g.workspace(N, d, K)
    a, = fits(X, C0, 5, ws, modes=(0,))
    b, = fits(X, C0, 5, ws, modes=(0,))
    assert a[0].tobytes() == b[0].tobytes() and a[1].tobytes() == b[1].tobytes()       # every time the same
    assert a[3].nonfinite_inputs == 1 and np.isfinite(a[0]).all() and (a[1] < K).all()
    fine = np.ones(N, bool)
    fine[odd] = False
    import paper_2503_13089_amd as cc
    out = torch.empty(N, dtype=torch.uint32, device="cuda")
    cc.assign(g.dev(X), g.dev(a[0]), out, None, ws, assign_mode=1)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy()[fine], a[1][fine])


@pytest.mark.parametrize("N,d,K,least", [(N4 + 5, 4, 8192, 443785728), (N8 + 5, 8, 8200, 323773952)])   # bytes that every call needs
def test_other_calls_on_the_workspace_of_a_fit(N, d, K, least):
    """What a fit by cells leaves behind, codes to start from included, changes nothing for other vectors of the same shape."""
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=1)
    Y = X[np.random.default_rng(2).permutation(N)] * np.float32(0.5)
    ws = g.workspace(N, d, K)
    Yd, C0d = g.dev(Y), g.dev(C0)
    first, = fits(X, C0, 4, ws, modes=(0,))
    want = torch.empty(N, dtype=torch.uint32, device="cuda")
    cc.assign(Yd, C0d, want, None, g.workspace(N, d, K), assign_mode=1)
    idx, _ = g.gpu_assign(Yd, C0d, ws=ws)
    assert np.array_equal(idx, want.cpu().numpy())
    again, = fits(X, C0, 4, ws, modes=(0,))
    assert again[0].tobytes() == first[0].tobytes() and again[1].tobytes() == first[1].tobytes()
    # the codes are there, where they lie in the workspace is not: a call with less of it
    idx, _ = g.gpu_assign(Yd, C0d, ws=ws[:least])
    assert np.array_equal(idx, want.cpu().numpy())
