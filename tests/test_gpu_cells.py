"""Large fits decide most vectors on a list of the centroids near their last one (Section 3.1: the codes are the argmin over
all centroids): at the edges of how cells, lists and their tiles are dealt out, every result has the bits of the
direct-form kernels."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N4, N8 = 1 << 22, 1 << 21   # cells of many vectors; the fewest are in test_gpu_cells_fewest.py


@pytest.mark.parametrize("N,d,K,iters,kind", [
    (N4, 4, 1024, 3, "plain"), (N4 + 77, 4, 1055, 9, "plain"), (N4 + 1, 3, 32768, 4, "plain"), (N4, 4, 2048, 4, "fp32"),
    (N4, 4, 4096, 4, "clumped"),
    (N8, 8, 1024, 9, "plain"), (N8 + 33, 8, 1025, 3, "plain"), (N8 + 1, 5, 65536, 3, "plain"), (N8 + 63, 6, 65500, 4, "plain"),
    (N8, 8, 2048, 3, "fp32"), (N8, 8, 4096, 4, "clumped"), (N8, 7, 1500, 4, "one value")])
def test_fits_by_cells_have_the_bits_of_the_direct_form(N, d, K, iters, kind):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    rng = np.random.default_rng(K)
    if kind == "fp32":          # no fp16 numbers: lists from their fp16 parts, far vectors on the fp32 matrix cores
        X = (X * np.float32(1.0009)).astype(np.float32)
    elif kind == "clumped":     # more centroids close together than a list has room for, and exact duplicates
        C0 = C0.copy()
        C0[K // 4:] = C0[0] + (rng.standard_normal((K - K // 4, d)) * 1e-4).astype(np.float16).astype(np.float32)
        C0[-8:] = C0[0]
    elif kind == "one value":   # one enormous cell
        X = X.copy()
        X[: 3 * N // 4] = X[0]
    Xd, ws = g.dev(X), g.workspace(N, d, K)
    got = []
    try:
        for mode in (0, 1):
            cc.set_assign_mode(mode)
            print(f"fit by cells N={N} d={d} K={K} iters={iters} {kind} mode {mode}", flush=True)
            got.append(g.gpu_fit(X, C0, iters, ws=ws, Xd=Xd))
    finally:
        cc.set_assign_mode(0)
    (C, idx, J, _), (C1, idx1, J1, _) = got
    assert C.tobytes() == C1.tobytes() and idx.tobytes() == idx1.tobytes()
    assert J == pytest.approx(J1, rel=1e-12)


@pytest.mark.parametrize("N,d,K", [(N4 + 77, 4, 8192), (N8 + 33, 6, 8200)])
def test_a_fit_by_cells_leaves_its_codes_as_the_next_call_s_hint(N, d, K):
    """An E-step that finds no codes of a previous one scores the whole order of tiles twice, with a bootstrap pass first."""
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    Xd, ws = g.dev(X), g.workspace(N, d, K)
    one_pass = -(-N // 512) * -(-K // 32)
    for call in ("assign", "lloyd_iter"):
        print(f"hint after a fit by cells N={N} d={d} K={K} {call}", flush=True)
        C, idx, _, _ = g.gpu_fit(X, C0, 4, ws=ws, Xd=Xd)
        Cd, out = g.dev(C), torch.empty(N, dtype=torch.uint32, device="cuda")
        if call == "assign":
            cc.assign(Xd, Cd, out, None, ws)
        else:
            cc.lloyd_iter(Xd, Cd, out, None, None, ws)
        torch.cuda.synchronize()
        st = cc.read_stats(ws)
        assert st.total_stages == one_pass
        # ... and the hint is each vector's own code: windows as wide as a converged E-step's
        assert np.array_equal(out.cpu().numpy(), idx)
        again = st.scored_stages
        cc.assign(Xd, g.dev(C), out, None, ws)
        torch.cuda.synchronize()
        assert cc.read_stats(ws).scored_stages == again and np.array_equal(out.cpu().numpy(), idx)


def clumps(N, d, K, seed):
    """K / 2 clumps, two centroids each: one in the middle of a clump and one so far beyond its end that the first E-step
    gives it the outermost vector only. That becomes its place, and from the next E-step on it has a quarter of the clump."""
    rng = np.random.default_rng(seed)
    m = K // 2
    centre = rng.uniform(-0.5, 0.5, size=(m, d)).astype(np.float16).astype(np.float32)
    h = 0.06
    X = np.repeat(centre, N // m, axis=0).reshape(m, N // m, d)
    u = rng.uniform(0.0, 0.9, size=(m, N // m))
    u[:, 0] = 1.0
    X = X + rng.normal(scale=0.01 * h, size=X.shape)
    X[:, 0] = centre                    # the outermost vector lies on the axis
    X[:, :, 0] += h * u
    C0 = np.repeat(centre, 2, axis=0)
    C0[0::2, 0] += 0.5 * h
    C0[1::2, 0] += 1.4 * h
    X = X.reshape(-1, d)
    X = X[rng.permutation(len(X))]
    return X.astype(np.float16).astype(np.float32), C0.astype(np.float32)


@pytest.mark.parametrize("N,d,K", [(N4, 4, 2048), (N8, 8, 2048)])
def test_cells_that_begin_with_one_vector_get_lists_when_they_grow(N, d, K):
    from tests import gpu_helpers as g

    X, C0 = clumps(N, d, K, seed=d)
    Xd, ws = g.dev(X), g.workspace(N, d, K)
    scored = []
    for iters in (5, 10):
        print(f"growing cells N={N} d={d} K={K} iters={iters}", flush=True)
        C, idx, _, st = g.gpu_fit(X, C0, iters, ws=ws, Xd=Xd)
        scored.append(st.scored_stages)
    assert 0.4 < np.bincount(idx, minlength=K)[1::2].sum() / N < 0.6     # every second cell has half a clump
    # tiles of 32 centroids per 512 vectors and E-step: 0.3 to 0.5 where the lists serve them, 2.8 to 3.0 where half of the
    # vectors go through the windows in every one
    assert (scored[1] - scored[0]) / 5 < 1.4 * N / 512


@pytest.mark.parametrize("N,d,K", [(N4, 4, 1024), (N8, 8, 1024)])
def test_profile_and_statistics_tell_lists_from_windows(N, d, K):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=5)
    Xd, C0d, ws, iters = g.dev(X), g.dev(C0), g.workspace(N, d, K), 5
    C, idx = torch.empty_like(C0d), torch.empty(N, dtype=torch.uint32, device="cuda")
    prof = cc.Profile(max_records=512)
    print(f"profile of a fit by cells N={N} d={d} K={K}", flush=True)
    cc.kmeans_fit(Xd, K, iters, C0d, C, idx, None, ws, profile=prof)
    ms, launches, dropped = prof.read()
    prof.close()
    st = cc.read_stats(ws)
    # a bootstrap and a first E-step by windows, `iters` more by cells: lists (direct form at d = 4), then far vectors
    assert dropped == 0 and launches["estep_direct"] == (iters if d == 4 else 0)
    assert launches["estep_f16"] == 2 + (iters if d == 4 else 2 * iters)
    assert all((ms[k] > 0.0) == (n > 0) for k, n in launches.items())
    # every vector meets at least its own centroid, none more than there are (pairs in units of 32 x 512; each of the K / 32
    # workgroups rounds its share)
    pairs = st.list_stages * 16384.0
    slack = iters * 16384.0 * K / 32
    assert iters * N - slack <= pairs <= iters * N * K + slack and st.list_stages <= st.scored_stages
