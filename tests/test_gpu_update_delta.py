"""Incremental M-step of a fit at the edges of its chunks (16384 vectors) and slices (at most 512, of 4 clusters at least): centroids and
codes are the bits of the same iterations made one call at a time, each of which sums every vector anew."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,d,K", [(32 * 16384, 4, 256), (32 * 16384 + 1, 4, 2049), (33 * 16384 - 1, 8, 8193), (32 * 16384 + 33, 16, 4097), (600_000, 6, 259),
                                   (16384 * 3 + 5, 4, 8192), (9000, 4, 8200), (4_300_000, 4, 33000), (2_200_000, 8, 1024)])
def test_a_fit_is_its_iterations_one_by_one(N, d, K):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    x[:N // 5] = x[N // 5]                         # many vectors that all change together
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    c0[::9] += 0.03                                # far from their vectors: most codes change in the first iterations
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    iters = 7
    print(f"fit and its iterations N={N} d={d} K={K}", flush=True)
    c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    cc.kmeans_fit(x, K, iters, c0, c, idx, j, ws)
    one = c0.clone()
    for _ in range(iters):
        cc.lloyd_iter(x, one, idx.clone(), None, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(c, one)
