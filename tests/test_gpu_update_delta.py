"""Incremental M-step of a fit at the edges of its chunks (16384 vectors), slices (at most 512, of 4 clusters at least) and rounds (2048 chunks): centroids are the
bits of the same iterations made one call at a time, each of which sums every vector anew, and codes those of an E-step for them."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,d,K,by_cells", [(3 << 19, 4, 2048, True), ((3 << 19) + 1, 4, 2049, True), ((3 << 19) + 16383, 6, 1025, True), (33 * 16384 - 1, 8, 8193, False),
                                            (32 * 16384 + 33, 16, 4097, False), (16384 * 3 + 5, 4, 8192, False), (9000, 4, 8200, False), (4_300_000, 4, 33000, True),
                                            (2_200_000, 8, 1024, True), (32 * 16384, 4, 256, False),
                                            (32 * 16384 + 1, 4, 2049, False), (600_000, 6, 259, False), (2048 * 16384, 4, 1030, True), (2049 * 16384 + 77, 4, 1030, True)])
def test_a_fit_is_its_iterations_one_by_one(N, d, K, by_cells):
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
    assert (cc.read_stats(ws).list_stages > 0) == by_cells   # one slice holds few clusters: only a fit by cells then sums incrementally
    one, codes = c0.clone(), torch.empty_like(idx)
    for _ in range(iters):
        cc.lloyd_iter(x, one, codes, None, None, ws)
    cc.assign(x, one, codes, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(c, one) and torch.equal(idx.view(torch.int32), codes.view(torch.int32))
