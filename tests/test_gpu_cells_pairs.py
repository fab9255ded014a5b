"""Lists of the cells at d = 5 .. 8 (Section 3.1) are made from pairs of 32 centroids: where the last pair is full, lacks one centroid or nearly all of
them, codes and centroids are those of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,K", [(8, 2048), (8, 2049), (6, 2079), (8, 2080), (7, 2081), (8, 2111), (5, 16385)])
def test_last_pair(d, K):
    import paper_2503_13089_amd as cc

    N = (1 << 21) + 77
    gen = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"pairs d={d} K={K} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 3, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
