"""Fits large enough (d = 6 .. 8, K >= 16384, N >= 2^21, N * K >= 1.2e11; d = 5 4.5e11) that the first E-step goes by cells too, grouped by the codes of a bootstrap and of one
look at the lists: codes and centroids are the bits of the same fit with every E-step over the whole codebook (Section 3.1: the
codes are the argmin over all centroids), the objective is the sum of the same numbers in another order."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,kind", [(8, "fp16"), (6, "fp16"), (8, "fp32"), (8, "clumped")])
def test_first_estep_by_cells_gives_the_bits_of_the_whole_codebook(d, kind):
    import paper_2503_13089_amd as cc

    N, K, iters = 18_400_011, 65536, 3
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    if kind == "clumped":   # a third of the vectors close to one of 3000 places: lists that run over, cells of every size
        place = torch.randn(3000, d, device="cuda", generator=gen).mul_(0.05)
        some = torch.randint(0, 3000, (N // 3,), device="cuda", generator=gen)
        x[:N // 3] = place[some] + 0.01 * x[:N // 3]
    if kind != "fp32":
        x = x.half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 3):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"first E-step by cells d={d} {kind} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, iters, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32), j))
    (c, idx, j), (c_whole, idx_whole, j_whole) = out
    assert torch.equal(c, c_whole) and torch.equal(idx, idx_whole)
    assert abs(j.item() - j_whole.item()) <= 2.0 ** -52 * N * j_whole.item()


@pytest.mark.parametrize("N,d,K", [(5_344_129, 7, 65500), (5_340_456, 8, 65536), (21_362_305, 8, 16384), (11_250_013, 5, 40000), (6_870_000, 5, 65500),
                                   (2_097_152, 8, 57221), (7_324_219, 6, 16384), (2_097_151, 7, 60000)])
def test_fits_at_the_line_have_the_bits_of_the_whole_codebook(N, d, K):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 3):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"line of first E-steps by cells N={N} d={d} K={K} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 4, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32), j))
    (c, idx, j), (c_whole, idx_whole, j_whole) = out
    assert torch.equal(c, c_whole) and torch.equal(idx, idx_whole)
    assert abs(j.item() - j_whole.item()) <= 2.0 ** -52 * N * j_whole.item()
