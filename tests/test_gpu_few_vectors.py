"""E-steps of few vectors (32, 64, 128 or 256 to a workgroup) at the edges of where each takes over, over the whole codebook and by windows, fp16
inputs and others: codes and means are the bits of the direct form; and fits whose M-step goes by slices although no order is kept."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,N,K", [(4, 8192, 2048), (4, 8193, 8192), (4, 49152, 1000), (4, 49153, 8200), (4, 65535, 8192), (4, 65536, 8192), (4, 524289, 1030),
                                   (8, 129, 128), (8, 8193, 8193), (8, 98304, 950), (8, 98305, 9000), (8, 1048577, 1100),
                                   (16, 701, 700), (16, 10001, 10000), (16, 131073, 8200), (16, 40001, 401), (6, 161, 129), (12, 65537, 8300)])
@pytest.mark.parametrize("kind", ["fp16", "fp32"])
def test_few_vectors_have_the_bits_of_the_direct_form(d, N, K, kind):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    c0 = torch.randn(K, d, device="cuda", generator=gen).mul_(0.02)
    c0[K // 2:K // 2 + 40] = c0[:40] if K >= 80 else c0[K // 2:K // 2 + 40]   # equal centroids: the lower index wins
    if kind == "fp16":
        x, c0 = x.half().float(), c0.half().float()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):   # automatic, direct form
        c, idx, counts = c0.clone(), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.empty(K, dtype=torch.uint32, device="cuda")
        print(f"few vectors d={d} N={N} K={K} {kind} mode={mode}", flush=True)
        for _ in range(2):
            cc.lloyd_iter(x, c, idx, None, counts, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32), counts.view(torch.int32)))
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("d,N,K", [(4, 5003, 999), (4, 1200003, 9001), (6, 1100003, 1027), (8, 70001, 8195), (16, 40003, 515), (16, 2200003, 1000)])
@pytest.mark.parametrize("apart", [1, 2, 4, 7])
def test_among_equal_neighbours_the_lowest_index_wins(d, N, K, apart):
    """Index recovery shares a group's candidates among four lanes: equal centroids in one lane's rows and in its neighbours'."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K + apart)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    c = torch.randn(K, d, device="cuda", generator=gen).mul_(0.02).half().float()
    n = (K - apart) // (2 * apart) * (2 * apart)
    pairs = c[:n].view(-1, 2, apart, d)
    pairs[:, 1] = pairs[:, 0]
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        idx, j = torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"equal neighbours d={d} N={N} K={K} apart={apart} mode={mode}", flush=True)
        cc.assign(x, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append(idx.view(torch.int32))
    assert torch.equal(*out)
