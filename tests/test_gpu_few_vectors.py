"""E-steps of few vectors (32, 64, 128 or 256 to a workgroup) at the edges of where each takes over and where the kernel with 512 to a workgroup does, over the
whole codebook and by windows, fp16 inputs and others: codes and means are the bits of the direct form; and fits whose M-step goes by slices although no
order is kept."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WHOLE, DIRECT = 3, 1   # cc_assign_mode


def iterations(d, N, K, kind, modes, by_windows=False):
    """Two iterations in either mode."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    c0 = torch.randn(K, d, device="cuda", generator=gen).mul_(0.02)
    c0[K // 2:K // 2 + 40] = c0[:40] if K >= 80 else c0[K // 2:K // 2 + 40]   # equal centroids: the lower index wins
    if kind == "fp16":
        x, c0 = x.half().float(), c0.half().float()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in modes:
        c, idx, counts = c0.clone(), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.empty(K, dtype=torch.uint32, device="cuda")
        print(f"few vectors d={d} N={N} K={K} {kind} mode={mode}", flush=True)
        for _ in range(2):
            cc.lloyd_iter(x, c, idx, None, counts, ws, assign_mode=mode)
        torch.cuda.synchronize()
        stats = cc.read_stats(ws)
        out.append((c, idx.view(torch.int32), counts.view(torch.int32)))
        if by_windows and mode == 0:
            assert 0 < stats.scored_stages <= stats.total_stages
    return out


# In the form that such a call takes by itself: some are small problems.
@pytest.mark.parametrize("d,N,K", [(4, 8192, 2048), (4, 8193, 8192), (4, 49152, 1000), (4, 49153, 8200), (4, 65535, 8192), (4, 65536, 8192), (4, 524289, 1030),
                                   (8, 129, 128), (8, 8193, 8193), (8, 98304, 950), (8, 98305, 9000), (8, 1048577, 1100),
                                   (16, 701, 700), (16, 10001, 10000), (16, 131073, 8200), (16, 40001, 401), (6, 161, 129), (12, 65537, 8300)])
@pytest.mark.parametrize("kind", ["fp16", "fp32"])
def test_few_vectors_have_the_bits_of_the_direct_form(d, N, K, kind):
    got, want = iterations(d, N, K, kind, (0, DIRECT))
    assert all(torch.equal(a, b) for a, b in zip(got, want))


# 32 to a workgroup up to 8192, 64 up to the next line, 128 or 256 up to the last, 512 beyond; of that kernel also its wide groups (d = 4, from 32768 centroids on)
@pytest.mark.parametrize("d,N,K", [(4, 8192, 2048), (4, 8193, 2047), (4, 49152, 1000), (4, 49153, 1001), (4, 1 << 20, 1030), (4, (1 << 20) + 1, 1030), (4, (1 << 20) + 33, 32769),
                                   (8, 129, 128), (8, 8192, 701), (8, 8193, 700), (8, 98304, 950), (8, 98305, 951), (8, 1 << 23, 131), (8, (1 << 23) + 33, 131),
                                   (8, (1 << 23) + 1, 450), (16, 701, 700), (16, 8193, 401), (16, 229376, 300), (16, 229377, 301), (16, 1 << 22, 130), (16, (1 << 22) + 33, 131),
                                   (16, (1 << 22) + 511, 500), (6, 161, 129), (12, 65537, 300)])
@pytest.mark.parametrize("kind", ["fp16", "fp32"])
def test_whole_codebook_has_the_bits_of_the_direct_form(d, N, K, kind):
    got, want = iterations(d, N, K, kind, (WHOLE, DIRECT))
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("d,N,K", [(4, 8192, 8192), (4, 8193, 8192), (4, 49152, 8200), (4, 49153, 8200), (4, 65535, 8192), (4, 65536, 8192), (4, 1 << 19, 8193),
                                   (4, (1 << 19) + 1, 8193), (8, 8192, 8192), (8, 8193, 8193), (8, 98304, 8200), (8, 98305, 9000), (8, 1 << 20, 8193), (8, (1 << 20) + 1, 8193),
                                   (16, 8192, 8192), (16, 10001, 10000), (16, 131072, 8200), (16, 131073, 8200), (16, 1 << 21, 8193), (16, (1 << 21) + 1, 8193), (12, 65537, 8300)])
@pytest.mark.parametrize("kind", ["fp16", "fp32"])
def test_windows_have_the_bits_of_the_direct_form(d, N, K, kind):
    got, want = iterations(d, N, K, kind, (0, DIRECT), by_windows=True)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


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
