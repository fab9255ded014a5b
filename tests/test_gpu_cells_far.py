"""Far vectors of a fit by cells go 32, 64, 128 or (d = 8) 256 to a workgroup, by how many there are (Section 3.1: the codes are the
argmin over all centroids): for each of these, with a codebook whose last group of tiles is not whole, codes and centroids are the bits
of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,d,K,share,least,most", [
    ((1 << 22) + 77, 4, 1055, 0.0005, 1, 8192), ((1 << 22) + 77, 4, 1055, 0.004, 8193, 16384), ((1 << 22) + 77, 4, 1055, 0.02, 16385, 1 << 22),
    ((1 << 21) + 33, 8, 1025, 0.0005, 1, 8192), ((1 << 21) + 33, 8, 1025, 0.004, 8193, 16384),
    ((1 << 21) + 33, 8, 1025, 0.02, 16385, 131072), ((1 << 21) + 33, 6, 1025, 0.15, 131073, 1 << 21)])
def test_far_vectors_have_the_codes_of_the_direct_form(N, d, K, share, least, most):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(K + d)
    places = torch.randn(K, d, device="cuda", generator=gen).mul_(0.05)
    x = places[torch.randint(0, K, (N,), device="cuda", generator=gen)] + 0.002 * torch.randn(N, d, device="cuda", generator=gen)
    x[:int(share * N)] += 0.05 * torch.randn(int(share * N), d, device="cuda", generator=gen)   # of no place in particular
    x = x.half().float()
    c0 = places.half().float()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"far vectors N={N} d={d} K={K} share={share} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 5, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        if mode == 0:
            far = int(ws[64:68].view(torch.int32).item())   # WsHeader::far_count
        out.append((c, idx.view(torch.int32)))
    print("far:", far, flush=True)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert least <= far <= most


@pytest.mark.parametrize("d,copies,seed", [(4, 131, 0), (8, 1092, 1)])
def test_more_than_half_of_the_vectors_far(d, copies, seed):
    """Every centroid many times over: no list has room for its cell's, so all vectors are far, 512 to a window, of one octave of
    norms or many."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(seed)
    K, N = 65500 // copies * copies, (3 << 19) + 1025
    x = (torch.randn(N, d, device="cuda", generator=gen) * 0.02 * torch.exp(torch.randn(N, 1, device="cuda", generator=gen))).half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K // copies]].repeat(copies, 1).contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"all far N={N} d={d} K={K} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 3, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        if mode == 0:
            far = int(ws[64:68].view(torch.int32).item())
        out.append((c, idx.view(torch.int32)))
    print("far:", far, flush=True)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert far > N // 2


@pytest.mark.parametrize("N,d,K,share,least,most", [
    ((3 << 19) + 77, 4, 1055, 0.0001, 1, 2048), ((3 << 19) + 77, 4, 1055, 0.02, 8192, 131072), ((1 << 22) + 77, 4, 1055, 0.15, 131073, 1 << 20),
    ((3 << 19) + 33, 8, 1025, 0.004, 1, 131072), ((1 << 21) + 33, 8, 1025, 0.15, 131073, 1 << 20)])
def test_far_vectors_that_are_no_fp16_numbers(N, d, K, share, least, most):
    """128 to a workgroup up to 2^17 of them, else 512; workgroups take turns."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(K + d)
    c0 = torch.randn(K, d, device="cuda", generator=gen).mul_(0.05)
    x = c0[torch.randint(0, K, (N,), device="cuda", generator=gen)] + 0.002 * torch.randn(N, d, device="cuda", generator=gen)
    x[:int(share * N)] += 0.05 * torch.randn(int(share * N), d, device="cuda", generator=gen)
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"far fp32 vectors N={N} d={d} K={K} share={share} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 5, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        if mode == 0:
            far = int(ws[64:68].view(torch.int32).item())
        out.append((c, idx.view(torch.int32)))
    print("far:", far, flush=True)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert least <= far <= most
