"""Small problems (Section 3.1's iteration in two launches) at the ends of the range of finite numbers: codes, counts, centroids and objectives have the bits of the
direct form, in variants that split the codebook among the waves of a workgroup and in those that do not."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# not split / split 8 ways, scores
SHAPES = [(1048577, 4, 64), (20000, 4, 130), (65537, 8, 3), (300001, 8, 50), (20000, 8, 130), (1000001, 16, 250), (32769, 16, 130)]


def results(x, c0, mode):
    import paper_2503_13089_amd as cc

    (N, d), K = x.shape, c0.shape[0]
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    c, one, counts = torch.empty_like(c0), c0.clone(), torch.empty(K, dtype=torch.uint32, device="cuda")
    idx = [torch.empty(N, dtype=torch.uint32, device="cuda") for _ in range(3)]
    j = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(3)]
    cc.kmeans_fit(x, K, 2, c0, c, idx[0], j[0], ws, assign_mode=mode)
    cc.lloyd_iter(x, one, idx[1], j[1], counts, ws, assign_mode=mode)
    cc.assign(x, c0, idx[2], j[2], ws, assign_mode=mode)
    torch.cuda.synchronize()
    return [one.view(torch.int32), counts.view(torch.int32), c.view(torch.int32)] + [i.view(torch.int32) for i in idx] + [v.view(torch.int64) for v in j]


@pytest.mark.parametrize("N,d,K", SHAPES)
def test_numbers_that_doubled_would_overflow(N, d, K):
    """Every 97th vector has a component of 1.5 * 2^127, and the first centroids are such vectors: finite distances, and sums that hold the component."""
    gen = torch.Generator(device="cuda").manual_seed(N + d + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    rows = torch.arange(0, N, 97, device="cuda")
    big = 1.5 * 2.0 ** 127
    x[rows, rows % d] = torch.where(rows // 97 % 2 == 0, big, -big)
    giants = min(2 * d, (K + 1) // 2)
    c0 = torch.cat([x[rows[:giants]], x[1 + 97 * torch.arange(K - giants, device="cuda") % (N - 1) // 97 * 97]]).contiguous()
    assert c0.shape == (K, d)
    print(f"giants N={N} d={d} K={K}", flush=True)
    got, want = results(x, c0, 0), results(x, c0, 1)
    assert (want[0].view(torch.float32).abs() > 2.0 ** 126).any()   # a mean holds it
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("N,d,K", SHAPES)
@pytest.mark.parametrize("levels", [2, 4, 8, 16])
def test_vectors_of_few_values(N, d, K, levels):
    """Numbers of 1 to 4 bits: centroids have doubles or lie equally near, and scores leave all vectors of a wave undecided, some or few."""
    gen = torch.Generator(device="cuda").manual_seed(N + d + K + levels)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(levels / 8).round_().clamp_(-levels // 2, levels // 2 - 1).mul_(0.125)
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    print(f"few values N={N} d={d} K={K} {levels}", flush=True)
    for a, b in zip(results(x, c0, 0), results(x, c0, 1)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("N,d,K", SHAPES)
@pytest.mark.parametrize("log2", [61, 62, 63, 64])
def test_norms_that_overflow_beside_finite_distances(N, d, K, log2):
    """Vectors and centroids of 2^60 to 2^66: some squared norms and some distances are finite, others not."""
    gen = torch.Generator(device="cuda").manual_seed(N + d + K + log2)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(2.0 ** log2)
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    c0[K // 2] = 0.0
    # one coordinate each: a centroid at 1.9e19, whose square is no finite number, is the nearest of the vector at 1e19, not the one at the origin
    x[:64] = 0.0
    x[:64, 0] = 1.0e19
    c0[K - 1] = 0.0
    c0[K - 1, 0] = 1.9e19
    print(f"norms N={N} d={d} K={K} 2^{log2}", flush=True)
    for a, b in zip(results(x, c0, 0), results(x, c0, 1)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("blocks", [1, 15, 16, 17, 112, 113, 127, 128, 129, 240, 241, 255, 256, 257, 511, 512])
def test_sums_of_any_number_of_workgroups(blocks):
    """Sixteen threads add the workgroups' sums of an entry, eight requests at a time: none is left out or counted twice, whatever their number (64 or 128 vectors each)."""
    N, d, K = 64 * blocks, 4, 5
    gen = torch.Generator(device="cuda").manual_seed(blocks)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    print(f"workgroups {blocks}", flush=True)
    for a, b in zip(results(x, c0, 0), results(x, c0, 1)):
        assert torch.equal(a, b)
