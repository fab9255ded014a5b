"""Small problems (Section 3.1's iteration in two launches): for each number of vectors to a lane and of ways to split the codebook, with centroids that
are equally near in one group of four, in several and in several parts of the codebook, and with distances that overflow, every
result has the bits of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(16384, 4, 1490), (1048577, 4, 64), (20000, 4, 130), (20000, 4, 111), (262145, 4, 700), (524288, 4, 64), (262145, 4, 113), (65537, 4, 111), (100001, 4, 899), (40000, 4, 3),
          (16384, 8, 575), (65537, 8, 3), (20000, 8, 700), (20000, 8, 111), (270001, 8, 575), (400003, 8, 574), (262145, 8, 64), (65537, 8, 113), (32769, 8, 2), (16384, 16, 299),
          (40000, 16, 1), (100001, 16, 113), (32769, 16, 130), (16384, 16, 390), (40000, 16, 64),
          (50335, 4, 84), (293837, 4, 74), (50241, 8, 90), (265738, 8, 43), (65998, 8, 9), (49292, 8, 259), (114585, 16, 8),
          (131202, 4, 68), (786486, 4, 5), (32914, 4, 24), (524748, 8, 4), (262239, 8, 3), (65642, 8, 25), (32797, 8, 23), (140583, 16, 41), (131137, 16, 43)]


@pytest.mark.parametrize("N,d,K", SHAPES)
@pytest.mark.parametrize("kind", ["fp16", "equal", "fp32", "huge"])
def test_small_problems_have_the_bits_of_the_direct_form(N, d, K, kind):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + d + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    if kind != "fp32":
        x = x.half().float()
    if kind == "huge":
        x[::97] *= 2.0 ** 110
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    if kind == "equal" and K > 2:
        c0[K // 2:] = c0[:K - K // 2].clone()
        c0[K - 1] = c0[0]
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        print(f"small scores N={N} d={d} K={K} {kind} mode={mode}", flush=True)
        c, one, counts = torch.empty_like(c0), c0.clone(), torch.empty(K, dtype=torch.uint32, device="cuda")
        idx = [torch.empty(N, dtype=torch.uint32, device="cuda") for _ in range(3)]
        j = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(3)]
        cc.kmeans_fit(x, K, 2, c0, c, idx[0], j[0], ws, assign_mode=mode)
        cc.lloyd_iter(x, one, idx[1], j[1], counts, ws, assign_mode=mode)
        cc.assign(x, c0, idx[2], j[2], ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append([c.view(torch.int32), one.view(torch.int32), counts.view(torch.int32)] + [i.view(torch.int32) for i in idx] + [v.view(torch.int64) for v in j])
    for a, b in zip(*out):
        assert torch.equal(a, b)
