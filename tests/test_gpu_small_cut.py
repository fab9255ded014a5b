"""A small fit gives a compute unit one workgroup or two, whichever leaves less to do (Section 3.1's iteration): where the number of
vectors per workgroup or of ways to split the codebook changes, either has the bits of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,d,K", [(16384, 4, 256), (16385, 4, 256), (32769, 16, 200), (49153, 8, 131), (65536, 4, 256), (65600, 4, 256),
                                   (98305, 4, 900), (131073, 4, 128), (512001, 4, 100)])
def test_one_or_two_workgroups_per_compute_unit(N, d, K):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"small cut N={N} d={d} K={K} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 3, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("N,d,K", [(65536, 4, 1024), (65537, 4, 832), (65537, 4, 833), (131072, 4, 832), (131073, 4, 832), (131073, 4, 560), (131073, 4, 561), (65536, 8, 700),
                                   (65537, 8, 700), (131072, 8, 608), (131073, 8, 608), (131073, 8, 512), (400003, 8, 368), (400003, 8, 369)])
@pytest.mark.parametrize("kind", ["fp16", "fp32"])
def test_where_small_problems_end(N, d, K, kind):
    """Either side of the lines between this form and the matrix cores: a fit, an iteration and an E-step alone have the bits of the direct form."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    x = x.half().float() if kind == "fp16" else x
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        print(f"end of small problems N={N} d={d} K={K} {kind} mode={mode}", flush=True)
        c, one, j = torch.empty_like(c0), c0.clone(), torch.zeros(1, dtype=torch.float64, device="cuda")
        idx = [torch.empty(N, dtype=torch.uint32, device="cuda") for _ in range(3)]
        cc.kmeans_fit(x, K, 3, c0, c, idx[0], j, ws, assign_mode=mode)
        cc.lloyd_iter(x, one, idx[1], None, None, ws, assign_mode=mode)
        cc.assign(x, c0, idx[2], None, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append([c, one] + [i.view(torch.int32) for i in idx])
    assert all(torch.equal(a, b) for a, b in zip(*out))
