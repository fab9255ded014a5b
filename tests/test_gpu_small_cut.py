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
