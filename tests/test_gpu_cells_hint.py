"""Where the vectors of a fit by cells stand in the norm order (Section 3.1's E-step pruned by codes) is written by its last grouping alone: after fits that
end before, with and after the later groupings, the next call finds the codes they left, each vector its own."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# groupings: d = 4 at iterations 1 and 5, d = 8 with so many vectors in the first one and at 2 and 5
@pytest.mark.parametrize("N,d,K,iters", [((1 << 21) + 3, 4, 8200, 3), ((1 << 21) + 3, 4, 8200, 5), ((1 << 21) + 3, 4, 8200, 6), ((1 << 21) + 3, 4, 8200, 8),
                                         ((1 << 23) - 9, 8, 16384, 3), ((1 << 23) - 9, 8, 16384, 5), ((1 << 23) - 9, 8, 16384, 6), ((1 << 23) - 9, 7, 16384, 7)])
def test_the_next_call_finds_the_codes(N, d, K, iters):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(iters)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02).half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    c, idx, out, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    print(f"hint N={N} d={d} K={K} iters={iters}", flush=True)
    cc.kmeans_fit(x, K, iters, c0, c, idx, j, ws)
    stages = []
    for _ in range(2):
        cc.assign(x, c, out, None, ws)
        torch.cuda.synchronize()
        st = cc.read_stats(ws)
        assert st.total_stages == -(-N // 512) * -(-K // 32)   # no bootstrap
        assert torch.equal(out.view(torch.int32), idx.view(torch.int32))
        stages.append(st.scored_stages)
    assert stages[0] == stages[1]   # windows as wide as the codes' own leave them
