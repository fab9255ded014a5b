"""Fits by cells of 5 to 8 numbers with 192 or more vectors per centroid leave out the vectors whose code provably cannot have changed
(Section 3.1: the codes are the argmin over all centroids): over many iterations, with codebooks at the edges of how the moves of the
centroids are kept, equal centroids, centroids that jump between clumps and inputs that are no fp16 numbers, codes, centroids and
objective are those of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = (1 << 21) + 45


@pytest.mark.parametrize("d,K,iters,kind", [
    (8, 1024, 14, "plain"), (8, 1031, 9, "equal"), (6, 10921, 12, "plain"), (5, 4097, 20, "clumps"), (8, 2049, 12, "fp32"), (7, 1500, 12, "tiny"),
    (8, 10924, 9, "plain")])   # the last: one centroid too many for the form
def test_codes_that_cannot_change_are_those_of_the_direct_form(d, K, iters, kind):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(d * K + iters)
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    if kind == "clumps":   # centroids start in one clump of many, and travel
        x += 0.2 * torch.randn(40, d, device="cuda", generator=gen)[torch.randint(0, 40, (N,), device="cuda", generator=gen)]
    if kind == "tiny":     # squares among the subnormal numbers
        x.mul_(2.0 ** -60)
    elif kind != "fp32":
        x = x.half().float()
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    if kind == "equal":
        c0[K // 2:] = c0[:K - K // 2].clone()
    if kind == "clumps":
        c0 = (c0 - c0.mean(0)) * 0.05 + x[0]
        c0 = c0.half().float().contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"bounds d={d} K={K} iters={iters} {kind} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, iters, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32), j))
    (c, idx, j), (c1, idx1, j1) = out
    assert torch.equal(c, c1) and torch.equal(idx, idx1)
    assert j.item() == pytest.approx(j1.item(), rel=1e-12)   # the same N numbers, added in another order in 64 bits
