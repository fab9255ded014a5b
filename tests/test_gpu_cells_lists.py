"""Lists of the cells at d = 5 .. 8 get their two radii from one product, scaled per cell (Section 3.1: the codes are the argmin over all
centroids): with magnitudes at both ends of what the scale can carry, radii that coincide and cells without a list, codes and centroids are
those of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, K = (1 << 21) + 5, 2051


@pytest.mark.parametrize("d,scale,kind", [(8, 2.0 ** -9, "plain"), (8, 2.0 ** 14, "plain"), (6, 1.0, "wide"), (8, 1.0, "wide"), (7, 2.0 ** 9, "offset"),
                                          (8, 1.0, "few values"), (5, 2.0 ** -40, "plain"), (8, 3.0e9, "plain")])
def test_lists_of_every_magnitude_hold_the_nearest(d, scale, kind):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(int(d + 8 * abs(scale) ** 0.1))
    x = torch.randn(N, d, device="cuda", generator=gen).mul_(0.02)
    if kind == "wide":         # magnitudes over six orders
        x *= torch.exp(3.0 * torch.randn(N, 1, device="cuda", generator=gen))
        x.clamp_(-200.0, 200.0)
    elif kind == "offset":     # far from the origin: norms large against the radii
        x += 1.0
    elif kind == "few values":   # most vectors on their centroid, radii of zero
        x = torch.where(torch.rand(N, 1, device="cuda", generator=gen) < 0.9, (x * 40).round() / 40, x)
    if scale * 0.02 > 1e-6 and scale < 1e6:
        x = (x * scale).clamp_(-60000.0, 60000.0).half().float()
    else:
        x = x * scale
    c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    ws = torch.empty(cc.workspace_bytes(N, d, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"lists d={d} scale={scale} {kind} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 6, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        out.append((c, idx.view(torch.int32)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
