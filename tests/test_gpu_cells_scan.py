"""Near vectors of 4 numbers are scored relative to their cell's centroid, four entries of its list at a time (Section 3.1: the codes are the argmin over
all centroids, the lowest index among equals): where several centroids are equally near, in one group or in several, and
where numbers are no fp16 numbers, codes and centroids are the bits of the direct form."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = (3 << 19) + 190


@pytest.mark.parametrize("K,copies,kind", [
    (3000, 2, "points"), (5000, 5, "points"), (33 * 400, 33, "points"), (2000, 1, "plain"), (2000, 1, "small"), (2000, 1, "fp32"), (60000, 1, "large")])
def test_near_vectors_have_the_codes_of_the_direct_form(K, copies, kind):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(K + copies)
    if kind == "points":   # as many vectors to either side of a centroid, which stays there: all its copies tie in every E-step
        distinct = torch.randint(-20, 21, (K // copies, 4), device="cuda", generator=gen).float() / 256
        half = distinct[torch.randint(0, K // copies, (N // 2,), device="cuda", generator=gen)]
        side = torch.randint(-1, 2, (N // 2, 4), device="cuda", generator=gen).float() / 1024
        x = torch.cat([half + side, half - side])
        c0 = distinct.repeat(copies, 1)[torch.randperm(K // copies * copies, device="cuda", generator=gen)].contiguous()
    else:
        x = 0.02 * torch.randn(N, 4, device="cuda", generator=gen)
        x = x.mul_({"small": 2.0 ** -2, "large": 2.0 ** 16}.get(kind, 1.0))
        if kind == "plain":
            x = x.half().float()
        c0 = x[torch.randperm(N, device="cuda", generator=gen)[:K]].contiguous()
    K = len(c0)
    ws = torch.empty(cc.workspace_bytes(N, 4, K), dtype=torch.uint8, device="cuda")
    out = []
    for mode in (0, 1):
        c, idx, j = torch.empty_like(c0), torch.empty(N, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        print(f"scan K={K} copies={copies} {kind} mode={mode}", flush=True)
        cc.kmeans_fit(x, K, 5, c0, c, idx, j, ws, assign_mode=mode)
        torch.cuda.synchronize()
        if mode == 0:
            near = 1.0 - int(ws[64:68].view(torch.int32).item()) / N   # WsHeader::far_count
        out.append((c, idx.view(torch.int32), j.item()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][2] == pytest.approx(out[1][2], rel=1e-12)
    print(f"near: {near:.3f}", flush=True)
    assert near > 0.5
