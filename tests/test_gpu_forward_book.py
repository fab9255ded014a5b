"""One to four rows through a layer with g = 4 (Section 3.2's layer listing), a column of the codebook in LDS or two or four of them
(up to 40960 and 20480 rows): in-features that leave a matrix-core step unfilled, fewer steps than waves, a padding column, infinite
inputs and entries, against the product with the rebuilt weight in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dt", ["float16", "bfloat16"])
@pytest.mark.parametrize("M,in_features,out_features,K,kind", [
    (1, 8, 4096, 200, ""), (2, 4096, 1029, 16384, ""),    # less than a step; a padding column, four columns
    (1, 14344, 600, 16385, ""), (2, 7176, 1000, 32769, ""),  # a last step of 8 in-features; two columns
    (4, 3592, 1200, 32768, ""), (3, 4096, 512, 10001, ""), (1, 8192, 8202, 65536, ""),
    (2, 4096, 1032, 20000, "x"), (1, 4096, 1032, 20000, "book")])
def test_few_rows_with_the_codebook_in_parts(M, in_features, out_features, K, kind, dt):
    import paper_2503_13089_amd as cc

    T = getattr(torch, dt)
    gen = torch.Generator(device="cuda").manual_seed(M + in_features + out_features + K)
    per_row = (out_features + 3) // 4
    x = torch.randn(M, in_features, device="cuda", generator=gen).to(T)
    book = (torch.randn(K, 4, device="cuda", generator=gen) * 0.05).to(T)
    codes = torch.randint(0, K, (in_features * per_row,), device="cuda", generator=gen)
    codes[:2], codes[-2:] = K - 1, 0
    bias = torch.randn(out_features, device="cuda", generator=gen).to(T)
    if kind == "x":        # an infinite activation leaves the other row alone
        x[0, 5] = float("inf")
    elif kind == "book":   # so does a row of the codebook that few codes use
        book[K - 3] = float("inf")
    y = torch.full((M, out_features), 9.0, dtype=T, device="cuda")
    ws = torch.empty(max(cc.layer_forward_workspace_bytes(M, in_features, out_features), 256), dtype=torch.uint8, device="cuda")
    print(f"few rows M={M} {in_features}->{out_features} K={K} {kind} {dt}", flush=True)
    cc.layer_forward(x, book, codes.to(torch.int32).to(torch.int16).view(torch.uint16), out_features, bias, y, ws)
    W = book.double().cpu()[codes.cpu()].reshape(in_features, per_row * 4)[:, :out_features]
    xd = x.double().cpu()
    want, mag = (xd @ W + bias.double().cpu()).numpy(), (xd.abs() @ W.abs()).numpy()
    got = y.double().cpu().numpy()
    odd = ~np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[odd & ~np.isnan(want)], want[odd & ~np.isnan(want)])
    tol = (2.0 ** -8 if dt == "bfloat16" else 2.0 ** -11) * np.abs(want) + in_features * 2.0 ** -24 * mag + 2.0 ** -24
    assert not (np.abs(got - want)[~odd] > tol[~odd]).any()
