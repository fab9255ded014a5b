"""The rebuilt weight at every sub-vector length (the layer listing of Section 3.2), 16 and 32 bits: rows that end inside a wave's
codes (often, for narrow matrices), widths of either parity, with and without padding, a single element, element counts on either
side of what a wave takes. The elements are the codebook's, exactly, and nothing past the end is written."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1), (7, 5), (1, 300), (513, 3), (129, 63), (40, 1029), (33, 2050), (5, 4097), (64, 512)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("g", range(1, 17))
def test_weight_rows(g, dtype):
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(g)
    for i, o in SHAPES + [(300, 8 * g), (3, 256 * g), (64, 65 * g - 1)]:
        for K in (1, 777, 65536):
            n = i * -(-o // g)
            codes = torch.randint(0, K, (n,), device="cuda", generator=gen)
            codes[-1] = K - 1
            book = torch.randn(K, g, device="cuda", generator=gen).to(dtype)
            out = torch.full((i * o + 64,), 9.0, dtype=dtype, device="cuda")
            print(f"weight {i}x{o} g={g} K={K} {dtype}", flush=True)
            cc.layer_weight(book, codes.to(torch.int32).to(torch.int16).view(torch.uint16), i, o, out[:i * o])
            assert torch.equal(out[:i * o].view(i, o), book[codes].reshape(i, -1)[:, :o])
            assert bool((out[i * o:] == 9.0).all())
