"""The rebuilt weight by parts of the codebook (g = 4, 16-bit, many codes): exact, at the sizes where parts and shares end."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("K", [4096, 4097, 20463, 20464, 20465, 40928, 40929, 61392, 61393, 65535, 65536])
@pytest.mark.parametrize("in_features,out_features,shift", [(2048, 4096, 0), (3000, 4204, 1), (4096, 8196, 0)])
def test_weight_by_parts_of_the_codebook(dt, K, in_features, out_features, shift):
    """`shift`: codes that begin 2 bytes past a word. The last two codes, and some at the ends of parts, are beyond or at K - 1."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(K + in_features)
    n = in_features * out_features // 4
    codes = torch.randint(0, K, (n + shift,), device="cuda", generator=gen, dtype=torch.int32)[shift:]
    codes[:4] = torch.tensor([0, K - 1, min(K, 65535), 65535], device="cuda", dtype=torch.int32)
    codes[-2:] = 65535
    buf = torch.empty(n + shift, dtype=torch.int16, device="cuda")
    buf[shift:] = codes.to(torch.int16)
    book = torch.randint(-(1 << 15), 1 << 15, (K, 4), device="cuda", generator=gen, dtype=torch.int32).to(torch.int16)   # any bits
    W = torch.empty((in_features, out_features), dtype=torch.int16, device="cuda")
    print(f"weight by parts K={K} {in_features}x{out_features} {dt}", flush=True)
    cc.layer_weight(book.view(dt), buf[shift:].view(torch.uint16), in_features, out_features, W.view(dt))
    assert torch.equal(W.view(-1, 4), book[codes.clamp(max=K - 1).long()])
