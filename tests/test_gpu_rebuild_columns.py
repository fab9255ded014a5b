"""The weight rebuilt for prefill batches (the layer listing of Section 3.2 and the quantised codebook of Section 4.4) by columns
of the codebook: rows of x with a single 1 read the rebuilt matrix back through the product, which is exact, so every element
must be the codebook's. Sizes on either side of where the row-by-row form ends, in-features and widths that do not fill a
fragment, one code column, the sizes of the codebook at which more columns fit, and no room for a laid-out codebook."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

M = 400  # the rebuilt route at every sub-vector length


def _unit_rows(i, dtype):
    rows = torch.arange(M, device="cuda")
    rows = torch.where(rows < M // 2, rows % i, (i - 1 - rows) % i)  # the first and the last in-features
    x = torch.zeros(M, i, dtype=dtype, device="cuda")
    x[torch.arange(M, device="cuda"), rows] = 1.0
    return rows, x


def _codes(i, o, g, K):
    gen = torch.Generator(device="cuda").manual_seed(i + 3 * o + g + K)
    codes = torch.randint(0, K, (i * -(-o // g),), device="cuda", generator=gen)
    codes[0], codes[-1] = K - 1, 0
    return gen, codes, codes.to(torch.int32).to(torch.int16).view(torch.uint16)


SHAPES = [(1024, 4096, 4, 65536), (1024, 4100, 4, 65536), (136, 32700, 4, 65500), (520, 8200, 8, 65536), (40, 13109, 9, 50000),
          (520, 1031, 9, 40961), (392, 3001, 6, 40960), (400, 2999, 5, 20481), (1032, 5003, 7, 20480), (392, 1500, 16, 8192),
          (392, 1400, 1, 8191), (264, 2050, 2, 300), (200, 2701, 3, 1), (65544, 9, 9, 700), (65544, 17, 9, 65536), (32776, 35, 15, 4096)]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("i,o,g,K", SHAPES)
def test_rebuilt_weight(i, o, g, K, dtype):
    import paper_2503_13089_amd as cc

    rows, x = _unit_rows(i, dtype)
    gen, codes, codes16 = _codes(i, o, g, K)
    book = (torch.randn(K, g, device="cuda", generator=gen) * 0.05).to(dtype)
    weight = book[codes].reshape(i, -1)[:, :o]
    y = torch.full((M, o), 9.0, dtype=dtype, device="cuda")
    ws = torch.full((cc.layer_forward_workspace_bytes(M, i, o),), 255, dtype=torch.uint8, device="cuda")  # NaN in either format
    print(f"rebuild {i}x{o} g={g} K={K} {dtype}", flush=True)
    cc.layer_forward(x, book, codes16, o, None, y, ws)
    assert torch.equal(y, weight[rows])


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("i,o,g,K", [(1032, 4099, 4, 65536), (136, 3001, 9, 50000), (520, 1031, 6, 30001), (264, 2050, 8, 4096), (72, 700, 5, 999)])
def test_rebuilt_integers(i, o, g, K, bits):
    import paper_2503_13089_amd as cc

    rows, x = _unit_rows(i, torch.bfloat16)
    gen, codes, codes16 = _codes(i, o, g, K)
    ints = torch.randint(-(1 << (bits - 1)), 1 << (bits - 1), (K * g + K * g % 2,), device="cuda", generator=gen)
    packed = ints if bits == 8 else (ints[0::2] & 15) | ((ints[1::2] & 15) << 4)
    qbook = packed.to(torch.uint8)[:(K * g * bits + 7) // 8].contiguous()
    weight = ints[:K * g].view(K, g)[codes].reshape(i, -1)[:, :o].to(torch.bfloat16)
    y = torch.full((M, o), 9.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.full((cc.layer_forward_q_workspace_bytes(M, i, o),), 255, dtype=torch.uint8, device="cuda")
    print(f"rebuild of integers {i}x{o} g={g} K={K} bits={bits}", flush=True)
    cc.layer_forward_q(x, qbook, bits, torch.ones(1, device="cuda"), K, g, codes16, o, None, y, ws)
    assert torch.equal(y, weight[rows])
