"""The forward pass with each column of the codebook in LDS (the layer listing of Section 3.2 and the quantised codebook of
Section 4.4; g = 4 .. 9): in-features short of a matrix-core step or not filling the last one, one code column, odd numbers of
them, row tiles and their edges, and codebooks on either side of the sizes at which the kernel changes, against the product
with the rebuilt weight in float64. A workspace without room for the kernel's own copies gives the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DTYPES = {"f16": (torch.float16, 2.0 ** -11), "bf16": (torch.bfloat16, 2.0 ** -8)}


def _inputs(M, i, o, g, K, dt):
    gen = torch.Generator(device="cuda").manual_seed(M * 7 + i + o * 3 + g + K)
    x = torch.randn(M, i, device="cuda", generator=gen).to(DTYPES[dt][0])
    codes = torch.randint(0, K, (i * -(-o // g),), device="cuda", generator=gen)
    codes[0], codes[-1] = K - 1, 0
    bias = torch.randn(o, device="cuda", generator=gen).to(DTYPES[dt][0])
    return gen, x, codes, bias


def _integers(n, bits, gen):
    return torch.randint(-(1 << (bits - 1)), 1 << (bits - 1), (n,), device="cuda", generator=gen, dtype=torch.int32)


def _stored(q, bits):
    """The codebook of these integers as it is stored."""
    if bits == 8:
        return q.to(torch.int8).view(torch.uint8)
    even = torch.nn.functional.pad(q & 15, (0, q.numel() % 2))
    return (even[0::2] | (even[1::2] << 4)).to(torch.uint8)


def _check(call, x, weight, scale, bias, dt, workspaces):
    """y against x . weight * scale + bias: half a unit of the format, and the accumulation of in_features terms in fp32."""
    M, o = x.shape[0], bias.shape[0]
    s = scale if scale is not None else 1.0
    want, size = (x.double() @ weight) * s + bias.double(), (x.double().abs() @ weight.abs()) * s
    tol = DTYPES[dt][1] * want.abs() + x.shape[1] * 2.0 ** -24 * size + 2.0 ** -24
    first = None
    for nbytes in workspaces:
        y = torch.full((M, o), 9.0, dtype=x.dtype, device="cuda")
        call(y, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
        assert bool(((y.double() - want).abs() <= tol).all())
        assert first is None or torch.equal(first, y)
        first = y


SHAPES = [(1, 8, 4, 4, 9), (2, 24, 30, 5, 33), (3, 40, 11, 9, 200), (16, 4096, 1029, 4, 65536), (17, 264, 515, 6, 65500),
          (32, 1032, 2001, 7, 20480), (33, 72, 700, 8, 20481), (64, 520, 300, 9, 40960), (65, 200, 1100, 4, 40961), (256, 136, 250, 8, 8191),
          (200, 1000, 90, 6, 8192), (1, 12296, 64, 8, 65536), (4, 4096, 4100, 4, 50000), (384, 64, 129, 5, 4096)]


@pytest.mark.parametrize("dt", list(DTYPES))
@pytest.mark.parametrize("M,i,o,g,K", SHAPES)
def test_forward_by_columns(M, i, o, g, K, dt):
    import paper_2503_13089_amd as cc

    gen, x, codes, bias = _inputs(M, i, o, g, K, dt)
    book = (torch.randn(K, g, device="cuda", generator=gen) * 0.05).to(x.dtype)
    weight = book.double()[codes].reshape(i, -1)[:, :o].contiguous()
    full, least = cc.layer_forward_workspace_bytes(M, i, o), 64 * M * o * 4
    codes16 = codes.to(torch.int32).to(torch.int16).view(torch.uint16)
    print(f"forward M={M} {i}->{o} g={g} K={K} {dt}", flush=True)
    _check(lambda y, ws: cc.layer_forward(x, book, codes16, o, bias, y, ws), x, weight, None, bias, dt, (full, min(full, least)))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("dt", list(DTYPES))
@pytest.mark.parametrize("M,i,o,g,K", SHAPES)
def test_forward_by_columns_with_the_quantised_codebook(M, i, o, g, K, dt, bits):
    import paper_2503_13089_amd as cc

    gen, x, codes, bias = _inputs(M, i, o, g, K, dt)
    q = _integers(K * g, bits, gen)
    qbook = _stored(q, bits)
    weight = q.double().reshape(K, g)[codes].reshape(i, -1)[:, :o].contiguous()
    scale = torch.full((1,), 0.0078125, device="cuda")
    full, least = cc.layer_forward_q_workspace_bytes(M, i, o), 64 * M * o * 4
    codes16 = codes.to(torch.int32).to(torch.int16).view(torch.uint16)
    print(f"forward_q M={M} {i}->{o} g={g} K={K} {dt} {bits} bits", flush=True)
    _check(lambda y, ws: cc.layer_forward_q(x, qbook, bits, scale, K, g, codes16, o, bias, y, ws), x, weight, 0.0078125, bias, dt,
           (full, min(full, least)))


@pytest.mark.parametrize("bits", [16, 8, 4])
@pytest.mark.parametrize("g", [4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("M,K", [(1, 1), (2, 3), (1, 65536), (3, 20480), (33, 40960)])
def test_columns_straight_from_the_codebook(M, K, g, bits):
    """The least workspace (none for 16 bits, sums of 64 slices for integers): every workgroup takes its columns out of rows of any
    alignment, the last entry of a row and the last row of the codebook among them."""
    import paper_2503_13089_amd as cc

    i, o, dt = 128, 70, "bf16"
    gen, x, codes, bias = _inputs(M, i, o, g, K, dt)
    codes16 = codes.to(torch.int32).to(torch.int16).view(torch.uint16)
    if bits == 16:
        book = (torch.randn(K, g, device="cuda", generator=gen) * 0.05).to(x.dtype)
        weight = book.double()[codes].reshape(i, -1)[:, :o].contiguous()
        _check(lambda y, ws: cc.layer_forward(x, book, codes16, o, bias, y, ws), x, weight, None, bias, dt, (cc.layer_forward_workspace_bytes(M, i, o), 0))
        return
    q = _integers(K * g, bits, gen)
    qbook, scale = _stored(q, bits), torch.full((1,), 0.125, device="cuda")
    weight = q.double().reshape(K, g)[codes].reshape(i, -1)[:, :o].contiguous()
    _check(lambda y, ws: cc.layer_forward_q(x, qbook, bits, scale, K, g, codes16, o, bias, y, ws), x, weight, 0.125, bias, dt,
           (cc.layer_forward_q_workspace_bytes(M, i, o), 64 * M * o * 4))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("dt", list(DTYPES))
@pytest.mark.parametrize("M,g,K", [(1, 4, 65536), (16, 5, 65536), (3, 6, 4096), (16, 8, 20480), (2, 8, 65536), (17, 9, 65536)])
def test_a_weight_of_zero_rounds_nothing(M, g, K, dt, bits):
    """Large inputs that meet integers of zero: their products are zero, so that the bound of the small terms' sum holds
    (2e-4 here; half a unit of fp32 at 8 times a large input would be 1.6e-2)."""
    import paper_2503_13089_amd as cc

    i, o = 264, 515
    gen, x, codes, bias = _inputs(M, i, o, g, K, dt)
    x, bias = x / 64, torch.zeros_like(bias)
    x[:, 5::32] = 32768.0 + 32.0 * torch.arange(M, device="cuda", dtype=torch.float32)[:, None]
    q = _integers(K * g, bits, gen).reshape(K, g)
    q[K // 2] = 0
    codes = codes.reshape(i, -1)
    codes[5::32] = K // 2
    codes = codes.reshape(-1)
    weight = q.double()[codes].reshape(i, -1)[:, :o].contiguous()
    qbook, scale = _stored(q.reshape(-1), bits), torch.ones(1, device="cuda")
    codes16 = codes.to(torch.int32).to(torch.int16).view(torch.uint16)
    _check(lambda y, ws: cc.layer_forward_q(x, qbook, bits, scale, K, g, codes16, o, bias, y, ws), x, weight, 1.0, bias, dt,
           (cc.layer_forward_q_workspace_bytes(M, i, o),))


@pytest.mark.parametrize("bits", [16, 8, 4])
@pytest.mark.parametrize("M", [1, 3, 40])
def test_infinite_inputs_reach_their_own_outputs_only(M, bits):
    import paper_2503_13089_amd as cc

    i, o, g, K = 264, 515, 6, 4096
    gen, x, codes, bias = _inputs(M, i, o, g, K, "bf16")
    x[M - 1, i - 3] = float("inf")
    codes16 = codes.to(torch.int32).to(torch.int16).view(torch.uint16)
    y = torch.empty(M, o, dtype=torch.bfloat16, device="cuda")
    if bits == 16:
        book = (torch.randn(K, g, device="cuda", generator=gen) * 0.05).bfloat16()
        book[7, 2] = float("inf")
        ws = torch.empty(cc.layer_forward_workspace_bytes(M, i, o), dtype=torch.uint8, device="cuda")
        cc.layer_forward(x, book, codes16, o, bias, y, ws)
    else:
        book = _integers(K * g, bits, gen)
        ws = torch.empty(cc.layer_forward_q_workspace_bytes(M, i, o), dtype=torch.uint8, device="cuda")
        cc.layer_forward_q(x, _stored(book, bits), bits, torch.ones(1, device="cuda"), K, g, codes16, o, bias, y, ws)
        book = book.reshape(K, g)
    weight = book.double()[codes].reshape(i, -1)[:, :o].contiguous()
    want = (x.double().cpu() @ weight.cpu() + bias.double().cpu()).numpy()
    got = y.double().cpu().numpy()
    odd = ~np.isfinite(want)
    assert odd.any() and (M == 1 or not odd.all())
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[odd & ~np.isnan(want)], want[odd & ~np.isnan(want)])
