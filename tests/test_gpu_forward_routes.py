"""The forward pass on either side of the row counts where it changes from gathering codebook rows to rebuilding the weight
(Section 3.2's layer listing), and the rebuilt route on the shortest and most ragged shapes that take it."""
import pytest

from tests import test_gpu_layer as layer

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

cc = layer.cc


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("M,in_features,out_features,g,K", [
    (128, 4096, 8200, 4, 65536), (129, 4096, 8200, 4, 65536),   # 2^25 weights and more
    (256, 2048, 2056, 8, 4096), (257, 2048, 2056, 8, 4096), (257, 2048, 2051, 4, 4096),   # 2^22
    (384, 512, 520, 4, 4096), (385, 512, 520, 4, 4096),
    (128, 264, 515, 3, 2000), (129, 264, 515, 3, 2000), (384, 264, 515, 6, 2000), (385, 264, 515, 6, 2000), (385, 264, 515, 9, 2000)])
def test_both_sides_of_a_change_of_route(cc, M, in_features, out_features, g, K, dt):
    layer.test_layer_forward(cc, M, in_features, out_features, g, K, True, dt)


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("M,in_features,out_features,g,K", [(400, 8, 40, 4, 100), (385, 16, 257, 4, 9), (390, 24, 33, 3, 50),
                                                            (513, 200, 300, 4, 500), (400, 4096, 130, 8, 4096),
                                                            (777, 264, 515, 5, 2000), (385, 1024, 2560, 4, 65536)])
def test_rebuilt_route_on_short_and_ragged_shapes(cc, M, in_features, out_features, g, K, dt):
    layer.test_layer_forward_many_rows_meets_the_definition_and_reads_out_weight_rows(cc, M, in_features, out_features, g, K, dt)


def test_workspace_for_the_rebuilt_route_alone_is_enough(cc):
    """Rows that the gathering route would serve, with room for the rebuilt weight only."""
    M, i, o, g, K, dense = 384, 264, 515, 6, 2000, 295936
    assert 0 < dense < cc.layer_forward_workspace_bytes(M, i, o)
    gen = torch.Generator(device="cuda").manual_seed(3)
    codes = torch.randint(0, K, (cc.layer_num_codes(i, o, g),), device="cuda", generator=gen).to(torch.int16).view(torch.uint16)
    book = (torch.randn(K, g, device="cuda", generator=gen) * 0.05).bfloat16()
    x = torch.randn(M, i, device="cuda", generator=gen).bfloat16()
    w = torch.empty(i, o, dtype=torch.bfloat16, device="cuda")
    cc.layer_weight(book, codes, i, o, w)
    want, size = x.double() @ w.double(), x.double().abs() @ w.double().abs()
    for nbytes in (dense, cc.layer_forward_workspace_bytes(M, i, o)):
        y = torch.full((M, o), 9.0, dtype=torch.bfloat16, device="cuda")
        cc.layer_forward(x, book, codes, o, None, y, torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        assert bool(((y.double() - want).abs() <= 2.0 ** -8 * want.abs() + i * 2.0 ** -24 * size).all())
    with pytest.raises(cc.CCError):
        cc.layer_forward(x, book, codes, o, None, y, torch.empty(dense - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("out_features", [1, 7, 8, 65, 255, 259, 518])   # the last piece of 8 columns whole and of each kind of part
@pytest.mark.parametrize("M,in_features", [(385, 8), (513, 40), (641, 1040)])   # whole tiles, one and 128 rows in the last; cut tiles
def test_a_tile_is_stored_to_its_ends_and_no_further(cc, M, in_features, out_features, dt):
    gen = torch.Generator(device="cuda").manual_seed(M + out_features)
    K, g = 500, 4
    codes = torch.randint(0, K, (cc.layer_num_codes(in_features, out_features, g),), device="cuda", generator=gen).to(torch.int16).view(torch.uint16)
    book = (torch.randn(K, g, device="cuda", generator=gen) * 0.05).to(dt)
    x = torch.randn(M, in_features, device="cuda", generator=gen).to(dt)
    bias = torch.randn(out_features, device="cuda", generator=gen).to(dt)
    w = torch.empty(in_features, out_features, dtype=dt, device="cuda")
    cc.layer_weight(book, codes, in_features, out_features, w)
    room = torch.full((M * out_features + 512,), 9.0, dtype=dt, device="cuda")
    y = room[:M * out_features].view(M, out_features)
    ws = torch.empty(cc.layer_forward_workspace_bytes(M, in_features, out_features), dtype=torch.uint8, device="cuda")
    cc.layer_forward(x, book, codes, out_features, bias, y, ws)
    want = x.double() @ w.double() + bias.double()
    size = x.double().abs() @ w.double().abs() + bias.double().abs()
    # exact products, in_features + 1 sums in fp32, one rounding
    tol = (2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -11) * want.abs() + (in_features + 1) * 2.0 ** -24 * size + 2.0 ** -24
    assert bool(((y.double() - want).abs() <= tol).all())
    assert bool((room[M * out_features:] == 9.0).all())
