"""A workspace without room for cells or for the form for small problems (Section 3.1's iteration in either way) is accepted by
every call, and gives the bits of one that has it."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# `least`: bytes of the arrays that every call needs
@pytest.mark.parametrize("N,d,K,least", [(1 << 22, 4, 1024, 442513408), (1 << 21, 6, 1500, 389461504),
                                         (20011, 6, 200, 4086016), (40000, 4, 300, 4620544)])
def test_calls_take_the_least_workspace(N, d, K, least):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    Xd = g.dev(X)
    ws = torch.empty(max(least, cc.workspace_bytes(N, d, K)), dtype=torch.uint8, device="cuda")
    got = []
    for nbytes in (least, ws.numel()):
        part = ws[:nbytes]
        print(f"workspace of {nbytes} bytes, N={N} d={d} K={K}", flush=True)
        C, idx, J, _ = g.gpu_fit(X, C0, 4, ws=part, Xd=Xd)
        a, Ja = g.gpu_assign(Xd, C, ws=part)
        Cl, il = g.dev(C), torch.empty(N, dtype=torch.uint32, device="cuda")
        cc.lloyd_iter(Xd, Cl, il, None, None, part)
        u, counts, _ = g.gpu_update(Xd, idx, C, ws=part)
        got.append((C, idx, a, Cl.cpu().numpy(), il.cpu().numpy(), u, counts, np.float64([J, Ja])))
    for p, q in zip(*got):
        assert p.tobytes() == q.tobytes()
    with pytest.raises(cc.CCError):
        g.gpu_fit(X, C0, 1, ws=ws[:least - 256], Xd=Xd)


def test_codebook_gradient_and_compression_take_the_least_workspace():
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(7)
    K, g, i, o, least = 4096, 8, 2048, 8192, 322862336
    n = cc.layer_num_codes(i, o, g)
    codes = torch.randint(0, K, (n,), device="cuda", generator=gen).to(torch.int16).view(torch.uint16)
    dw = torch.randn(i, o, device="cuda", generator=gen)
    for grad in (dw, dw.bfloat16()):
        res = []
        for nbytes in (least, cc.workspace_bytes(n, g, K)):
            out = torch.empty(K, g, device="cuda")
            print(f"gradient {grad.dtype}, workspace of {nbytes} bytes", flush=True)
            cc.layer_codebook_grad(grad, codes, K, g, out, torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
            res.append(out.cpu().numpy().tobytes())
        assert res[0] == res[1]
    K, g, i, o, least = 65500, 6, 4096, 4096, 615840256
    w = (torch.randn(o, i, device="cuda", generator=gen) * 0.02).bfloat16()
    n = cc.layer_num_codes(i, o, g)
    ids = torch.randperm(n, device="cuda", generator=gen)[:K].to(torch.int32).view(torch.uint32)
    res = []
    for nbytes in (least, cc.layer_compress_workspace_bytes(o, i, g, K)):
        book, out = torch.empty(K, g, dtype=torch.bfloat16, device="cuda"), torch.empty(n, dtype=torch.uint16, device="cuda")
        print(f"compression, workspace of {nbytes} bytes", flush=True)
        cc.layer_compress(w, g, 4, ids, book, out, None, torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        res.append((book.view(torch.int16).cpu().numpy().tobytes(), out.view(torch.int16).cpu().numpy().tobytes()))
    assert res[0] == res[1]
