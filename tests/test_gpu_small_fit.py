"""Small problems take a form of their own (Section 3.1's iteration in two launches): at the edges of how it
deals the vectors out, every result has the bits of the direct-form kernels and of the fused matrix-core route."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,d,K", [(1, 4, 1), (63, 4, 5), (65, 8, 64), (4097, 16, 129),
                                   (32768, 4, 300), (32769, 4, 300),    # 1 -> 2 groups of 64 vectors per workgroup
                                   (65537, 8, 257), (131073, 16, 130),  # codebook split 4 and 2 ways
                                   (262145, 4, 1000), (300001, 4, 3),   # not split; a handful of large clusters
                                   (40000, 4, 1496), (40000, 4, 1497),  # the largest codebook that fits, the first that does not
                                   (20011, 6, 200)])                    # padded sub-vectors
def test_small_problems_have_the_bits_of_the_other_routes(N, d, K):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    X[-1] = X[0]  # an exact duplicate
    Xd, ws = g.dev(X), g.workspace(N, d, K)
    got = {}
    try:
        for mode in (0, 1, 3):
            cc.set_assign_mode(mode)
            print(f"small problem N={N} d={d} K={K} mode {mode}", flush=True)
            C, idx, J, st = g.gpu_fit(X, C0, 3, ws=ws, Xd=Xd)
            assert st.assign_calls == 4
            Cl, il = g.dev(C0), torch.empty(N, dtype=torch.uint32, device="cuda")
            counts, Jl = torch.empty(K, dtype=torch.uint32, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
            cc.lloyd_iter(Xd, Cl, il, Jl, counts, ws)
            torch.cuda.synchronize()
            got[mode] = (C, idx, Cl.cpu().numpy(), il.cpu().numpy(), counts.cpu().numpy(), np.float64([J, float(Jl.item())]))
    finally:
        cc.set_assign_mode(0)
    for mode in (1, 3):
        for a, b in zip(got[0], got[mode]):
            assert a.tobytes() == b.tobytes(), mode
