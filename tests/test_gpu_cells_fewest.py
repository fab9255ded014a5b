"""Fits at the line from which E-steps go by cells (1.5 * 2^20 vectors, 24 per centroid), on either side of it: centroids, codes and cost have the bits of the
direct-form kernels, with few vectors to a cell and many cells without a list."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N0 = 3 << 19


@pytest.mark.parametrize("N,d,K,by_cells", [(N0, 4, 65536, True), (N0 + 31, 3, 1024, True), (N0, 8, 65536, True), (N0 + 63, 6, 1025, True), (N0 + 1, 5, 20000, True),
                                            (N0 - 1, 8, 4096, False), (N0, 4, 65537, False), (N0, 8, 1023, False)])
def test_fits_of_few_vectors_to_a_cell_have_the_bits_of_the_direct_form(N, d, K, by_cells):
    import paper_2503_13089_amd as cc
    from tests import gpu_helpers as g

    X, C0 = workloads.make_small(N, d, K, seed=N + d + K)
    Xd, ws = g.dev(X), g.workspace(N, d, K)
    got = []
    try:
        for mode in (0, 1):
            cc.set_assign_mode(mode)
            print(f"fit at the line of cells N={N} d={d} K={K} mode {mode}", flush=True)
            got.append(g.gpu_fit(X, C0, 7, ws=ws, Xd=Xd))
            if mode == 0:
                assert (cc.read_stats(ws).list_stages > 0) == by_cells
    finally:
        cc.set_assign_mode(0)
    (C, idx, J, _), (C1, idx1, J1, _) = got
    assert C.tobytes() == C1.tobytes() and idx.tobytes() == idx1.tobytes()
    assert J == pytest.approx(J1, rel=1e-12)
