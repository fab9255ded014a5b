"""What workspaces hold: cells (large fits, the E-step of Section 3.1) and the form for small problems take little beyond the
arrays that every call needs, and a workspace without room for them is still accepted (tests/test_gpu_workspace.py)."""
import pytest

import paper_2503_13089_amd as cc


# (N, d, K): bytes of the arrays that every call needs, and how many times that the full size may be
@pytest.mark.parametrize("N,d,K,least,times", [
    (1 << 20, 4, 4096, 111327488, 1.0),          # neither form
    (1 << 22, 4, 1024, 442513408, 1.13), (11272192, 4, 65536, 1207075328, 1.13), (29360128, 8, 65536, 4545749504, 1.09),
    (4096 * 683, 6, 65500, 535936256, 1.85),     # the lists do not fit the M-step's buffer
    (40000, 4, 300, 4620544, 1.0), (20011, 6, 200, 4086016, 1.25)])
def test_workspace_is_little_more_than_every_call_needs(N, d, K, least, times):
    assert least <= cc.workspace_bytes(N, d, K) <= times * least
