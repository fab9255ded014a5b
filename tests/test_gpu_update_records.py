"""M-step and 16-bit gradients whose rows go along in the order of the slices: chunks of fp16 numbers, of bf16 numbers and of others side by
side, at the edges of chunks (3584 rows, 1792 of 16) and slices, and gradients at places that no wide load can read."""
import numpy as np
import pytest
import torch

from oracle import layer as L
from tests import gpu_helpers as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,per_slice", [(4, 4096), (8, 2048), (16, 1024)])
@pytest.mark.parametrize("chunks,rest,slices,short", [(300, 0, 2, 0), (300, 1, 16, 1), (299, 3583, 5, 40), (40, 9, 16, 36), (10, 1800, 3, 0)])
def test_rows_in_slice_order_are_the_fixed_point_sums(d, per_slice, chunks, rest, slices, short):
    N, K = chunks * 3584 + rest, slices * per_slice - short
    rng = np.random.default_rng(N + K + d)
    X = (0.02 * rng.standard_normal((N, d))).astype(np.float16).astype(np.float32)
    X[0], X[1], X[2] = 2.0 ** -24, -65504.0, -0.0                          # fp16's ends
    bf = slice(4 * 3584, 6 * 3584 + 7)                               # bf16 numbers below what fp16 holds, and a chunk of both
    X[bf] = ((1e-5 * rng.standard_normal(X[bf].shape)).astype(np.float32).view(np.uint32) & 0xffff0000).view(np.float32)
    X[7 * 3584 + 5, d - 1] = np.float32(1) / 3                       # one number in a chunk that is neither
    idx = rng.integers(0, K, size=N).astype(np.uint32)
    idx[N // 2:N // 2 + 9000] = K - 1
    idx[[0, 77, N - 1]] = K, 2**31, 2**32 - 1                        # no cluster
    prev = rng.standard_normal((K, d)).astype(np.float32)
    keep = idx < K
    for bad in (False, True):
        if bad:
            X[N // 3, d - 1], X[N - 2, 0] = np.inf, np.nan
        print(f"rows by slices N={N} d={d} K={K} non-finite={bad}", flush=True)
        got, counts, stats = g.gpu_update(X, idx, prev)
        assert stats.skipped_vectors == 3 and stats.nonfinite_inputs == int(bad)
        terms = np.rint(np.ldexp(np.where(np.isfinite(X), X, 0).astype(np.float64), stats.fixed_point_exp)).astype(np.int64)
        n = np.bincount(idx[keep], minlength=K)
        order = np.argsort(idx[keep], kind="stable")
        sums = np.zeros((K, d), np.int64)
        sums[n > 0] = np.add.reduceat(terms[keep][order], np.concatenate(([0], np.cumsum(n)))[:-1][n > 0], axis=0)
        want = np.where(n[:, None] > 0, np.ldexp(sums.astype(np.float64), -stats.fixed_point_exp) / np.maximum(n, 1)[:, None], prev)
        assert np.array_equal(counts, n) and got.tobytes() == want.astype(np.float32).tobytes()


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("in_features,out_features,gl,K,shift", [
    (300, 1000, 6, 65500, 0), (301, 777, 5, 300, 0), (512, 448, 7, 4000, 0), (257, 1793, 9, 1024, 0), (260, 2049, 16, 3000, 0), (520, 257, 3, 20000, 0),
    (520, 260, 4, 3000, 2), (300, 1024, 8, 9000, 6), (600, 900, 15, 65536, 0), (40000, 1, 4, 50, 0), (33000, 3, 8, 5000, 0)])
def test_16_bit_gradients_at_any_place(dt, in_features, out_features, gl, K, shift):
    """Sub-vector lengths without wide loads, padded last ones, a gradient that begins `shift` numbers past 16 bytes: the exact sums."""
    import paper_2503_13089_amd as cc

    n = L.num_codes(in_features, out_features, gl)
    assert n >= 32768
    rng = np.random.default_rng(in_features + out_features + gl)
    buf = torch.from_numpy(rng.standard_normal(in_features * out_features + shift).astype(np.float32) * 1e-3).to(dt).cuda()
    G = buf[shift:].view(in_features, out_features)
    codes_np = rng.integers(0, K, size=n).astype(np.uint16)
    codes = torch.from_numpy(codes_np.view(np.int16)).cuda().view(torch.uint16)
    out = torch.full((K, gl), 3.0, device="cuda")
    ws = torch.empty(cc.workspace_bytes(max(n, K), gl, K), dtype=torch.uint8, device="cuda")
    print(f"gradient in place {in_features}x{out_features} g={gl} K={K} {dt} shift={shift}", flush=True)
    cc.layer_codebook_grad(G, codes, K, gl, out, ws)
    want = L.gather_backward(G.float().cpu().numpy(), codes_np, K, gl)
    assert np.array_equal(out.cpu().numpy(), want.astype(np.float32))


@pytest.mark.parametrize("N,K", [((3 << 22) + 3585, 10241), ((3 << 22) + 1, 16384), (3 << 22, 12000), ((3 << 22) + 7, 10240), ((3 << 22) + 7, 16385)])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_rows_in_wide_slices(N, K, shift):
    """From 3 * 2^22 vectors on 10241 to 16384 clusters are cut into slices of 4096; chunks of fp16 numbers, of bf16 numbers and of neither in turn, and four rows
    that decide how all others are read. The exact integer sums, in torch."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.randn(N, 4, device="cuda", generator=gen).mul_(0.02)
    kind = ((torch.arange(N, device="cuda") // 3584 + shift) % 3)[:, None]
    x = torch.where(kind == 0, x.half().float(), torch.where(kind == 1, x.bfloat16().float() * 2.0 ** -12, x))
    idx = torch.randint(0, K, (N,), device="cuda", generator=gen, dtype=torch.int32)
    prev, out = torch.zeros(K, 4, device="cuda"), torch.empty(K, 4, device="cuda")
    counts, ws = torch.empty(K, dtype=torch.uint32, device="cuda"), g.workspace(N, 4, K)
    print(f"wide slices N={N} K={K} shift={shift}", flush=True)
    cc.update(x, idx.view(torch.uint32), prev, out, counts, ws)
    e = cc.read_stats(ws).fixed_point_exp
    codes = idx.long()
    sums = torch.zeros(K, 4, dtype=torch.int64, device="cuda").index_add_(0, codes, torch.round(torch.ldexp(x.double(), torch.tensor(float(e), device="cuda"))).long())
    n = torch.bincount(codes, minlength=K)
    want = torch.ldexp(sums.double(), torch.tensor(float(-e), device="cuda")) / n.clamp(min=1)[:, None]
    assert torch.equal(counts.view(torch.int32).long(), n)
    assert torch.equal(out.cpu(), torch.where((n > 0)[:, None], want, prev.double()).float().cpu())


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("in_features,out_features,gl,K", [(1024, 16384, 16, 4096), (1024, 16400, 16, 4096), (2049, 8192, 16, 65536), (2048, 8192, 8, 4097), (2049, 8192, 8, 4097),
                                                           (2049, 8192, 8, 40960), (2049, 8192, 8, 40961), (2049, 8192, 8, 63489)])
def test_16_bit_gradients_on_either_side_of_2_24_numbers(dt, in_features, out_features, gl, K):
    """Rows of 8 and 16 go along up to 2^24 numbers, and at 8 with 21 to 31 slices; otherwise entries are left. Numbers whose sums are exact in fp32."""
    import paper_2503_13089_amd as cc

    gen = torch.Generator(device="cuda").manual_seed(out_features + K)
    n = L.num_codes(in_features, out_features, gl)
    G = torch.randint(-127, 128, (in_features, out_features), device="cuda", generator=gen).double().mul_(2.0 ** -18)
    idx = torch.randint(0, K, (n,), device="cuda", generator=gen)
    codes = idx.to(torch.int32).to(torch.int16).view(torch.uint16)
    out, ws = torch.full((K, gl), 3.0, device="cuda"), torch.empty(cc.workspace_bytes(max(n, K), gl, K), dtype=torch.uint8, device="cuda")
    print(f"gradient at 2^24 numbers {in_features}x{out_features} g={gl} K={K} {dt}", flush=True)
    cc.layer_codebook_grad(G.to(dt), codes, K, gl, out, ws)
    want = torch.zeros(K, gl, dtype=torch.float64, device="cuda").index_add_(0, idx, G.view(n, gl))
    assert torch.equal(out.cpu(), want.float().cpu())


@pytest.mark.parametrize("N,K,scale,least", [(300 * 3584 + 5, 8192, 0, 0), (300 * 3584, 5000, 0, 1e-9), (40000, 9000, 100, 0), (70001, 20000, -90, 0), (70001, 20000, -126, 0), (3_000_001, 65536, -20, 1e-13),
                                               (32768, 30000, 0, 0), (33000, 6000, 0, 1e-9), (99468, 10680, 0, 0), (150001, 33000, 0, 0), (250245, 4179, 0, 1e-9)])   # few steps to a wave
def test_terms_of_few_bits_and_others_side_by_side(N, K, scale, least):
    """bf16 numbers of ordinary range, whose terms have at most 30 bits above a common unit, `least`: with a few among them that have not, over the
    exponents where the scale of the sums meets its ends."""
    rng = np.random.default_rng(N + K)
    X = ((0.02 * rng.standard_normal((N, 4))).astype(np.float32).view(np.uint32) & 0xffff0000).view(np.float32)
    if least:
        some = rng.integers(0, N, 50)
        X[some, rng.integers(0, 4, 50)] = ((least * rng.standard_normal(50)).astype(np.float32).view(np.uint32) & 0xffff0000).view(np.float32)
    X = ((np.ldexp(X, scale)).astype(np.float32).view(np.uint32) & 0xffff0000).view(np.float32)
    idx = rng.integers(0, K, size=N).astype(np.uint32)
    prev = rng.standard_normal((K, 4)).astype(np.float32)
    print(f"few bits N={N} K={K} scale={scale} least={least}", flush=True)
    got, counts, stats = g.gpu_update(X, idx, prev)
    terms = np.rint(np.ldexp(X.astype(np.float64), stats.fixed_point_exp)).astype(np.int64)
    n = np.bincount(idx, minlength=K)
    order = np.argsort(idx, kind="stable")
    sums = np.zeros((K, 4), np.int64)
    sums[n > 0] = np.add.reduceat(terms[order], np.concatenate(([0], np.cumsum(n)))[:-1][n > 0], axis=0)
    want = np.where(n[:, None] > 0, np.ldexp(sums.astype(np.float64), -stats.fixed_point_exp) / np.maximum(n, 1)[:, None], prev)
    assert np.array_equal(counts, n) and got.tobytes() == want.astype(np.float32).tobytes()
