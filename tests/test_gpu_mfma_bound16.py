"""Pins what the E-step by cells at d = 8 assumes of v_mfma_f32_16x16x32_f16 (Section 3.1: the codes must be the true argmin), as
tests/test_gpu_mfma_bound.py does for the 32x32x16 instruction: the result of one instruction from zero, or of two chained
ones, is within 16 * 2^-24 * S of the exact sum, S as defined there.
"""
import numpy as np
import pytest

from tests import test_gpu_mfma_bound as bound

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ULPS_ASSUMED = 16.0


def run(A, B, C):
    import paper_2503_13089_amd as cc

    T = A.shape[0]
    D = torch.empty((T, 16, 16), dtype=torch.float32, device="cuda")
    cc.mfma_f16_probe16(torch.from_numpy(A.astype(np.float16)).cuda(), torch.from_numpy(B.astype(np.float16)).cuda(),
                        torch.from_numpy(C.astype(np.float32)).cuda(), D)
    torch.cuda.synchronize()
    return D.cpu().numpy().astype(np.float64)


def kernel_like(scale, sigma_log2, rng, tiles, two):
    """The kernel's layout: 24 slots for three fp16 parts of a centroid's eight components against -2 x, three for the norm
    against 2^8, 2^-3, 2^-14. two: inputs that are no fp16 numbers; what -2 x has beyond its fp16 part goes first, without the norm."""
    sigma = 2.0 ** sigma_log2
    x = (rng.standard_normal((tiles, 16, 8)) * scale).astype(np.float32).astype(np.float64)
    if not two:
        x = bound.f16(x)
    c = (x + rng.standard_normal(x.shape) * scale * 0.1).astype(np.float32).astype(np.float64)
    A, B, low = np.zeros((tiles, 16, 32)), np.zeros((tiles, 16, 32)), np.zeros((tiles, 16, 32))
    rest, hi = (c * sigma).astype(np.float32).astype(np.float64), bound.f16(-2.0 * x)
    for p in range(3):
        h = bound.f16(rest)
        A[:, :, 8 * p:8 * p + 8], B[:, :, 8 * p:8 * p + 8], low[:, :, 8 * p:8 * p + 8] = h, hi, bound.f16(-2.0 * x - hi)
        rest = rest - h
    norm = ((c ** 2).sum(-1) * sigma).astype(np.float32).astype(np.float64)
    for slot, m in ((24, 2.0 ** 8), (25, 2.0 ** -3), (26, 2.0 ** -14)):
        A[:, :, slot], B[:, :, slot] = bound.f16(norm / m), m
        norm = norm - A[:, :, slot] * m
    if two:
        A, B = np.concatenate([A, A], -1), np.concatenate([low, B], -1)
    return A, B, np.zeros((tiles, 16))


def cut(sets):
    """An operand set of 32 rows as twice as many tiles of 16."""
    A, B, C = sets
    T, _, S = A.shape
    return A.reshape(2 * T, 16, S), B.reshape(2 * T, 16, S), C.reshape(2 * T, 16)


def test_accumulation_of_the_16x16x32_instruction_stays_inside_the_assumed_bound():
    rng = np.random.default_rng(20250314)
    sets = []
    for two in (False, True):
        for scale in (1.0, 1e-1, 1e-2, 1e-3, 1e-4, 3e-5, 1e-5, 1e-6):
            for sl in (18, 13, 8, 3, -3):
                if scale * 2.0 ** sl > 8000.0 or 8 * (5 * scale) ** 2 * 2.0 ** sl > 2.0 ** 23:
                    continue  # the kernel never scales its centroids out of the fp16 range
                sets.append((f"kernel layout scale={scale:g} sigma=2^{sl} two={two}", kernel_like(scale, sl, rng, 16, two)))
    for S in (32, 64):
        sets.append((f"cancellation, {S} slots", cut(bound.cancellation(S, rng, 24))))
        sets.append((f"subnormal factors, {S} slots", cut(bound.subnormals(S, rng, 24))))
        for nz in (1, 2, 3, 7, 15, 16, 24, 27, 31, 32, 48, 64):
            if nz <= S:
                sets.append((f"wide exponents, {nz} of {S} slots", cut(bound.wide_exponents(S, rng, 8, nz))))
    worst, outputs = 0.0, 0
    for name, (A, B, C) in sets:
        print(name, flush=True)
        D = run(A, B, C)
        exact, W = bound.exact_and_weight(A, B, C)
        err = np.abs(D - exact)
        ratio = float((err / (bound.U * W + 1e-300)).max())
        worst, outputs = max(worst, ratio), outputs + D.size
        assert np.all(err <= ULPS_ASSUMED * bound.U * W), f"{name}: error {ratio:.2f} x 2^-24 x inflated sum of |terms|"
    print(f"{outputs} results, worst error = {worst:.2f} x 2^-24 x S (the kernel assumes {ULPS_ASSUMED:g})")
    assert worst <= 0.75 * ULPS_ASSUMED, "the margin on the assumed accumulation bound is nearly used up"


def test_probe_reproduces_exact_small_integer_products():
    rng = np.random.default_rng(3)
    for S in (32, 64):
        A = rng.integers(-8, 9, size=(4, 16, S)).astype(np.float64)
        B = rng.integers(-8, 9, size=(4, 16, S)).astype(np.float64)
        C = rng.integers(-100, 101, size=(4, 16)).astype(np.float64)
        assert np.array_equal(run(A, B, C), (A[:, :, None, :] * B[:, None, :, :]).sum(-1) + C[:, :, None])
