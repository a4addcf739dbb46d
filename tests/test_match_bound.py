"""The correlation matcher's candidate bound on the CPU: with pixels rounded to
float16, half distances in float32 truncated to bfloat16 and the K-th smallest
of 128 group bests widened as the kernel widens it, every one of the K-1
nearest blocks (oracle keys) passes the bound, for every reference of a tile,
on noisy, smooth, tie-heavy and extreme images."""
import numpy as np
import pytest

from paper_2103_10765_amd import synth

R, S, SIDE = 19, 39, 48
F32 = np.float32


def _bf16(x, up=False):
    return ((np.asarray(x, F32).view(np.uint32) & 0xFFFF0000) | (0xFFFF if up else 0)).view(F32)


def _image(kind, n=96):
    rng = np.random.default_rng(5)
    y, x = np.mgrid[:n, :n]
    if kind == "noisy":
        return synth.make_case(n, n, 25 / 255, 3)[1]
    if kind == "smooth":
        return synth.to_u16(synth.clean_image(n, n, 3))
    if kind == "levels":
        return (np.where((x // 29 + y // 23) % 2, 65000, 9000) + rng.integers(-3, 4, (n, n))).astype(np.uint16)
    if kind == "constant":
        return np.full((n, n), 40000, np.uint16)
    if kind == "checkerboard":
        return ((x + y) % 2 * 65535).astype(np.uint16)
    return rng.choice(np.array([0, 65535], np.uint16), (n, n))


@pytest.mark.parametrize("K", [16, 32])
@pytest.mark.parametrize("kind", ["noisy", "smooth", "levels", "constant", "checkerboard", "extremes"])
def test_bound_keeps_the_nearest_blocks(kind, K):
    Z = _image(kind).astype(np.int64)
    cy, cx = np.mgrid[:SIDE, :SIDE]
    group = ((cy % 8) * 16 + cx % 16).ravel()
    term = (F32(2.0 ** -15) * (cy * S + cx)).astype(F32)
    for p0, q0 in ((0, 0), (12, 36), (60, 24), (84, 84)):
        reg = Z[np.ix_(np.arange(p0 - R, p0 - R + 55) % 96, np.arange(q0 - R, q0 - R + 55) % 96)]
        exact = np.lib.stride_tricks.sliding_window_view(reg, (8, 8)).reshape(SIDE, SIDE, 64)
        a = ((reg - reg[R + 8, R + 8]) * F32(0.5)).astype(np.float16).astype(F32)
        a = np.lib.stride_tricks.sliding_window_view(a, (8, 8)).reshape(SIDE, SIDE, 64)
        start = (F32(0.5) * (a * a).sum(-1, dtype=F32) + term).astype(F32)
        for u in range(4):
            for v in range(4):
                y, x = R + 3 * u, R + 3 * v
                inside = np.zeros((SIDE, SIDE), bool)
                inside[3 * u:3 * u + S, 3 * v:3 * v + S] = True
                half = ((start + start[y, x]) - a @ a[y, x]).astype(F32)
                best = np.full(128, np.inf, F32)
                np.minimum.at(best, group, np.where(inside, _bf16(np.maximum(half, 0)), np.inf).ravel())
                kth = _bf16(np.sort(best)[K - 1], up=True)
                nb, t = np.sqrt(F32(2) * start[y, x]) * F32(1.000002), np.sqrt(F32(2) * kth) * F32(1.000002)
                t2 = t + F32(1.01 / 2048) * (4 * nb + 2 * t)
                bound = _bf16(F32(0.500002) * t2 * t2 + F32(1 / 65536) * (nb + t2) ** 2)
                passes = inside & (_bf16(half) <= bound)
                key = ((exact - exact[y, x]) ** 2).sum(-1) * 2048 + (cy - 3 * u) * S + (cx - 3 * v)
                key = np.where(inside, key, 1 << 60)
                key[y, x] = 1 << 60
                nearest = np.argsort(key, axis=None)[:K - 1]
                assert passes.ravel()[nearest].all(), (p0, q0, u, v)
