"""The kernel's own bound (csrc/match_bound.h, compiled here for the host) over
approximate distances formed as the correlation matcher forms them: each of the
K-1 nearest blocks (oracle keys) passes it, at every grid of candidate blocks."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2103_10765_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_10765_amd", "csrc")
F32 = np.float32
TILES = ((0, 0), (12, 36), (48, 60), (84, 84))

SOURCE = """
#include <cmath>
#include "match_bound.h"
// (a square root 10^-6 too small, as the kernel's may be)
extern "C" float bound(float half, float hn) {
  return gbm3d::widened_bound(half, hn, [](float x) { return std::sqrt(x) * 0.999999f; });
}
extern "C" float tie_step() { return gbm3d::kTieStep; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bound")
    (d / "bound.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "bound.cpp"), "-o", str(d / "bound.so")], check=True)
    L = ctypes.CDLL(str(d / "bound.so"))
    L.bound.restype = L.tie_step.restype = ctypes.c_float
    L.bound.argtypes = [ctypes.c_float, ctypes.c_float]
    return L


def _bf16(x, up=False):
    return ((np.asarray(x, F32).view(np.uint32) & 0xFFFF0000) | (0xFFFF if up else 0)).view(F32)


def _image(kind, n):
    rng = np.random.default_rng(11)
    y, x = np.mgrid[:n, :n]
    if kind == "noisy":
        return synth.make_case(n, n, 25 / 255, 3)[1]
    if kind == "smooth and far":   # high contrast without noise: the widening matters most
        return np.clip(32768 + 60000 * np.sin(x / 9.0) * np.cos(y / 13.0), 0, 65535).astype(np.uint16)
    if kind == "levels":
        return (np.where((x // 29 + y // 23) % 2, 65000, 300) + rng.integers(-40, 41, (n, n))).astype(np.uint16)
    if kind == "low noise":
        return np.clip(synth.clean_image(n, n, 3) * 65535 + rng.normal(0, 60, (n, n)), 0, 65535).astype(np.uint16)
    if kind == "rounding":
        # One reference of a tile lies alone (a dark ring around it) among cells of
        # two levels.  Halved and rounded to f16 the three are 16400 (for 16407.5),
        # 16912 (16904.5) and 15912 (15909.5): the second is the first's nearer
        # neighbour, 497 a pixel against 498, and looks the farther one, 512
        # against 488
        cells = rng.choice([33809, 31819], (n // 10 + 1, n // 10 + 1))
        z = np.kron(cells, np.ones((10, 10), np.int64))[:n, :n]
        for p0, q0 in TILES[:3]:
            z[np.ix_(np.arange(p0 - 7, p0 + 15) % n, np.arange(q0 + 2, q0 + 24) % n)] = 0
            z[p0:p0 + 8, q0 + 9:q0 + 17] = 32815
        return z.astype(np.uint16)
    return np.where(rng.random((n, n)) < 0.01, 65535, 777).astype(np.uint16)


def _approximate(img, R, p0, q0, step):
    """A tile's exact blocks and half distances (rows and columns of candidates)."""
    n, side = img.shape[0], 2 * R + 10
    reg = img[np.ix_(np.arange(p0 - R, p0 - R + side + 7) % n, np.arange(q0 - R, q0 - R + side + 7) % n)].astype(np.int64)
    exact = np.lib.stride_tricks.sliding_window_view(reg, (8, 8)).reshape(side, side, 64)
    a = ((reg - reg[R + 8, R + 8]) * F32(0.5)).astype(np.float16).astype(F32)
    a = np.lib.stride_tricks.sliding_window_view(a, (8, 8)).reshape(side, side, 64)
    cy, cx = np.mgrid[:side, :side]
    start = (F32(0.5) * (a * a).sum(-1, dtype=F32) + F32(step) * (cy * (2 * R + 1) + cx)).astype(F32)
    return exact, a, start, cy, cx


@pytest.mark.parametrize("kind", ["noisy", "smooth and far", "levels", "low noise", "dots", "rounding"])
@pytest.mark.parametrize("R,K", [(19, 16), (19, 32), (15, 32), (11, 16), (7, 32), (3, 16)])
def test_kernel_bound_keeps_the_nearest_blocks(lib, kind, R, K):
    n, S = 90, 2 * R + 1
    img = _image(kind, n)
    for p0, q0 in TILES:
        exact, a, start, cy, cx = _approximate(img, R, p0, q0, lib.tie_step())
        group = ((cy % 8) * 16 + cx % 16).ravel()
        for u in range(0, 4, 3):
            for v in range(4):
                y, x = R + 3 * u, R + 3 * v
                inside = (cy >= 3 * u) & (cy < 3 * u + S) & (cx >= 3 * v) & (cx < 3 * v + S)
                half = ((start + start[y, x]) - a @ a[y, x]).astype(F32)
                best = np.full(128, np.inf, F32)
                np.minimum.at(best, group, np.where(inside, _bf16(np.maximum(half, 0)), np.inf).ravel())
                kth = np.sort(best)[K - 1]
                bound = lib.bound(float(_bf16(kth, up=True)), float(start[y, x])) if np.isfinite(kth) else np.inf
                passes = inside & (_bf16(half) <= (_bf16(F32(bound)) if np.isfinite(bound) else np.inf))
                key = ((exact - exact[y, x]) ** 2).sum(-1) * 2048 + (cy - 3 * u) * S + (cx - 3 * v)
                key = np.where(inside, key, 1 << 60)
                key[y, x] = 1 << 60
                assert passes.ravel()[np.argsort(key, axis=None)[:K - 1]].all(), (p0, q0, u, v)


def test_position_term_is_below_a_unit_of_distance(lib):
    # half distances are whole multiples of 1/8; a candidate's and a reference's
    # terms are at most row 47, column 47 of a window of 39
    assert 0 < 2 * lib.tie_step() * (47 * 39 + 47) < 1 / 8
