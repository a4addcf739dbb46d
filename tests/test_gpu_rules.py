"""The rules that choose a kernel's shape do not choose a slow one: times of
the same work by two routes on one GPU, compared with each other (the smallest
of several runs; the margins are wider than such runs differ)."""
import numpy as np
import pytest

from paper_2103_10765_amd import synth

pytestmark = pytest.mark.gpu

SIG = 25.0 / 255.0


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2103_10765_amd import gbm3d
    return gbm3d


@pytest.fixture(scope="module")
def ctx(G):
    c = G.Context(0)
    yield c
    c.close()


def up(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def kernel_ms(ctx, kernel, run):
    run()
    best = float("inf")
    ctx.timing(True)
    try:
        for _ in range(8):
            ctx.timing_reset()
            run()
            run()
            ms, n = ctx.timing_read(kernel)
            best = min(best, ms / n)
    finally:
        ctx.timing(False)
    return best


@pytest.mark.parametrize("S", [21, 39])
@pytest.mark.parametrize("n", [192, 320, 384, 416, 448, 480])
def test_group_tiles_of_a_single_image(G, ctx, n, S):
    """A batch's group launches take the largest reference tiles whatever the
    number of tiles; a single image's tiles are chosen by that number and are
    never much slower."""
    x = up(synth.make_case(n, n, SIG, 3)[1])
    pilot = up(synth.make_case(n, n, SIG / 12, 3)[1])
    for K in (2, 8, 16, 32):
        p = G.default_params(search=S, k_ht=K, k_wiener=K)
        for kernel, one, batch in (
                ("group_ht", lambda: ctx.basic(x, SIG, p),
                 lambda: ctx.denoise_batch([x], [SIG], params=p, basic_only=True)),
                ("group_wiener", lambda: ctx.wiener(x, pilot, SIG, p),
                 lambda: ctx.denoise_batch([x], [SIG], pilots=[pilot], params=p))):
            a, b = kernel_ms(ctx, kernel, one), kernel_ms(ctx, kernel, batch)
            print(kernel, n, S, K, f"{1e3 * a:.1f} us, largest tiles {1e3 * b:.1f} us", flush=True)
            assert a <= 1.2 * b, (kernel, n, S, K, a, b)


@pytest.mark.parametrize("K", [2, 8])
def test_small_windows_cost_less(G, ctx, K):
    """Matching 1024 x 1024: windows of 3, 7, 11 and 15 take at most a given
    part of the default window's time (which has 169, 31, 12 and 7 times their
    candidates)."""
    x = up(synth.make_case(1024, 1024, SIG, 3)[1])
    t = {S: kernel_ms(ctx, "bm", lambda: ctx.match(x, K, G.default_params(search=S))) for S in (3, 7, 11, 15, 39)}
    print("matching 1024^2", K, {S: round(1e3 * v, 1) for S, v in t.items()}, flush=True)
    for S, part in ((3, 0.25), (7, 0.5), (11, 0.65), (15, 0.65)):
        assert t[S] <= part * t[39], (S, t)


def _image(kind, n):
    rng = np.random.default_rng(5)
    y, x = np.mgrid[:n, :n]
    if kind == "levels":
        return (np.where((x // 29 + y // 23) % 2, 60000, 4000) + rng.integers(-3, 4, (n, n))).astype(np.uint16)
    if kind == "checkerboard":
        return ((x + y) % 2 * 65535).astype(np.uint16)
    if kind == "stripes":
        return (x // 3 % 2 * 65535).astype(np.uint16)
    return np.tile(rng.integers(0, 65536, (8, 8)), (n // 8, n // 8)).astype(np.uint16)


@pytest.mark.parametrize("K", [16, 32])
def test_matching_time_hardly_depends_on_the_image(G, ctx, K):
    """Flat levels and periodic textures, where hundreds of candidates come near
    the K-th best, take at most 3.2 times a noisy image's time."""
    t = {}
    for kind in ("noisy", "levels", "checkerboard", "stripes", "period 8"):
        x = up(synth.make_case(512, 512, SIG, 3)[1] if kind == "noisy" else _image(kind, 512))
        t[kind] = kernel_ms(ctx, "bm", lambda: ctx.match(x, K))
    print("matching 512^2", K, {k: round(1e3 * v, 1) for k, v in t.items()}, flush=True)
    assert max(t.values()) <= 3.2 * t["noisy"], t


def test_one_long_list_does_not_slow_a_first_estimate(G, ctx):
    """First estimates of 128 x 128 images: in some a tile or two have one
    reference with 450 to 480 near candidates in some 1000.  They cost about
    what the others do."""
    def ms(sigma, seed):
        x = up(synth.make_case(128, 128, sigma / 255, seed)[1])
        q = ctx.quantize(ctx.basic(x, sigma / 255))
        return kernel_ms(ctx, "bm", lambda: ctx.match(q, 32))
    plain = max(ms(25, seed) for seed in (18, 22))
    t = {c: ms(*c) for c in ((25, 20), (25, 24), (50, 16), (50, 20))}
    print("matching first estimates", round(1e3 * plain, 1), {c: round(1e3 * v, 1) for c, v in t.items()}, flush=True)
    assert max(t.values()) <= 1.25 * plain, (plain, t)


def test_autotuner_compares_whole_stages(G):
    """512 x 512, window 11, K = 16: matching alone is a little faster shift-wise
    (1), matching with the stage's stacks by the correlation kernel (2), whose
    launch writes them too."""
    c = G.Context(0)
    try:
        x = up(synth.make_case(512, 512, SIG, 3)[1])
        p = G.default_params(search=11)
        assert c.autotune(x, 16, reps=50, params=p)[0] == 2
        # a group size of no stage: matching alone
        assert c.autotune(x, 8, reps=2, params=p)[0] in (1, 2)
    finally:
        c.close()
