"""GPU parity: the HIP path through the C ABI against the fp64 CPU oracle on
the same seeded inputs.

Bars: match indices bit-exact (exact integer distances, lower-rank tie rule);
filtered outputs within max-abs 2e-4 on the [0, 1] scale and PSNR within
0.01 dB.  For stage 1, pixels covered by a group holding a hard-threshold
decision within 1e-5 (relative) of tau are excluded from the max-abs check,
because float32 coefficients may decide those differently; such groups must
be rare.  Full-size images are checked on sampled references and windows the
oracle evaluates exactly.
"""
import sys

import numpy as np
import pytest

from oracle import gbm3d_oracle as O
from paper_2103_10765_amd import synth

pytestmark = pytest.mark.gpu

SIG = 25.0 / 255.0
MAXABS = 2e-4
PSNR_TOL = 0.01


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    return t


@pytest.fixture(scope="module")
def G(torch):
    from paper_2103_10765_amd import gbm3d
    return gbm3d


@pytest.fixture(scope="module")
def ctx(G):
    c = G.Context(0)
    yield c
    c.close()


def up(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def oparams(G, gp):
    return O.DEFAULT.with_(search=gp.search, k_ht=gp.k_ht, k_wiener=gp.k_wiener, ht_a=gp.ht_a, ht_b=gp.ht_b)


# ---------------------------------------------------------------------------
# patch stacks
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("shape", [(40, 45), (67, 200), (9, 130)])
def test_stack_parity(torch, G, ctx, kind, shape):
    H, W = shape
    say("stack", kind, shape)
    _, Z = synth.make_case(H, W, SIG, 31)
    S = ctx.stack(up(torch, Z), kind).cpu().numpy().reshape(H, W, 8, 8)
    z = Z.astype(np.float64) / 65535.0
    ys, xs = np.meshgrid(np.arange(H), np.arange(W), indexing="ij")
    P = O._blocks(z, ys.ravel(), xs.ravel(), 8)
    ref = O.bior2d_forward(P) if kind == 0 else O.dct2d_forward(P)
    err = np.abs(S.reshape(-1, 8, 8) - ref).max()
    assert err < 1e-5, err


# ---------------------------------------------------------------------------
# block matching
# ---------------------------------------------------------------------------

MATCH_CASES = [
    # (H, W, search, K, seed)
    (39, 39, 39, 16, 1),
    (48, 51, 15, 8, 2),
    (128, 128, 39, 16, 3),
    (128, 128, 39, 32, 4),
    (100, 131, 21, 4, 5),
    (67, 190, 39, 32, 6),
    (45, 400, 9, 2, 7),
]


METHODS = [1, 2]   # shift-wise, correlation (matrix cores)


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("H,W,S,K,seed", MATCH_CASES)
def test_match_bit_exact(torch, G, ctx, H, W, S, K, seed, method):
    say("match", H, W, S, K, "method", method)
    _, Z = synth.make_case(H, W, SIG, seed)
    p = G.default_params(search=S, bm_method=method)
    got = ctx.match(up(torch, Z), K, p).cpu().numpy().astype(np.int64)
    exp = O.match(Z, K, O.DEFAULT.with_(search=S))
    bad = np.nonzero((got != exp).any(axis=1))[0]
    assert bad.size == 0, (bad[:5], got[bad[:2]], exp[bad[:2]])


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("kind", ["flat", "lowbits", "periodic", "extremes"])
def test_match_ties(torch, G, ctx, kind, method):
    H, W, S, K = 60, 70, 15, 16
    say("match ties", kind, "method", method)
    rng = np.random.default_rng(40)
    if kind == "flat":
        Z = np.full((H, W), 777, dtype=np.uint16)
    elif kind == "lowbits":
        Z = rng.integers(0, 3, size=(H, W)).astype(np.uint16)
    elif kind == "periodic":
        Z = np.tile(rng.integers(0, 65536, size=(5, 7)), (12, 10))[:H, :W].astype(np.uint16)
    else:
        Z = (rng.integers(0, 2, size=(H, W)) * 65535).astype(np.uint16)
    p = G.default_params(search=S, bm_method=method)
    got = ctx.match(up(torch, Z), K, p).cpu().numpy().astype(np.int64)
    exp = O.match(Z, K, O.DEFAULT.with_(search=S))
    assert np.array_equal(got, exp)


@pytest.mark.parametrize("method", METHODS)
def test_match_full_size_sampled(torch, G, ctx, method):
    """512 x 512, search 39, K = 16 and 32: 400 sampled references."""
    _, Z = synth.single_image_case(512, SIG, 2)
    ids = np.random.default_rng(0).choice(O.n_refs(512, 512, 3), 400, replace=False)
    for K in (16, 32):
        say("match 512 sampled K", K, "method", method)
        got = ctx.match(up(torch, Z), K, method=method).cpu().numpy().astype(np.int64)[ids]
        exp = O.match(Z, K, O.DEFAULT, ref_ids=ids)
        assert np.array_equal(got, exp)


@pytest.mark.parametrize("method", METHODS)
def test_match_max_width_sampled(torch, G, ctx, method):
    """The widest supported image (W = 32768), 40 rows; sampled references."""
    H, W = 40, 32768
    say("match max width", "method", method)
    _, Z = synth.make_case(H, W, SIG, 8)
    ids = np.random.default_rng(1).choice(O.n_refs(H, W, 3), 200, replace=False)
    got = ctx.match(up(torch, Z), 16, method=method).cpu().numpy().astype(np.int64)[ids]
    exp = O.match(Z, 16, O.DEFAULT, ref_ids=ids)
    assert np.array_equal(got, exp)


# ---------------------------------------------------------------------------
# stage 1
# ---------------------------------------------------------------------------

FLAG_MAXABS = 5e-3   # bound on pixels near a flipped hard-threshold decision
# Near-threshold groups: at most 1e-3 of the groups, with a floor of 3 groups
# for the small images here (the oracle on these inputs gives 0 in most cases,
# 3 of 1408 groups at 96 x 130, sigma 15/255, and 1 of 288 with K = 32), and at
# most 12% of the checked pixels covered by them (measured at most 10.4%).
FLAG_GROUP_FLOOR = 3
FLAG_GROUP_FRAC = 1e-3
FLAG_PIXEL_FRAC = 0.12


def _check_stage1(Yg, Yo, idx, margin, p, clean=None, ref_ids=None, window=None):
    """max-abs <= 2e-4 off the pixels of near-threshold groups; those pixels
    within 5e-3 (one flipped coefficient of size ~tau spread over ~100
    overlapping blocks); near-threshold groups rare; PSNR within 0.01 dB."""
    H, W = Yg.shape
    flag = O.flagged_pixels(H, W, idx, margin, p, ref_ids=ref_ids)
    n_flag_groups = int((margin < 1e-5).sum())
    if window is not None:
        rows, cols = window
        Yg, Yo, flag = Yg[np.ix_(rows, cols)], Yo[np.ix_(rows, cols)], flag[np.ix_(rows, cols)]
        if clean is not None:
            clean = clean[np.ix_(rows, cols)]
    say(f"  near-threshold groups {n_flag_groups} of {len(margin)}, flagged pixels {flag.mean():.4f}")
    assert n_flag_groups <= max(FLAG_GROUP_FLOOR, FLAG_GROUP_FRAC * len(margin)), n_flag_groups
    assert flag.mean() <= FLAG_PIXEL_FRAC, flag.mean()
    err = np.abs(Yg - Yo)
    assert err[~flag].max() <= MAXABS, (err[~flag].max(), n_flag_groups)
    if flag.any():
        assert err[flag].max() <= FLAG_MAXABS, err[flag].max()
    if clean is not None:
        d = abs(O.psnr(Yg, clean) - O.psnr(Yo, clean))
        assert d <= PSNR_TOL, d
    return n_flag_groups


@pytest.mark.parametrize("H,W,S,sigma,seed", [(128, 128, 39, 25 / 255, 1), (96, 130, 21, 15 / 255, 9),
                                              (64, 64, 39, 50 / 255, 10), (39, 41, 39, 25 / 255, 11)])
def test_basic_parity(torch, G, ctx, H, W, S, sigma, seed):
    say("basic", H, W, S, sigma)
    clean, Z = synth.make_case(H, W, sigma, seed)
    gp = G.default_params(search=S)
    p = oparams(G, gp)
    Yg = ctx.basic(up(torch, Z), sigma, gp).cpu().numpy().astype(np.float64)
    Yo, (idx, margin, _, _) = O.basic_estimate(Z, sigma, p, return_parts=True)
    _check_stage1(Yg, Yo, idx, margin, p, clean)


@pytest.mark.parametrize("H,W,S,seed,k_ht", [(128, 128, 39, 1, 16), (96, 130, 21, 9, 16), (39, 41, 39, 11, 16),
                                              (70, 77, 21, 20, 2), (64, 90, 15, 21, 8), (81, 64, 39, 22, 32)])
def test_basic_recompute_equals_stack(torch, G, ctx, H, W, S, seed, k_ht):
    """Stage 1 with each matched block's spectrum computed inside the group
    kernel from its pixels equals the stack path bit for bit (the same
    separable passes in the same order), and so do both stages; against the
    oracle as any stage-1 result.  Every group size's launch shape (chunks of
    K blocks for K <= 8, of 16 for K = 32)."""
    say("basic recompute", H, W, S, "k_ht", k_ht)
    clean, Z = synth.make_case(H, W, SIG, seed)
    Zt = up(torch, Z)
    gp = G.default_params(search=S, k_ht=k_ht)
    gr = G.default_params(search=S, k_ht=k_ht, ht_source=G.HT_RECOMPUTE)
    a = ctx.basic(Zt, SIG, gp).cpu().numpy()
    b = ctx.basic(Zt, SIG, gr).cpu().numpy()
    assert np.array_equal(a, b)
    assert np.array_equal(ctx.denoise(Zt, SIG, gp).cpu().numpy(), ctx.denoise(Zt, SIG, gr).cpu().numpy())
    p = oparams(G, gp)
    Yo, (idx, margin, _, _) = O.basic_estimate(Z, SIG, p, return_parts=True)
    _check_stage1(b.astype(np.float64), Yo, idx, margin, p, clean)


def test_recompute_refused_for_batches(torch, G, ctx):
    _, Z = synth.make_case(64, 64, SIG, 12)
    with pytest.raises(G.GBM3DError):
        ctx.denoise_batch([up(torch, Z)], [SIG], params=G.default_params(ht_source=G.HT_RECOMPUTE))
    with pytest.raises(G.GBM3DError):
        ctx.basic(up(torch, Z), SIG, G.default_params(ht_source=7))


@pytest.mark.parametrize("weight", [1, 2])
def test_basic_weight_variants(torch, G, ctx, weight):
    H, W = 60, 66
    clean, Z = synth.make_case(H, W, SIG, 12)
    gp = G.default_params(search=15, ht_weight=weight)
    p = oparams(G, gp).with_(ht_weight={1: "nnz", 2: "unit"}[weight])
    Yg = ctx.basic(up(torch, Z), SIG, gp).cpu().numpy().astype(np.float64)
    Yo, (idx, margin, _, _) = O.basic_estimate(Z, SIG, p, return_parts=True)
    _check_stage1(Yg, Yo, idx, margin, p, clean)


@pytest.mark.parametrize("k_ht,k_wiener", [(2, 4), (8, 8), (32, 16)])
def test_group_sizes_parity(torch, G, ctx, k_ht, k_wiener):
    """Both stages at the other group sizes (32 stage-1 blocks go through the
    transform scratch in two passes; small groups keep the next group's
    spectra in flight)."""
    H, W, S = 52, 47, 15
    say("group sizes", k_ht, k_wiener)
    clean, Z = synth.make_case(H, W, SIG, 16)
    gp = G.default_params(search=S, k_ht=k_ht, k_wiener=k_wiener)
    p = oparams(G, gp)
    Yg = ctx.basic(up(torch, Z), SIG, gp).cpu().numpy().astype(np.float64)
    Yo, (idx, margin, _, _) = O.basic_estimate(Z, SIG, p, return_parts=True)
    _check_stage1(Yg, Yo, idx, margin, p, clean)
    pilot = O.quantize(Yo)
    Yw = ctx.wiener(up(torch, Z), up(torch, pilot), SIG, gp).cpu().numpy().astype(np.float64)
    Ywo = O.wiener_estimate(Z, pilot, SIG, p)
    assert np.abs(Yw - Ywo).max() <= MAXABS


def test_basic_zero_threshold_identity(torch, G, ctx):
    _, Z = synth.make_case(70, 80, SIG, 13)
    gp = G.default_params(search=21, ht_a=0.0, ht_b=0.0)
    Yg = ctx.basic(up(torch, Z), SIG, gp).cpu().numpy()
    assert np.abs(Yg - Z / 65535.0).max() < 1e-5


def test_basic_constant_image(torch, G, ctx):
    Z = np.full((50, 61), 40000, dtype=np.uint16)
    Yg = ctx.basic(up(torch, Z), SIG).cpu().numpy()
    Yw = ctx.wiener(up(torch, Z), up(torch, Z), SIG).cpu().numpy()
    assert np.abs(Yg - 40000 / 65535.0).max() < 2e-6
    assert np.abs(Yw - 40000 / 65535.0).max() < 2e-6


def _windows(H, W, h, w):
    # interior, top-left corner (wraps) and bottom-right corner (wraps)
    return [(H // 2 - h // 2, W // 3, h, w), (H - h // 2, W - w // 2, h, w), (5, W - 7, h, w)]


def test_basic_full_size_windows(torch, G, ctx):
    """512 x 512 at sigma 25/255: three 24 x 24 windows evaluated exactly by the oracle."""
    clean, Z = synth.single_image_case(512, SIG, 2)
    Yg = ctx.basic(up(torch, Z), SIG).cpu().numpy().astype(np.float64)
    p = O.DEFAULT
    for (y0, x0, h, w) in _windows(512, 512, 24, 24):
        say("basic 512 window", y0, x0)
        ids = O.refs_for_window(512, 512, p, y0, x0, h, w)
        Yo, (idx, margin, _, _) = O.basic_estimate(Z, SIG, p, ref_ids=ids, return_parts=True)
        rows, cols = (y0 + np.arange(h)) % 512, (x0 + np.arange(w)) % 512
        _check_stage1(Yg, Yo, idx, margin, p, ref_ids=ids, window=(rows, cols))


# ---------------------------------------------------------------------------
# stage 2 (pilot given as an input)
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("H,W,S,sigma,seed", [(128, 128, 39, 25 / 255, 1), (80, 99, 15, 50 / 255, 14),
                                              (39, 39, 39, 15 / 255, 15)])
def test_wiener_parity(torch, G, ctx, H, W, S, sigma, seed):
    say("wiener", H, W, S, sigma)
    clean, Z = synth.make_case(H, W, sigma, seed)
    gp = G.default_params(search=S)
    p = oparams(G, gp)
    pilot = O.quantize(O.basic_estimate(Z, sigma, p))          # the oracle's own pilot
    Yg = ctx.wiener(up(torch, Z), up(torch, pilot), sigma, gp).cpu().numpy().astype(np.float64)
    Yo = O.wiener_estimate(Z, pilot, sigma, p)
    assert np.abs(Yg - Yo).max() <= MAXABS
    assert abs(O.psnr(Yg, clean) - O.psnr(Yo, clean)) <= PSNR_TOL


@pytest.mark.parametrize("k", [2, 4, 8, 16, 32])
@pytest.mark.parametrize("H,W,S", [(22, 25, 15), (24, 21, 7), (46, 49, 39)])
def test_wiener_group_sizes_at_tile_edges(torch, G, ctx, k, H, W, S):
    """Stage 2 at every group size, on images of eight references a side and of
    one more (a tile that is full, or holds a single row or column of groups),
    with windows of a fraction and of the whole footprint; the sums are rounded
    to 2^-40 and the transforms are float32, far inside MAXABS."""
    say("wiener group sizes", k, H, W, S)
    _, Z = synth.make_case(H, W, SIG, 19)
    gp = G.default_params(search=S, k_wiener=k)
    pilot = O.quantize(synth.make_case(H, W, SIG / 5, 19)[1] / 65535.0)
    Yg = ctx.wiener(up(torch, Z), up(torch, pilot), SIG, gp).cpu().numpy().astype(np.float64)
    assert np.abs(Yg - O.wiener_estimate(Z, pilot, SIG, oparams(G, gp))).max() <= MAXABS


def test_wiener_full_size_windows(torch, G, ctx):
    """512 x 512: pilot = the clean image quantised (an input both sides take)."""
    clean, Z = synth.single_image_case(512, SIG, 2)
    pilot = synth.to_u16(clean)
    Yg = ctx.wiener(up(torch, Z), up(torch, pilot), SIG).cpu().numpy().astype(np.float64)
    for (y0, x0, h, w) in _windows(512, 512, 20, 20):
        say("wiener 512 window", y0, x0)
        ids = O.refs_for_window(512, 512, O.DEFAULT, y0, x0, h, w)
        Yo = O.wiener_estimate(Z, pilot, SIG, O.DEFAULT, ref_ids=ids)
        rows, cols = (y0 + np.arange(h)) % 512, (x0 + np.arange(w)) % 512
        assert np.abs(Yg[np.ix_(rows, cols)] - Yo[np.ix_(rows, cols)]).max() <= MAXABS


# ---------------------------------------------------------------------------
# both stages, quantisation
# ---------------------------------------------------------------------------

def test_denoise_end_to_end(torch, G, ctx):
    say("denoise 128")
    clean, Z = synth.make_case(128, 128, SIG, 1)
    Zt = up(torch, Z)
    basic = torch.empty((128, 128), dtype=torch.float32, device="cuda")
    q = torch.empty((128, 128), dtype=torch.uint16, device="cuda")
    Yg = ctx.denoise(Zt, SIG, basic_out=basic, q_out=q).cpu().numpy().astype(np.float64)
    Y, Yb, Q = O.denoise(Z, SIG)
    assert abs(O.psnr(Yg, clean) - O.psnr(Y, clean)) <= PSNR_TOL
    # the intermediate outputs are the stage-1 call's and its quantisation
    b2 = ctx.basic(Zt, SIG).cpu().numpy()
    assert np.array_equal(basic.cpu().numpy(), b2)
    assert np.array_equal(q.cpu().numpy(), O.quantize(basic.cpu().numpy().astype(np.float64)))
    # stage 2 from the GPU's own pilot is the Wiener call with that pilot, bit for bit
    Yw = ctx.wiener(Zt, q, SIG).cpu().numpy()
    assert np.array_equal(Yw, Yg.astype(np.float32))
    # the two stages improve on each other
    assert O.psnr(Yg, clean) > O.psnr(basic.cpu().numpy(), clean) > O.psnr(Z / 65535.0, clean)


def test_quantize_bit_exact(torch, G, ctx):
    rng = np.random.default_rng(50)
    k = rng.integers(0, 65536, size=4000)
    x = np.concatenate([(k + 0.5) / 65535.0, k / 65535.0, rng.uniform(-0.5, 1.5, 4000),
                        [np.nan, -0.0, 0.0, 1.0, np.inf, -np.inf]]).astype(np.float32)
    got = ctx.quantize(up(torch, x)).cpu().numpy()
    exp = O.quantize(x.astype(np.float64))
    exp[np.isinf(x) & (x > 0)] = 65535
    assert np.array_equal(got, exp)


def test_invalid_arguments_launch_nothing(torch, G, ctx):
    Z = up(torch, np.zeros((64, 64), dtype=np.uint16))
    out = torch.full((64, 64), -7.0, device="cuda")
    for kw, sigma in [(dict(search=40), SIG), (dict(k_ht=3), SIG), ({}, 0.0), (dict(step=2), SIG)]:
        with pytest.raises(G.GBM3DError) as e:
            ctx.basic(Z, sigma, G.default_params(**kw), out=out)
        assert e.value.status in (G.EINVAL, G.EUNSUPPORTED)
    torch.cuda.synchronize()
    assert (out == -7.0).all()
    small = up(torch, np.zeros((20, 64), dtype=np.uint16))
    with pytest.raises(G.GBM3DError):
        ctx.match(small, 16)


def test_side_stream_and_repeat(torch, G, ctx):
    """Aggregation sums are 64-bit fixed point, so repeated runs (any stream,
    any wave interleaving) are bit-identical."""
    _, Z = synth.make_case(100, 100, SIG, 16)
    Zt = up(torch, Z)
    a = ctx.denoise(Zt, SIG).cpu().numpy()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b = ctx.denoise(Zt, SIG, stream=s)
    s.synchronize()
    torch.cuda.synchronize()
    assert np.array_equal(a, b.cpu().numpy())
    for _ in range(3):
        assert np.array_equal(a, ctx.denoise(Zt, SIG).cpu().numpy())


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("split", [1, 2, 4])
def test_match_workgroup_shapes_agree(torch, G, ctx, split, method):
    """Every workgroup shape of both matching kernels gives the oracle's indices."""
    say("match workgroup shape", split, "method", method)
    _, Z = synth.make_case(90, 200, SIG, 17)
    for K in (16, 32):
        exp = O.match(Z, K, O.DEFAULT.with_(search=21))
        got = ctx.match(up(torch, Z), K, G.default_params(search=21), split=split,
                        method=method).cpu().numpy().astype(np.int64)
        assert np.array_equal(got, exp)


def test_methods_give_identical_denoising(torch, G, ctx):
    """Same indices, so both stages give bit-identical outputs with either
    matching kernel (single image and batch)."""
    say("denoise shift vs corr")
    clean, Z = synth.make_case(200, 230, SIG, 18)
    Zt = up(torch, Z)
    a = ctx.denoise(Zt, SIG, G.default_params(bm_method=1)).cpu().numpy()
    b = ctx.denoise(Zt, SIG, G.default_params(bm_method=2)).cpu().numpy()
    assert np.array_equal(a, b)
    imgs, sig = _batch_inputs(torch, 4, 39, 140, 720)
    ra = [o.cpu().numpy() for o in ctx.denoise_batch(imgs, sig, params=G.default_params(bm_method=1))]
    rb = [o.cpu().numpy() for o in ctx.denoise_batch(imgs, sig, params=G.default_params(bm_method=2), graph=True)]
    torch.cuda.synchronize()
    for x, y in zip(ra, rb):
        assert np.array_equal(x, y)


def test_autotune_records_and_reloads(torch, G, ctx, tmp_path):
    """The autotuner times every matching variant (and, for K = k_ht, both
    stage-1 group-kernel shapes), keyed by (K, search, shape class); its
    choices are then used for auto params (same indices, same estimate), and
    survive a save / load."""
    say("autotune")
    _, Z = synth.make_case(150, 160, SIG, 19)
    Zt = up(torch, Z)
    m, sp, ms = ctx.autotune(Zt, 16, reps=2)
    assert m in (1, 2) and sp in (1, 2, 4) and ms > 0
    p21 = G.default_params(search=21)
    m21, sp21, _ = ctx.autotune(Zt, 16, reps=2, params=p21)
    exp = O.match(Z, 16, O.DEFAULT)
    assert np.array_equal(ctx.match(Zt, 16).cpu().numpy().astype(np.int64), exp)
    assert np.array_equal(ctx.match(Zt, 16, p21).cpu().numpy().astype(np.int64),
                          O.match(Z, 16, O.DEFAULT.with_(search=21)))
    path = str(tmp_path / "tune.txt")
    ctx.tune_save(path)
    rows = [ln.split() for ln in open(path).read().splitlines()]
    bm = {int(r[2]): r for r in rows if r[0] == "bm"}
    ht = {int(r[2]): r for r in rows if r[0] == "ht"}
    assert [int(x) for x in bm[39][4:6]] == [m, sp] and [int(x) for x in bm[21][4:6]] == [m21, sp21]
    assert set(ht) == {21, 39} and all(int(r[4]) in (0, 1) for r in ht.values())
    cls = int(ht[39][3])
    c2 = G.Context(0)
    try:
        c2.tune_load(path)
        assert np.array_equal(c2.match(Zt, 16).cpu().numpy().astype(np.int64), exp)
        # both stage-1 shapes give the same estimate, bit for bit
        outs = []
        for shape in (0, 1):
            f = tmp_path / f"shape{shape}.txt"
            f.write_text(f"ht 16 39 {cls} {shape} 0.1\n")
            c2.tune_load(str(f))
            outs.append(c2.basic(Zt, SIG).cpu().numpy())
        assert np.array_equal(outs[0], outs[1])
        bad = tmp_path / "bad.txt"
        bad.write_text("bm 16 39 5 9 1 0.1\n")
        with pytest.raises(G.GBM3DError):
            c2.tune_load(str(bad))
        with pytest.raises(G.GBM3DError):
            ctx.autotune(Zt, 16, reps=0)
    finally:
        c2.close()


# ---------------------------------------------------------------------------
# batches (persistent launches over per-image work lists, hipGraph replay)
# ---------------------------------------------------------------------------

def _batch_inputs(torch, n, lo, hi, seed):
    rng = np.random.default_rng(seed)
    imgs, sig = [], []
    for i in range(n):
        H, W = int(rng.integers(lo, hi + 1)), int(rng.integers(lo, hi + 1))
        s = float(rng.uniform(10, 50) / 255)
        _, Z = synth.make_case(H, W, s, seed + 1 + i)
        imgs.append(up(torch, Z))
        sig.append(s)
    return imgs, sig


def test_batch_equals_single_calls(torch, G, ctx):
    """Uneven sizes (incl. ragged and minimum), mixed pilots: every batch output
    equals the single-image call bit for bit."""
    say("batch vs single")
    imgs, sig = _batch_inputs(torch, 7, 39, 150, 700)
    pil = [None, None, up(torch, synth.to_u16(np.random.default_rng(1).random(tuple(imgs[2].shape)))), None,
           None, None, None]
    outs = ctx.denoise_batch(imgs, sig, pilots=pil)
    torch.cuda.synchronize()
    for i, (x, s, pl) in enumerate(zip(imgs, sig, pil)):
        ref = ctx.denoise(x, s) if pl is None else ctx.wiener(x, pl, s)
        assert np.array_equal(outs[i].cpu().numpy(), ref.cpu().numpy()), i
    basic = ctx.denoise_batch(imgs[:3], sig[:3], basic_only=True)
    for i in range(3):
        assert np.array_equal(basic[i].cpu().numpy(), ctx.basic(imgs[i], sig[i]).cpu().numpy())


@pytest.mark.parametrize("k", [2, 4, 8, 16, 32])
@pytest.mark.parametrize("H,W", [(24, 25), (190, 196), (200, 211)])
def test_single_image_tiles_equal_batch_tiles(torch, G, ctx, k, H, W):
    """A single image's group launches take smaller reference tiles than a
    batch's where the image has few; the sums are integers, so both give the
    same bits (sizes on both sides of a rule's line and at ragged tile edges)."""
    say("tile shapes", k, H, W)
    gp = G.default_params(search=15, k_ht=k, k_wiener=k)
    x = up(torch, synth.make_case(H, W, SIG, 23)[1])
    assert torch.equal(ctx.denoise_batch([x], [SIG], params=gp)[0], ctx.denoise(x, SIG, gp))


@pytest.mark.parametrize("S", [15, 31, 39])
def test_stacks_beside_matching_equal_separate_launches(torch, G, ctx, S):
    """The matching launches write the stacks too, in workgroups of two stack
    items spread among the tiles (odd counts of items, images narrower and
    shorter than an item); while launches are timed each kernel runs by itself.
    Same bits, for every shape of the matcher's candidate grid, single and
    batched."""
    gp = G.default_params(search=S)
    xs = [up(torch, synth.make_case(H, W, SIG, 29 + H)[1]) for H, W in [(39, 40), (45, 131), (201, 77)]]
    runs = []
    try:
        for timed in (False, True):
            say("stacks beside matching", S, "timed" if timed else "together")
            ctx.timing(timed)
            runs.append([ctx.denoise(x, SIG, gp) for x in xs] + ctx.denoise_batch(xs, [SIG] * 3, params=gp))
            torch.cuda.synchronize()
    finally:
        ctx.timing(False)
    for a, b in zip(*runs):
        assert torch.equal(a, b)


def test_batch_many_small_images_equal_single_calls(torch, G, ctx):
    """Many images of 39..64 px (several images share each 64-item block of
    every phase's item -> image table) around two larger ones, some with a
    pilot (no stage-1 items, also as the first and the last image): every
    batch output equals the single-image call bit for bit, eager and under
    graph replay."""
    say("batch many small")
    imgs, sig = _batch_inputs(torch, 46, 39, 64, 1300)
    big, bsig = _batch_inputs(torch, 2, 200, 260, 1400)
    imgs = imgs[:20] + big[:1] + imgs[20:] + big[1:]
    sig = sig[:20] + bsig[:1] + sig[20:] + bsig[1:]
    rng = np.random.default_rng(1500)
    pil = [None] * len(imgs)
    for i in (0, 7, 8, 30, len(imgs) - 1):
        pil[i] = up(torch, synth.to_u16(rng.random(tuple(imgs[i].shape))))
    refs = [(ctx.denoise(x, s) if pl is None else ctx.wiener(x, pl, s)).cpu().numpy()
            for x, s, pl in zip(imgs, sig, pil)]
    outs = ctx.denoise_batch(imgs, sig, pilots=pil)
    torch.cuda.synchronize()
    for i in range(len(imgs)):
        assert np.array_equal(outs[i].cpu().numpy(), refs[i]), i
    outs = [torch.full(tuple(x.shape), -1.0, device="cuda") for x in imgs]
    for rep in range(2):
        ctx.denoise_batch(imgs, sig, pilots=pil, outs=outs, graph=True)
        torch.cuda.synchronize()
        for i in range(len(imgs)):
            assert np.array_equal(outs[i].cpu().numpy(), refs[i]), (rep, i)


def test_batch_graph_replays_match_eager(torch, G, ctx):
    """Captured once, replayed several times with eager work and syncs in
    between; every replay equals the eager batch."""
    say("batch graph")
    imgs, sig = _batch_inputs(torch, 5, 40, 120, 800)
    eager = [o.cpu().numpy() for o in ctx.denoise_batch(imgs, sig)]
    outs = [torch.full(tuple(x.shape), -1.0, device="cuda") for x in imgs]
    for rep in range(4):
        for o in outs:
            o.fill_(-1.0)
        ctx.denoise_batch(imgs, sig, outs=outs, graph=True)
        torch.cuda.synchronize()
        _ = ctx.denoise(imgs[0], sig[0])          # eager work between replays
        torch.cuda.synchronize()
        for i in range(len(imgs)):
            assert np.array_equal(outs[i].cpu().numpy(), eager[i]), (rep, i)
    # new output buffers, same shapes: the graph is reused with the new pointers
    outs2 = [torch.empty(tuple(x.shape), device="cuda") for x in imgs]
    ctx.denoise_batch(imgs, sig, outs=outs2, graph=True)
    torch.cuda.synchronize()
    for i in range(len(imgs)):
        assert np.array_equal(outs2[i].cpu().numpy(), eager[i])


def test_batch_oracle_psnr(torch, G, ctx):
    """Batch outputs against the oracle's own two-stage run (PSNR within 0.01 dB)."""
    rng = np.random.default_rng(900)
    cases = [synth.make_case(int(h), int(w), s, 901 + i)
             for i, (h, w, s) in enumerate(zip(rng.integers(48, 90, 3), rng.integers(48, 90, 3),
                                               rng.uniform(10, 50, 3) / 255))]
    sig = [float(s) for s in rng.uniform(10, 50, 3) / 255]
    cases = [synth.make_case(c[1].shape[0], c[1].shape[1], s, 911 + i) for i, (c, s) in enumerate(zip(cases, sig))]
    p = G.default_params(search=21)
    outs = ctx.denoise_batch([up(torch, Z) for _, Z in cases], sig, params=p)
    for (clean, Z), s, o in zip(cases, sig, outs):
        Y, _, _ = O.denoise(Z, s, O.DEFAULT.with_(search=21))
        assert abs(O.psnr(o.cpu().numpy().astype(np.float64), clean) - O.psnr(Y, clean)) <= PSNR_TOL


# ---------------------------------------------------------------------------
# the large single image (4096 x 4096 with edge-rich rectangles)
# ---------------------------------------------------------------------------

@pytest.fixture(scope="module")
def large_case():
    return synth.large_image_case(4096, SIG, 4)


@pytest.mark.parametrize("method", METHODS)
def test_large_match_sampled(torch, G, ctx, large_case, method):
    """4096 x 4096, search 39, K = 16: 300 sampled references bit-exact."""
    _, Z = large_case
    say("match 4096 sampled", "method", method)
    ids = np.random.default_rng(3).choice(O.n_refs(4096, 4096, 3), 300, replace=False)
    got = ctx.match(up(torch, Z), 16, method=method).cpu().numpy().astype(np.int64)[ids]
    exp = O.match(Z, 16, O.DEFAULT, ref_ids=ids)
    assert np.array_equal(got, exp)


def test_large_stages_windows(torch, G, ctx, large_case):
    """4096 x 4096: stage 1 and stage 2 (pilot = clean image quantised) on
    windows that the oracle evaluates exactly (interior and wrapping)."""
    clean, Z = large_case
    Zt = up(torch, Z)
    say("basic 4096")
    Yg = ctx.basic(Zt, SIG).cpu().numpy().astype(np.float64)
    p = O.DEFAULT
    for (y0, x0, h, w) in _windows(4096, 4096, 16, 16):
        say("basic 4096 window", y0, x0)
        ids = O.refs_for_window(4096, 4096, p, y0, x0, h, w)
        Yo, (idx, margin, _, _) = O.basic_estimate(Z, SIG, p, ref_ids=ids, return_parts=True)
        rows, cols = (y0 + np.arange(h)) % 4096, (x0 + np.arange(w)) % 4096
        _check_stage1(Yg, Yo, idx, margin, p, ref_ids=ids, window=(rows, cols))
    del Yg
    pilot = synth.to_u16(clean)
    say("wiener 4096")
    Yw = ctx.wiener(Zt, up(torch, pilot), SIG).cpu().numpy().astype(np.float64)
    for (y0, x0, h, w) in _windows(4096, 4096, 12, 12):
        say("wiener 4096 window", y0, x0)
        ids = O.refs_for_window(4096, 4096, O.DEFAULT, y0, x0, h, w)
        Yo = O.wiener_estimate(Z, pilot, SIG, O.DEFAULT, ref_ids=ids)
        rows, cols = (y0 + np.arange(h)) % 4096, (x0 + np.arange(w)) % 4096
        assert np.abs(Yw[np.ix_(rows, cols)] - Yo[np.ix_(rows, cols)]).max() <= MAXABS


def _tie_image(kind, H, W):
    rng = np.random.default_rng(77)
    y, x = np.mgrid[:H, :W]
    if kind == "checkerboard":     # half the window at distance zero
        return ((y + x) % 2 * 65535).astype(np.uint16)
    if kind == "two levels":       # flat regions far apart, noise of a few units: near ties at large norms
        return (np.where((x // 29 + y // 23) % 2, 52000, 9000) + rng.integers(-3, 4, (H, W))).astype(np.uint16)
    return np.tile(rng.integers(0, 65536, (8, 8)), (H // 8 + 1, W // 8 + 1))[:H, :W].astype(np.uint16)


@pytest.mark.parametrize("kind", ["checkerboard", "two levels", "period 8"])
@pytest.mark.parametrize("S,K", [(39, 16), (39, 32), (31, 32), (21, 16), (7, 32), (3, 2)])
def test_match_many_near_ties(torch, G, ctx, kind, S, K):
    """Images on which many more candidates than K come near the K-th best
    (the correlation matcher's candidate lists are cut, and go through its
    queue in several parts), for every shape of its candidate grid."""
    H, W = 53, 82
    say("match near ties", kind, S, K)
    Z = _tie_image(kind, H, W)
    got = ctx.match(up(torch, Z), K, G.default_params(search=S, bm_method=2)).cpu().numpy().astype(np.int64)
    exp = O.match(Z, K, O.DEFAULT.with_(search=S))
    bad = np.nonzero((got != exp).any(axis=1))[0]
    assert bad.size == 0, (bad[:5], got[bad[:2]], exp[bad[:2]])


def _hard_image(kind, H, W):
    rng = np.random.default_rng(83)
    y, x = np.mgrid[:H, :W]
    if kind == "strokes":          # black on white: many blocks at the same nonzero distance
        z = np.full((H, W), 65535)
        for _ in range(H * W // 90):
            a, b = rng.integers(0, H), rng.integers(0, W)
            h, w = (1, 5) if rng.random() < 0.5 else (6, 1)
            z[a:a + h, b:b + w] = 0
        return z.astype(np.uint16)
    if kind == "dots":             # most blocks constant
        return np.where(rng.random((H, W)) < 0.004, 65535, 12345).astype(np.uint16)
    if kind == "steps":            # smooth ramps between far levels
        return (np.clip(32768 + 60000 * np.sin(x / 9.0) * np.cos(y / 13.0), 0, 65535)).astype(np.uint16)
    if kind == "levels":
        return (np.where((x // 29 + y // 23) % 2, 60000, 4000) + rng.integers(-128, 129, (H, W))).astype(np.uint16)
    if kind == "stripes":
        return (x // 3 % 2 * 65535).astype(np.uint16)
    if kind == "rounding":         # f16 roundings that put the nearer candidates last, around lone references
        z = np.kron(rng.choice([33809, 31819], (H // 10 + 1, W // 10 + 1)), np.ones((10, 10), np.int64))[:H, :W]
        for p0, q0 in ((12, 36), (48, 60)):
            z[p0 - 7:p0 + 15, q0 + 2:q0 + 24] = 0
            z[p0:p0 + 8, q0 + 9:q0 + 17] = 32815
        return z.astype(np.uint16)
    return np.tile(rng.integers(0, 65536, (16, 4)), (H // 16 + 1, W // 4 + 1))[:H, :W].astype(np.uint16)


@pytest.mark.parametrize("kind", ["strokes", "dots", "steps", "levels", "stripes", "rounding", "period 16 x 4"])
@pytest.mark.parametrize("S,K", [(39, 2), (39, 16), (39, 32), (33, 32), (21, 16), (23, 32), (15, 32), (9, 8), (7, 16)])
def test_match_exact_pass(torch, G, ctx, kind, S, K):
    """Images on whose tiles the correlation matcher's bound leaves hundreds of
    candidates per reference, so that exact keys of all pairs give the limit:
    every shape of its grid, an image larger than the region and its margin."""
    H, W = 86, 101
    say("match exact pass", kind, S, K)
    Z = _hard_image(kind, H, W)
    got = ctx.match(up(torch, Z), K, G.default_params(search=S, bm_method=2)).cpu().numpy().astype(np.int64)
    exp = O.match(Z, K, O.DEFAULT.with_(search=S))
    bad = np.nonzero((got != exp).any(axis=1))[0]
    assert bad.size == 0, (bad[:5], got[bad[:2]], exp[bad[:2]])
