"""Kernels at the sizes where their tilings can go wrong (edges, remainders, smallest and largest
of a range), against the oracle or plain FP64 definitions."""

import numpy as np
import pytest

from paper_2406_14542_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


@pytest.fixture(scope="module")
def P():
    import paper_2406_14542_amd as P
    P.lib()
    return P


SIZES = [12, 128, 128, 128, 1]


@pytest.mark.parametrize("n", [15, 16, 17, 32, 33, 16383, 16385, 16449, 32832])
def test_mlp_tiles(P, oracle_mod, n):
    """Tiles of 64 points (blocks of 16, halves of 32), up to 256 blocks that stride over the
    tiles.  FP32 sums of up to 128 terms per layer and, for the gradient, 64-point tile sums:
    rounding 2^-24 sqrt(128) per layer, four layers, is below 3e-6; 1e-5 and 2e-5 leave room for
    the functions' own ulp."""
    print(f"[mlp n={n}]", flush=True)
    rng = np.random.default_rng(n)
    flat32 = oracle_mod.mlp_pack(oracle_mod.mlp_init(SIZES, seed=3)).astype(np.float32)
    p64 = oracle_mod.mlp_unpack(flat32.astype(np.float64), SIZES)
    X = rng.standard_normal((n, 12)).astype(np.float32)
    gy = (0.5 + rng.uniform(size=n)).astype(np.float32)
    y = P.mlp_forward(dev(flat32), dev(X), 0.37).cpu().numpy()
    yw, cache = oracle_mod.mlp_forward(p64, X.astype(np.float64), 0.37)
    assert y.shape == (n,) and rel(y, yw) <= 1e-5, rel(y, yw)
    g = P.mlp_backward(dev(flat32), dev(X), dev(gy), 0.37).cpu().numpy()
    gw = oracle_mod.mlp_pack(oracle_mod.mlp_backward(p64, cache, gy.astype(np.float64), 0.37))
    assert rel(g, gw) <= 2e-5, rel(g, gw)
    # every point counts once: the output bias's gradient is the sum of the points' terms alone
    assert abs(g[-1] - gw[-1]) <= 2e-5 * abs(gw[-1])


def mrel(a, b, lmax, mmax):
    """relative L2 distance in the <.,.>_m norm"""
    _, ms = inputs.ell_of_index(lmax, mmax)
    w = np.where(ms == 0, 1.0, 2.0)
    return float(np.sqrt((w * np.abs(a - b) ** 2).sum() / (w * np.abs(b) ** 2).sum()))


@pytest.mark.parametrize("lmax,mmax,mode,det", [
    (5, 5, "fused", False), (125, 125, "paper", False), (126, 60, "fused", True),
    (253, 253, "fused", False), (254, 254, "paper", True), (700, 699, "fused", False),
    (1279, 1279, "fused", False), (1300, 700, "fused", True), (2049, 2049, "fused", False)])
def test_one_map_adjoint(P, oracle_mod, lmax, mmax, mode, det):
    """The adjoint of one map at the edges of its ring-pair splits (64 pairs per sub-block; 1, 2, 4
    and 6 pairs per lane from 1, 129, 641 and 1025 pairs on), and the same map as the fifth of a
    batch: within the plan's eps = 1e-12 times the margin of the other FP64 tests."""
    print(f"[one map lmax={lmax} mmax={mmax} {mode} det={det}]", flush=True)
    rng = np.random.default_rng(lmax)
    th, ph = inputs.uniform_points(rng, 61)
    d = rng.standard_normal((5, th.size))
    ref = oracle_mod.adjoint(lmax, mmax, th, ph, d[4:])
    p = P.Plan(lmax, mmax, dev(th), dev(ph), 1e-12, dfs_mode=mode, deterministic=det)
    one = p.adjoint(dev(d[4:])).cpu().numpy()
    assert mrel(one, ref, lmax, mmax) <= 1e-11
    assert np.all(one[0, :lmax + 1].imag == 0.0)
    five = p.adjoint(dev(d)).cpu().numpy()
    assert mrel(five[4:], ref, lmax, mmax) <= 1e-11
    if det:
        assert np.array_equal(p.adjoint(dev(d[4:])).cpu().numpy(), one)
        assert np.array_equal(five[4], one[0])
    p.status()


@pytest.mark.parametrize("lmax,mmax,B,mode", [
    (0, 0, 1, "fused"), (1, 1, 1, "fused"), (6, 6, 3, "paper"), (7, 3, 7, "fused"),
    (8, 8, 4, "fused"), (126, 126, 2, "paper"), (127, 127, 4, "fused"), (319, 300, 4, "fused"),
    (1279, 1279, 1, "fused"), (1280, 1280, 1, "fused"), (1280, 1279, 6, "fused"),
    (2050, 2050, 4, "fused")])
def test_synthesis_splits(P, oracle_mod, lmax, mmax, B, mode):
    """The Legendre synthesis at the edges of its splits: fewer degrees than a chunk of 8, columns
    of one degree, 64 pairs per sub-block, one and two sub-blocks per wave (up to 160 / 641 pairs),
    batches that split into 4 + 2 + 1 maps; points down to 1e-4 from the poles.  Bound: the plan's
    eps = 1e-12 times the margin of the other FP64 tests."""
    print(f"[synthesis lmax={lmax} mmax={mmax} B={B} {mode}]", flush=True)
    rng = np.random.default_rng(7 * lmax + B)
    th, ph = inputs.uniform_points(rng, 53)
    th[:2] = [1e-4, np.pi - 1e-4]
    alm = inputs.red_alm(rng, lmax, mmax, B)
    p = P.Plan(lmax, mmax, dev(th), dev(ph), 1e-12, dfs_mode=mode)
    f = p.synthesis(dev(alm)).cpu().numpy()
    assert rel(f, oracle_mod.synthesis(lmax, mmax, th, ph, alm)) <= 1e-11


@pytest.mark.parametrize("lmax,mmax,B,dtype,mode", [
    (14, 14, 1, "f64", "fused"), (17, 3, 2, "f64", "fused"), (23, 23, 1, "mixed", "paper"),
    (40, 37, 3, "f64", "fused"), (55, 41, 5, "f64", "paper"), (78, 78, 1, "mixed", "fused"),
    (100, 90, 2, "f64", "fused"), (134, 134, 1, "f64", "fused"), (190, 167, 4, "mixed", "fused"),
    (223, 223, 1, "f64", "fused"), (311, 300, 1, "f64", "fused"), (438, 400, 1, "f64", "fused"),
    (540, 540, 2, "mixed", "fused"), (1000, 900, 1, "f64", "fused"), (1500, 1500, 1, "f64", "fused"),
    (2100, 1050, 1, "f64", "fused"), (2300, 800, 1, "f64", "fused"), (2120, 2120, 1, "mixed", "fused"),
    (4320, 700, 1, "mixed", "fused")])
def test_general_lengths(P, oracle_mod, lmax, mmax, B, dtype, mode):
    """Fine-grid transforms of lengths other than 2^K and 5 2^K, both directions: all radices, one
    and several butterflies per thread, lengths just below and above 8192 and the LDS limit.
    Bounds: eps times the margin of the other tests (1e-11 FP64, 1e-5 mixed)."""
    eps = 1e-12 if dtype == "f64" else 1e-5
    tol = 1e-11 if dtype == "f64" else 1e-5
    rng = np.random.default_rng(11 * lmax + mmax)
    th, ph = inputs.uniform_points(rng, 61)
    p = P.Plan(lmax, mmax, dev(th), dev(ph), eps, dtype=dtype, dfs_mode=mode)
    print(f"[lengths lmax={lmax} mmax={mmax} B={B} {dtype} {mode}]", flush=True)
    alm = inputs.red_alm(rng, lmax, mmax, B)
    f = p.synthesis(dev(alm)).cpu().numpy()
    assert rel(f, oracle_mod.synthesis(lmax, mmax, th, ph, alm)) <= tol
    d = rng.standard_normal((B, th.size))
    c = p.adjoint(dev(d)).cpu().numpy()
    assert mrel(c, oracle_mod.adjoint(lmax, mmax, th, ph, d), lmax, mmax) <= tol


@pytest.mark.parametrize("width,n,B,taps", [
    (9, 1, 1, "poly"), (9, 777, 4, "poly"), (10, 5000, 2, "poly"), (11, 5000, 3, "exact"),
    (12, 255, 1, "poly"), (12, 257, 5, "poly"), (13, 5000, 1, "exact"), (14, 20000, 7, "poly"),
    (15, 3, 4, "poly"), (15, 5000, 1, "poly"), (16, 5000, 4, "exact"), (16, 20000, 1, "poly")])
def test_tile_spreading(P, width, n, B, taps):
    """The tile kernel of the wide FP64 spreading against the band sweep (a deterministic plan's
    kernel: the same taps, another split and order): one point, fewer and more points than a batch
    of 256 in a tile, all of a tile's points in one quadrant, both poles, the phi wrap, every batch
    remainder.  Bound 1e-12: the sums have at most a few thousand terms of rounding 1e-16."""
    print(f"[tile spreading w={width} n={n} B={B} {taps}]", flush=True)
    rng = np.random.default_rng(width * 1000 + n)
    th, ph = inputs.uniform_points(rng, n)
    k = n // 3
    th[:k] = 1.3 + 0.02 * rng.random(k)
    ph[:k] = 2.0 + 0.02 * rng.random(k)
    if n > 100:
        th[k:k + 4] = [0.0, np.pi, 1e-5, np.pi - 1e-5]
        ph[k + 4:k + 8] = [0.0, 2 * np.pi - 1e-9, 1e-9, np.pi]
    d = dev(rng.standard_normal((B, n)))
    c = [P.Plan(90, 77, dev(th), dev(ph), 1e-8, width=width, kernel_eval=taps, deterministic=det).adjoint(d)
         .cpu().numpy() for det in (False, True)]
    assert mrel(c[0], c[1], 90, 77) <= 1e-12


@pytest.mark.parametrize("lmax,B,dtype,mode", [
    (30, 2, "f64", "fused"), (63, 3, "f64", "paper"), (63, 9, "mixed", "fused"), (127, 6, "f64", "fused"),
    (255, 1, "f64", "fused"), (300, 7, "f64", "fused"), (511, 5, "f64", "fused")])
def test_batches_in_one_launch(P, lmax, B, dtype, mode):
    """Maps transformed together give what each gives alone: row passes of several maps in one
    launch, the last maps of a batch in one spreading or interpolation launch, short columns with
    the DFT over the doubled circle.  A map's arithmetic does not depend on its batch but for the
    order of some sums: 1e-13 FP64, 1e-6 mixed (sums of FP32)."""
    print(f"[batch lmax={lmax} B={B} {dtype} {mode}]", flush=True)
    rng = np.random.default_rng(lmax + B)
    th, ph = inputs.uniform_points(rng, 700)
    eps = 1e-12 if dtype == "f64" else 1e-5
    p = P.Plan(lmax, lmax, dev(th), dev(ph), eps, dtype=dtype, dfs_mode=mode)
    alm, d = dev(inputs.red_alm(rng, lmax, lmax, B)), dev(rng.standard_normal((B, 700)))
    f, c = p.synthesis(alm).cpu().numpy(), p.adjoint(d).cpu().numpy()
    tol = 1e-13 if dtype == "f64" else 1e-6
    for b in range(B):
        assert rel(f[b], p.synthesis(alm[b:b + 1].contiguous()).cpu().numpy()[0]) <= tol
        assert mrel(c[b], p.adjoint(d[b:b + 1].contiguous()).cpu().numpy()[0], lmax, lmax) <= tol


@pytest.mark.parametrize("lmax,mmax,s,F,det,mode", [
    (1, 1, 1, 1, False, "fused"), (2, 2, 2, 3, True, "fused"), (6, 5, 3, 2, False, "paper"),
    (125, 125, 2, 1, False, "fused"), (126, 126, 1, 2, True, "paper"), (254, 200, 2, 1, True, "fused"),
    (255, 255, 2, 2, False, "fused"), (509, 509, 30, 1, False, "fused"), (1023, 1000, 2, 1, False, "fused"),
    (1500, 300, 1, 2, False, "fused")])
def test_spin_adjoint_edges(P, oracle_mod, lmax, mmax, s, F, det, mode):
    """The Wigner-d adjoint where its split can go wrong: fewer degrees than a chunk of four and
    every remainder, 64 and 128 ring pairs per wave and one more, columns that stay scaled for
    long (m near mmax), one and two fields, partial arrays.  Bound as in the spin tests (1e-11)."""
    print(f"[spin adjoint lmax={lmax} mmax={mmax} s={s} F={F} det={det} {mode}]", flush=True)
    rng = np.random.default_rng(3 * lmax + s)
    th, ph = inputs.uniform_points(rng, 59)
    d = rng.standard_normal((F, 2, th.size))
    p = P.Plan(lmax, mmax, dev(th), dev(ph), 1e-12, deterministic=det, dfs_mode=mode)
    c = p.adjoint_spin(s, dev(d)).cpu().numpy()
    ref = oracle_mod.spin_adjoint(lmax, mmax, s, th, ph, d)
    assert mrel(c, ref, lmax, mmax) <= 1e-11
    if det:
        assert np.array_equal(p.adjoint_spin(s, dev(d)).cpu().numpy(), c)
    p.status()


@pytest.mark.parametrize("width,n,B,eps", [
    (9, 1, 4, 1e-6), (9, 710, 1, 1e-6), (9, 711, 2, 1e-6), (9, 711, 5, 1e-6), (10, 127, 3, 1e-7),
    (10, 384, 4, 1e-7), (10, 385, 4, 1e-7), (11, 129, 1, 1e-8), (11, 276, 3, 1e-8), (11, 277, 3, 1e-8),
    (12, 222, 4, 1e-9), (12, 223, 7, 1e-9), (13, 255, 1, 1e-10), (13, 256, 1, 1e-10), (13, 257, 6, 1e-10),
    (14, 168, 4, 1e-11), (14, 169, 4, 1e-11), (15, 512, 1, 1e-11), (15, 513, 4, 1e-11),
    (16, 128, 5, 1e-11), (16, 141, 1, 1e-11), (16, 142, 1, 1e-11), (16, 3000, 2, 1e-11)])
def test_spreading_kernels(P, width, n, B, eps):
    """Both tile kernels of the wide FP64 spreading at the line between them (60 + 650 / (w - 8)
    points a tile; one tile holds all points here), one point fewer and more than their batches of
    128 and 256 points, every remainder of a batch of maps: against the band sweep of
    a deterministic plan, which has the same taps.  Sums of at most 3000 terms agree to 1e-12."""
    print(f"[spreading w={width} n={n} B={B}]", flush=True)
    rng = np.random.default_rng(width * 1000 + n)
    # the first taps of all points within one tile: 20 cells around its middle
    g = P.geometry(90, 77, eps, width=width)
    at = [int(0.4 * m / 64) * 32 + 16 + 0.5 * width for m in (g["n1"], g["n2"])]
    th = (at[0] + 10.0 * (2 * rng.random(n) - 1)) * 2 * np.pi / g["n1"]
    ph = (at[1] + 10.0 * (2 * rng.random(n) - 1)) * 2 * np.pi / g["n2"]
    d = dev(rng.standard_normal((B, n)))
    plans = [P.Plan(90, 77, dev(th), dev(ph), eps, width=width, deterministic=det)
             for det in (False, True)]
    g = plans[0].geometry
    assert g["ntiles_used"] == 1 and g["kernel_eval"] == 0
    c = [p.adjoint(d).cpu().numpy() for p in plans]
    assert mrel(c[0], c[1], 90, 77) <= 1e-12


@pytest.mark.parametrize("lmax,mmax,s,F,det", [
    (126, 126, 2, 1, True), (255, 255, 2, 1, False), (255, 255, 1, 2, True), (511, 511, 3, 1, False),
    (767, 200, 2, 1, True), (1022, 40, 2, 1, True), (1023, 40, 2, 2, False), (1023, 40, 2, 2, True),
    (1151, 33, 1, 1, True)])
def test_spin_adjoint_waves(P, oracle_mod, lmax, mmax, s, F, det):
    """The Wigner-d adjoint's spans counted from the equator: a pole's pair alone in the last wave
    (129, 257, 385, 513 and 577 pairs at two or three per lane), blocks of one to four waves, the
    deterministic split on either side of 512 pairs; points next to the poles, so that column
    m = s, to which alone the pole's pair contributes, is checked by itself.  Bound as in the spin
    tests (1e-11)."""
    print(f"[spin waves lmax={lmax} mmax={mmax} s={s} F={F} det={det}]", flush=True)
    rng = np.random.default_rng(5 * lmax + s)
    th, ph = inputs.uniform_points(rng, 41)
    th[:4] = [0.0, 1e-3, np.pi - 1e-3, np.pi]
    d = rng.standard_normal((F, 2, th.size))
    p = P.Plan(lmax, mmax, dev(th), dev(ph), 1e-12, deterministic=det)
    c = p.adjoint_spin(s, dev(d)).cpu().numpy()
    ref = oracle_mod.spin_adjoint(lmax, mmax, s, th, ph, d)
    assert mrel(c, ref, lmax, mmax) <= 1e-11
    _, ms = inputs.ell_of_index(lmax, mmax)
    assert rel(c[..., ms == s], ref[..., ms == s]) <= 1e-11
    if det:
        assert np.array_equal(p.adjoint_spin(s, dev(d)).cpu().numpy(), c)


@pytest.mark.parametrize("lmax,mmax,mode,det", [
    (60, 60, "fused", False), (254, 200, "paper", True), (503, 503, "fused", False), (503, 90, "fused", True),
    (511, 90, "fused", True), (511, 511, "paper", False), (629, 80, "fused", True), (639, 80, "fused", True),
    (639, 639, "fused", False), (1259, 40, "fused", True), (1279, 40, "fused", True)])
def test_left_over_map(P, oracle_mod, lmax, mmax, mode, det):
    """One map by itself and as the fifth of a batch, at the lines between the adjoint's kernels and
    splits: up to 256 ring pairs a map left over joins the group before it (253 and 257 pairs), one
    to two pairs per lane after 320 (316, 321), two to four after 640 (631, 641).  A deterministic plan
    gives the same bits for both.  Bound as in test_one_map_adjoint."""
    print(f"[left over lmax={lmax} mmax={mmax} {mode} det={det}]", flush=True)
    rng = np.random.default_rng(lmax + mmax)
    th, ph = inputs.uniform_points(rng, 47)
    d = rng.standard_normal((5, th.size))
    ref = oracle_mod.adjoint(lmax, mmax, th, ph, d)
    p = P.Plan(lmax, mmax, dev(th), dev(ph), 1e-12, dfs_mode=mode, deterministic=det)
    one, five = p.adjoint(dev(d[4:])).cpu().numpy(), p.adjoint(dev(d)).cpu().numpy()
    assert mrel(one, ref[4:], lmax, mmax) <= 1e-11 and mrel(five, ref, lmax, mmax) <= 1e-11
    if det:
        assert np.array_equal(five[4], one[0])
    p.status()


def plan_scratch(p, B):
    """bytes of one of a plan's two work buffers for B maps (the largest intermediate of either mode),
    of the tile subgrids of wide FP64 kernels, and of the row spectrum that rocFFT's row plans need"""
    g = p.geometry
    e = 8 if p.dtype == "f64" else 4
    per = max(g["n1"] * (g["n2"] // 2 + 1) * 2 * e, g["n1"] * g["n2"] * e,
              g["nrings"] * (g["nphi"] // 2 + 1) * 16, (g["mmax"] + 1) * g["ntorus"] * 16)
    wide = e == 8 and g["width"] > 8
    sub = g["ntiles_used"] * (g["width"] + 31) * 48 * e * min(B, 4) if wide else 0
    h = g["n2"] // 2
    while h % 2 == 0:
        h //= 2
    rows = g["n1"] * (g["n2"] // 2 + 1) * 2 * e if e == 4 and h not in (1, 5) else 0
    return B * per, sub, rows


@pytest.mark.parametrize("lmax,n,B,dtype,eps", [
    (511, 2000000, 1, "f64", 1e-10), (255, 400000, 8, "f64", 1e-12), (500, 300000, 3, "f64", 1e-12),
    (383, 100000, 8, "mixed", 1e-5)])
def test_scratch_of_first_calls(P, lmax, n, B, dtype, eps):
    """Device memory that a plan takes in its first calls: two work buffers, the second at least as
    large as the subgrids of the maps spread together, and the packed point values of a group.  (Row
    spectra and subgrids lie in the work buffers, but for those of mixed plans of general length,
    which rocFFT transforms.)  Slack: the allocator's granules."""
    print(f"[scratch lmax={lmax} n={n} B={B} {dtype}]", flush=True)
    rng = np.random.default_rng(lmax)
    th, ph = (dev(x) for x in inputs.uniform_points(rng, n))
    d = torch.randn(B, n, device="cuda", dtype=torch.float64)
    for _ in range(2):  # the first plan loads the kernels and fills torch's cache
        p = P.Plan(lmax, lmax, th, ph, eps, dtype=dtype)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        c = p.adjoint(d)
        f = p.synthesis(c)
        torch.cuda.synchronize()
        used = free - torch.cuda.mem_get_info()[0]
        work, sub, rows = plan_scratch(p, B)
        del p, c, f
    most = work + max(work, sub) + rows + 8 * n * (4 if B >= 4 else 1)
    assert used <= most + (12 << 20), (used, most)


@pytest.mark.parametrize("lmax,mmax,dtype,mode,sigma", [
    (63, 63, "f64", "fused", 2.0), (90, 77, "f64", "paper", 2.0), (100, 100, "f64", "fused", 1.25),
    (127, 40, "f64", "paper", 1.25), (127, 127, "mixed", "fused", 2.0), (90, 90, "mixed", "paper", 2.0)])
def test_growing_batches(P, lmax, mmax, dtype, mode, sigma):
    """Batches of 1, 6, 2 and 9 maps through one plan (scratch that grows and is used in part) give
    what new plans give, row spectra behind the bands or, at sigma = 1.25 and few maps, apart: the
    same arithmetic but for the order of some sums (1e-13 FP64, 1e-6 mixed)."""
    print(f"[growing lmax={lmax} mmax={mmax} {dtype} {mode} {sigma}]", flush=True)
    rng = np.random.default_rng(lmax + mmax)
    th, ph = (dev(x) for x in inputs.uniform_points(rng, 900))
    eps, tol = (1e-8, 1e-13) if dtype == "f64" else (1e-4, 1e-6)
    new = lambda: P.Plan(lmax, mmax, th, ph, eps, dtype=dtype, dfs_mode=mode, sigma=sigma)
    p = new()
    for B in (1, 6, 2, 9, 1):
        alm, d = dev(inputs.red_alm(rng, lmax, mmax, B)), dev(rng.standard_normal((B, 900)))
        q = new()
        assert rel(p.synthesis(alm).cpu().numpy(), q.synthesis(alm).cpu().numpy()) <= tol
        c = p.adjoint(d).cpu().numpy()
        assert mrel(c, q.adjoint(d).cpu().numpy(), lmax, mmax) <= tol


@pytest.mark.parametrize("lmax,mmax,B,mode", [
    (48, 48, 2, "fused"), (1890, 300, 1, "fused"), (2010, 200, 1, "fused"), (2010, 2010, 1, "paper"),
    (2200, 2200, 1, "fused"), (4100, 4100, 1, "fused"), (4230, 4210, 1, "paper")])
def test_general_lengths_fp64(P, oracle_mod, lmax, mmax, B, mode):
    """The FP64 general-length kernels where the lists above do not reach: radix 2 (98 = 7 7 2), columns of
    7680 and 8064 (1024 threads at 8 values each), rows of 8064, rows of 8400 and 8640 (9 values per thread
    in the row kernels, above mmax 4096), columns of 8960.  Bound as there."""
    print(f"[lengths lmax={lmax} mmax={mmax} B={B} {mode}]", flush=True)
    rng = np.random.default_rng(13 * lmax + mmax)
    th, ph = inputs.uniform_points(rng, 29)
    p = P.Plan(lmax, mmax, dev(th), dev(ph), 1e-12, dfs_mode=mode)
    alm = inputs.red_alm(rng, lmax, mmax, B)
    f = p.synthesis(dev(alm)).cpu().numpy()
    assert rel(f, oracle_mod.synthesis(lmax, mmax, th, ph, alm)) <= 1e-11
    d = rng.standard_normal((B, th.size))
    c = p.adjoint(dev(d)).cpu().numpy()
    assert mrel(c, oracle_mod.adjoint(lmax, mmax, th, ph, d), lmax, mmax) <= 1e-11
