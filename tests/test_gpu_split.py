"""fp32 contractions on the bf16 matrix cores (csrc/split_f32.h): ordinary
values to fp32 accuracy, and values the three-part split does not hold --
infinities, NaN, magnitudes that round to infinity in bf16 or whose rest falls
below its smallest value -- computed as fp32, against float64."""
import numpy as np
import pytest

import paper_2603_08957_amd as tre

pytestmark = pytest.mark.gpu

# (einsum, promoted, extents, tiles): one shape for each kernel and operand layout
SHAPES = {
    "gemm128_krow": ("ik,kn->in", "ik", {"i": 128, "k": 256, "n": 128}, {"i": 128, "k": 128}),
    "gemm128_row_row": ("ki,kn->in", "ik", {"i": 128, "k": 64, "n": 256}, {"i": 128, "k": 32}),
    "gemm128_k_k": ("ik,nk->in", "ik", {"i": 128, "k": 64, "n": 128}, {"i": 128, "k": 32}),
    "tile_krun_rows": ("ik,kn->in", "ik", {"i": 120, "k": 80, "n": 70}, {"i": 40, "k": 40}),
    "tile_rows_krun": ("ki,nk->in", "ik", {"i": 100, "k": 102, "n": 33}, {"i": 50, "k": 51}),
    "tile_gather_short_k": ("ik,kn->in", "ik", {"i": 51, "k": 27, "n": 17}, {"i": 17, "k": 9}),
}


def values(kind, rng, shape):
    """Two operands' values; special ones in a few places of the first."""
    a = rng.standard_normal(shape[0]).astype(np.float32)
    b = rng.standard_normal(shape[1]).astype(np.float32)
    at = rng.choice(a.size, size=3, replace=False)
    if kind == "inf":
        a.flat[at] = [np.inf, -np.inf, np.inf]
    elif kind == "nan":
        a.flat[at] = np.nan
    elif kind == "largest":  # rounds to infinity in bf16, its products stay finite
        a.flat[at] = np.float32(3.4e38)
        b *= np.float32(1e-3)
    elif kind == "tiny":  # every value: low parts below 2^-126
        a *= np.float32(1e-35)
    elif kind == "tiny_times_huge":
        a *= np.float32(1e-36)
        b *= np.float32(1e30)
    return a, b


def relation(x, labels, upper, extents, tiles):
    """A dense array as a relation holding every key."""
    shape, order_key, order_tile, radix = [], [], [], []
    for c in labels:
        t = tiles[c] if c in upper else extents[c]
        shape += [extents[c] // t, t]
    x = x.reshape(shape)
    for i, c in enumerate(labels):
        (order_key if c in upper else order_tile).append(2 * i)
        order_tile.append(2 * i + 1)
        if c in upper:
            radix.append(shape[2 * i])
    n = int(np.prod(radix)) if radix else 1
    keys = np.stack(np.unravel_index(np.arange(n), radix), axis=1).astype(np.int32) if radix else \
        np.zeros((1, 0), np.int32)
    return keys, np.ascontiguousarray(x.transpose(order_key + sorted(order_tile))).reshape(n, -1)


def run(shape, a, b):
    import torch

    einsum, upper, ext, til = shape
    ops, out = einsum.split("->")
    la, lb = ops.split(",")
    plan = tre.Plan(einsum, upper, ext, til, "f32")
    (ak, at), (bk, bt) = relation(a, la, upper, ext, til), relation(b, lb, upper, ext, til)
    o = tre.einsum(plan, *(torch.from_numpy(x).cuda() for x in (ak, at, bk, bt)))
    keys = [c for c in out if c in upper]
    tile = [til[c] if c in upper else ext[c] for c in out]
    grid = [ext[c] // til[c] for c in keys]
    w = o.w_tiles.cpu().numpy().reshape(grid + tile)
    assert o.n_w == int(np.prod(grid))
    # the promoted labels' grid dims go in front of their tile dims
    perm, g = [], 0
    for i, c in enumerate(out):
        if c in upper:
            perm.append(g)
            g += 1
        perm.append(len(grid) + i)
    return plan, w.transpose(perm).reshape([ext[c] for c in out])


@pytest.mark.parametrize("kind", ["normal", "inf", "nan", "largest", "tiny", "tiny_times_huge"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_split_against_float64(name, kind):
    shape = SHAPES[name]
    einsum, _, ext, _ = shape
    ops = einsum.split("->")[0].split(",")
    rng = np.random.default_rng(7)
    a, b = values(kind, rng, [tuple(ext[c] for c in o) for o in ops])
    plan, got = run(shape, a, b)
    assert plan.kernel_class == ("gemm128" if name.startswith("gemm128") else "gemm")
    with np.errstate(invalid="ignore", over="ignore"):
        ref = np.einsum(einsum, a.astype(np.float64), b.astype(np.float64))
        mag = np.einsum(einsum, np.abs(a).astype(np.float64), np.abs(b).astype(np.float64))
    fin = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    # fp32 sums of K products: at most (K + 1) 2^-24 of the sum of magnitudes,
    # in practice sqrt(K): K is at most 256
    assert np.max(np.abs(got[fin] - ref[fin]) / mag[fin]) <= 16 * 2.0 ** -24
    if kind == "normal":
        assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-6


def three_way(tp, tq, m, r, n_u, rng, kind="normal"):
    """A[i, r] = sum_jk T[i, j, k] B[j, r] C[k, r] on n_u random tuples of a
    5 x 4 x 4 key grid, with the float64 value and magnitude per output tuple."""
    import torch

    ext = {"i": 5 * m, "j": 4 * tp, "k": 4 * tq, "r": r}
    til = {"i": m, "j": tp, "k": tq}
    ids = np.sort(rng.choice(80, size=n_u, replace=False))
    tk = np.stack([ids // 16, ids // 4 % 4, ids % 4], 1).astype(np.int32)
    t, b = values(kind, rng, [(n_u, m, tp, tq), (4, tp, r)])
    c = rng.standard_normal((4, tq, r)).astype(np.float32)
    if kind == "largest":  # the products with C are summed first, in fp32: 3.4e38 x 4 x 1e-3 fits
        c *= np.float32(1e-3)
    rows, at = np.unique(tk[:, 0], return_inverse=True)
    ref, mag = np.zeros((len(rows), m, r)), np.zeros((len(rows), m, r))
    with np.errstate(invalid="ignore", over="ignore"):
        for s in range(n_u):
            args = (t[s].astype(np.float64), b[tk[s, 1]].astype(np.float64), c[tk[s, 2]].astype(np.float64))
            ref[at[s]] += np.einsum("ijk,jr,kr->ir", *args)
            mag[at[s]] += np.einsum("ijk,jr,kr->ir", *(np.abs(x) for x in args))
    k1 = torch.arange(4, dtype=torch.int32, device="cuda").reshape(4, 1)
    wk, wt, nt = tre.execute3("ijk,jr,kr->ir", "ijk", ext, til, torch.from_numpy(tk).cuda(),
                              torch.from_numpy(t.reshape(n_u, -1)).cuda(), k1, torch.from_numpy(b.reshape(4, -1)).cuda(),
                              k1.clone(), torch.from_numpy(c.reshape(4, -1)).cuda())
    assert nt == n_u and np.array_equal(wk.cpu().numpy()[:, 0], rows)
    return wt.cpu().numpy().reshape(ref.shape), ref, mag


@pytest.mark.parametrize("tq", [4, 12, 16, 20, 32, 36, 48, 52, 64])
def test_three_operands_against_float64(tq):
    """Every count of 16-wide steps, whole and partial, with 1 to 64 rows of p
    (fewer than the wavefronts that share them too), partial row and column blocks."""
    rng = np.random.default_rng(tq)
    for tp, m, r, n_u in ((1, 5, 7, 40), (3, 32, 64, 61), (8, 33, 65, 17), (32, 40, 70, 9), (64, 16, 40, 30)):
        got, ref, mag = three_way(tp, tq, m, r, n_u, rng)
        # (tp tq n products summed in fp32, in practice well below sqrt(n) 2^-24)
        assert np.max(np.abs(got - ref) / mag) <= 32 * 2.0 ** -24


@pytest.mark.parametrize("kind", ["inf", "nan", "largest", "tiny", "tiny_times_huge"])
def test_three_operands_split(kind):
    got, ref, mag = three_way(8, 32, 32, 64, 20, np.random.default_rng(3), kind)
    fin = np.isfinite(ref)
    # (infinities: the fp32 sums may meet +inf - inf where float64's do, and only there)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.max(np.abs(got[fin] - ref[fin]) / mag[fin]) <= 32 * 2.0 ** -24


# (scale of the first operand, of the second): subnormal values whose products
# are not, values below bf16's smallest (2^-133), parts below its smallest
# normal value, products and sums that are subnormal, and large ones
SCALES = {
    "subnormal": (1e-39, 1e9),
    "subnormal_times_large": (1e-39, 1e30),
    "below_bf16": (1e-42, 3e4),
    "low_parts": (3e-36, 1e3),
    "small": (1e-12, 1e-12),
    "tiny_products": (1e-19, 1e-19),
    "subnormal_products": (1e-20, 3e-21),
    "large": (1e18, 1e18),
}


@pytest.mark.parametrize("scale", list(SCALES))
@pytest.mark.parametrize("name", list(SHAPES))
def test_split_magnitudes(name, scale):
    """Operands scaled over fp32's range, some zeros among them, against float64."""
    shape = SHAPES[name]
    einsum, _, ext, _ = shape
    ops = einsum.split("->")[0].split(",")
    rng = np.random.default_rng(11)
    a, b = ((rng.standard_normal([ext[c] for c in o]) * s).astype(np.float32) for o, s in zip(ops, SCALES[scale]))
    a[rng.random(a.shape) < 0.2] = 0
    _, got = run(shape, a, b)
    ref = np.einsum(einsum, a.astype(np.float64), b.astype(np.float64))
    mag = np.einsum(einsum, np.abs(a).astype(np.float64), np.abs(b).astype(np.float64))
    # as above, and where products or sums are subnormal their roundings, at
    # most 2^-150 each: six products and six sums for every k
    assert np.all(np.abs(got - ref) <= 16 * 2.0 ** -24 * mag + 12 * ext["k"] * 2.0 ** -150)
    if scale in ("subnormal", "subnormal_times_large", "below_bf16"):
        assert np.count_nonzero(got) > 0.99 * got.size


@pytest.mark.parametrize("scale", list(SCALES))
def test_three_operands_magnitudes(scale):
    import torch

    sa, sb = SCALES[scale]
    rng = np.random.default_rng(12)
    ext, til = {"i": 70, "j": 24, "k": 64, "r": 70}, {"i": 35, "j": 12, "k": 16}
    ids = np.sort(rng.choice(16, size=13, replace=False))
    tk = np.stack([ids // 8, ids // 4 % 2, ids % 4], 1).astype(np.int32)
    t = (rng.standard_normal((13, 35, 12, 16)) * sa).astype(np.float32)
    t[rng.random(t.shape) < 0.2] = 0
    b = rng.standard_normal((2, 12, 70)).astype(np.float32)
    c = (rng.standard_normal((4, 16, 70)) * sb).astype(np.float32)
    k = [torch.arange(n, dtype=torch.int32, device="cuda").reshape(n, 1) for n in (2, 4)]
    wk, wt, nt = tre.execute3("ijk,jr,kr->ir", "ijk", ext, til, torch.from_numpy(tk).cuda(),
                              torch.from_numpy(t.reshape(13, -1)).cuda(), k[0], torch.from_numpy(b.reshape(2, -1)).cuda(),
                              k[1], torch.from_numpy(c.reshape(4, -1)).cuda())
    assert nt == 13
    rows, at = np.unique(tk[:, 0], return_inverse=True)
    ref, mag, pmag = (np.zeros((len(rows), 35, 70)) for _ in range(3))
    for s in range(13):
        args = [x.astype(np.float64) for x in (t[s], b[tk[s, 1]], c[tk[s, 2]])]
        ref[at[s]] += np.einsum("ijk,jr,kr->ir", *args)
        mag[at[s]] += np.einsum("ijk,jr,kr->ir", *(np.abs(x) for x in args))
        pmag[at[s]] += np.abs(args[1]).sum(0)[None]
    got = wt.cpu().numpy().reshape(ref.shape)
    # (the sums over k may be subnormal before the factor of the j operand meets them)
    assert np.all(np.abs(got - ref) <= 32 * 2.0 ** -24 * mag + 12 * 16 * 2.0 ** -150 * (pmag + 13 * 12))
    assert np.count_nonzero(got) > 0.99 * got.size


def with_tails(kind, rng, a, b):
    """a's contracted index last, b's first: values below bf16's grid (2^-133)
    among ordinary ones, whose loss shows in no sum ("tails") or in every sum,
    beside one row of huge values ("huge"), in a few places of one chunk."""
    if kind == "tails":
        a[rng.random(a.shape) < 0.5] *= np.float32(1e-43)
        b[rng.random(b.shape) < 0.1] *= np.float32(1e-40)
    else:
        k = a.shape[-1] - 3
        a *= np.float32(1e-6)
        a[..., k] = np.float32(3e-43)
        b[k] = np.float32(1e38)


@pytest.mark.parametrize("kind", ["tails", "huge"])
@pytest.mark.parametrize("name", ["gemm128_krow", "gemm128_long", "tile_krun_rows", "tile_waves"])
def test_split_tails(name, kind):
    shape = {**SHAPES, "gemm128_long": ("ik,kn->in", "ik", {"i": 128, "k": 1024, "n": 128}, {"i": 128, "k": 128}),
             "tile_waves": ("ik,kn->in", "i", {"i": 40 * 3000, "k": 48, "n": 40}, {"i": 40})}[name]
    einsum, _, ext, _ = shape
    rng = np.random.default_rng(21)
    a = rng.standard_normal((ext["i"], ext["k"])).astype(np.float32)
    b = rng.standard_normal((ext["k"], ext["n"])).astype(np.float32)
    with_tails(kind, rng, a, b)
    _, got = run(shape, a, b)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    mag = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)
    assert np.max(np.abs(got - ref) / mag) <= 16 * 2.0 ** -24


@pytest.mark.parametrize("kind", ["tails", "huge", "huge_q"])
def test_three_operands_tails(kind):
    import torch

    rng = np.random.default_rng(22)
    ext, til = {"i": 64, "j": 24, "k": 80, "r": 70}, {"i": 32, "j": 12, "k": 40}
    tk = np.stack(np.unravel_index(np.arange(8), (2, 2, 2)), 1).astype(np.int32)
    t = rng.standard_normal((8, 32, 12, 40)).astype(np.float32)
    b = rng.standard_normal((2, 12, 70)).astype(np.float32)
    c = rng.standard_normal((2, 40, 70)).astype(np.float32)
    if kind == "huge_q":  # the value that is lost is Q's
        t[..., 7] = np.float32(1e38)
        t[..., :7] *= np.float32(1e-6)
        t[..., 8:] *= np.float32(1e-6)
        c[:, 7] = np.float32(3e-43)
    else:
        for x in c:
            with_tails(kind, rng, t, x)
    k1 = torch.arange(2, dtype=torch.int32, device="cuda").reshape(2, 1)
    _, wt, nt = tre.execute3("ijk,jr,kr->ir", "ijk", ext, til, torch.from_numpy(tk).cuda(),
                             torch.from_numpy(t.reshape(8, -1)).cuda(), k1, torch.from_numpy(b.reshape(2, -1)).cuda(),
                             k1.clone(), torch.from_numpy(c.reshape(2, -1)).cuda())
    assert nt == 8
    ref, mag = np.zeros((2, 32, 70)), np.zeros((2, 32, 70))
    for s in range(8):
        args = [x.astype(np.float64) for x in (t[s], b[tk[s, 1]], c[tk[s, 2]])]
        ref[tk[s, 0]] += np.einsum("ijk,jr,kr->ir", *args)
        mag[tk[s, 0]] += np.einsum("ijk,jr,kr->ir", *(np.abs(x) for x in args))
    assert np.max(np.abs(wt.cpu().numpy().reshape(ref.shape) - ref) / mag) <= 32 * 2.0 ** -24
