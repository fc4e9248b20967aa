"""fp32 contractions on the bf16 matrix cores (csrc/split_f32.h): ordinary
values to fp32 accuracy, and values the three-part split does not hold --
infinities, NaN, magnitudes that round to infinity in bf16 or whose low parts
fall below its smallest normal value -- computed as fp32, against float64."""
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
