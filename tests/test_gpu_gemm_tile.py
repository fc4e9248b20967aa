"""The GEMM class on tiles of any size: every way an operand is loaded, K at
and around its chunks (16 fp32, 32 bf16), blocks of one and two MFMA tiles
with full and partial last rows, a workgroup and a wavefront per block, units
that split a key -- against float64."""
import numpy as np
import pytest

import paper_2603_08957_amd as tre
import workloads

pytestmark = pytest.mark.gpu

K_EDGES = [8, 15, 16, 17, 31, 32, 33, 47, 64, 100]
ROW_EDGES = [16, 31, 32, 33, 63, 64, 65, 96, 130]
# operand layouts: k contiguous or rows contiguous, each side
LAYOUTS = {"kk": "ik,nk->in", "kr": "ik,kn->in", "rk": "ki,nk->in", "rr": "ki,kn->in"}


def check(einsum, upper, ext, til, dtype, keep=0.8, seed=0, path="gemm", **plan_kw):
    import torch

    rng = np.random.default_rng(seed)
    la, lb = einsum.split("->")[0].split(",")
    rels = [workloads.random_relation(rng, x, upper, ext, til, dtype, keep) for x in (la, lb)]
    plan = tre.Plan(einsum, upper, ext, til, dtype, **plan_kw)
    assert plan.kernel_class == path

    def dev(r):
        t = r["tiles"]
        t = torch.from_numpy(t.view(np.int16)).cuda().view(torch.bfloat16) if dtype == "bf16" else \
            torch.from_numpy(t).cuda()
        return torch.from_numpy(r["keys"]).cuda(), t

    o = tre.einsum(plan, *dev(rels[0]), *dev(rels[1]), want_pairs=True, timing=True)
    assert o.timing["contract_path"] == "gemm"
    vals = [workloads.bf16_bits_to_f32(r["tiles"]) if dtype == "bf16" else r["tiles"] for r in rels]
    shapes = [[til[c] if c in upper else ext[c] for c in x] for x in (la, lb)]
    pairs = o.pairs.cpu().numpy()
    n_w = o.n_w
    wkeys = {tuple(k): i for i, k in enumerate(o.w_keys.cpu().numpy())}
    out = einsum.split("->")[1]
    w_shape = [til[c] if c in upper else ext[c] for c in out]
    ref, mag = np.zeros([n_w] + w_shape), np.zeros([n_w] + w_shape)
    ka, kb = [c for c in la if c in upper], [c for c in lb if c in upper]
    for u, v in pairs:
        at = dict(zip(ka, rels[0]["keys"][u])) | dict(zip(kb, rels[1]["keys"][v]))
        i = wkeys[tuple(at[c] for c in out if c in upper)]
        a = vals[0][u].reshape(shapes[0]).astype(np.float64)
        b = vals[1][v].reshape(shapes[1]).astype(np.float64)
        ref[i] += np.einsum(einsum, a, b)
        mag[i] += np.einsum(einsum, np.abs(a), np.abs(b))
    got = o.w_tiles.cpu().numpy().reshape(ref.shape)
    assert len(pairs) > 0
    # exact products summed in fp32: a few 2^-24 of the sum of magnitudes
    assert np.max(np.abs(got - ref) / np.maximum(mag, 1e-30)) <= 16 * 2.0 ** -24
    return o


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_k_edges(layout, dtype):
    for k in K_EDGES:
        check(LAYOUTS[layout], "ik", {"i": 80, "k": 3 * k, "n": 48}, {"i": 40, "k": k}, dtype, seed=k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_row_edges(layout, dtype):
    for i, m in enumerate(ROW_EDGES):
        n = ROW_EDGES[-1 - i]
        check(LAYOUTS[layout], "ik", {"i": 2 * m, "k": 72, "n": n}, {"i": m, "k": 36}, dtype, seed=m)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_offsets_not_affine(dtype):
    # rows and the contracted index made of two labels each, in two orders; a batch label
    check("aibj,bjn->ain", "", {"a": 5, "i": 8, "b": 6, "j": 7, "n": 40}, {}, dtype, keep=1.0)
    check("haik,hkn->hain", "k", {"h": 3, "a": 2, "i": 20, "k": 66, "n": 34}, {"k": 33}, dtype, keep=1.0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_short_units(dtype):
    """Thousands of one-pair units: a wavefront per block."""
    check("ik,kn->in", "i", {"i": 2500 * 17, "k": 40, "n": 33}, {"i": 17}, dtype, keep=1.0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_keys_split_between_units(dtype):
    o = check("ik,kn->in", "ik", {"i": 40, "k": 90 * 20, "n": 35}, {"i": 20, "k": 20}, dtype, max_pairs_per_unit=7)
    assert o.timing["n_partials"] > 0
