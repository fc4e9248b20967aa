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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_k,big,n", [(401, 1500, 1), (1300, 1200, 3), (70, 900, 2)])
def test_keys_of_very_different_lengths(n_k, big, n, dtype):
    """One to three keys of `big` pairs among keys of two: the long ones are cut
    (their units' partial tiles summed with the outputs), the others are not."""
    import torch

    rng = np.random.default_rng(n_k)
    tj, tk, feat = 20, 24, 33
    keys = {(k, j) for k in range(n_k) for j in (3, 9)} | {(5 + 7 * i, j) for i in range(n) for j in range(big)}
    vk = np.array(sorted(keys), dtype=np.int32)
    u = rng.standard_normal((big, feat * tj)).astype(np.float32)
    v = rng.standard_normal((len(vk), tk * tj)).astype(np.float32)
    dev = [torch.from_numpy(x).cuda() for x in (u, v)]
    if dtype == "bf16":
        dev = [x.to(torch.bfloat16) for x in dev]
        u, v = (x.float().cpu().numpy() for x in dev)
    plan = tre.Plan("ij,kj->ki", "jk", {"i": feat, "j": big * tj, "k": n_k * tk}, {"j": tj, "k": tk}, dtype)
    assert plan.kernel_class == "gemm"
    uk = torch.arange(big, dtype=torch.int32, device="cuda").reshape(big, 1)
    o = tre.einsum(plan, uk, dev[0], torch.from_numpy(vk).cuda(), dev[1], timing=True)
    assert 0 < o.timing["n_split_segments"] <= n and o.n_w == n_k
    ref, mag = np.zeros((n_k, tk, feat)), np.zeros((n_k, tk, feat))
    for k in {5 + 7 * i for i in range(n)} | {0, 1, n_k - 1}:
        at = np.flatnonzero(vk[:, 0] == k)
        a = v[at].reshape(-1, tk, tj).transpose(1, 0, 2).reshape(tk, -1).astype(np.float64)
        b = u[vk[at, 1]].reshape(-1, feat, tj).transpose(0, 2, 1).reshape(-1, feat).astype(np.float64)
        ref[k], mag[k] = a @ b, np.abs(a) @ np.abs(b)
        got = o.w_tiles[k].cpu().numpy().reshape(tk, feat)
        # (30,000 products at most in one sum, in practice well below its square root)
        assert np.max(np.abs(got - ref[k]) / mag[k]) <= 16 * 2.0 ** -24
    assert torch.equal(o.w_keys.cpu()[:, 0], torch.arange(n_k, dtype=torch.int32))
    assert bool((o.w_tiles.abs().sum(1) > 0).all())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("b,j", [(1, 24), (3, 8), (2, 16), (5, 24), (4, 32)])
def test_contracted_runs(b, j, dtype):
    """Contracted indices in runs of eight that are not affine (labels b and j
    apart), on one side, on the other and on both; K below and above a chunk."""
    n = {"s": 3, "i": 37, "b": b, "j": j, "n": 35}
    check("sbij,sbjn->sin", "s", n, {"s": 1}, dtype, keep=1.0)
    check("sbjn,sbij->sin", "s", n, {"s": 1}, dtype, keep=1.0)
    check("sbij,sbnj->sin", "s", n, {"s": 1}, dtype, keep=1.0)


@pytest.mark.parametrize("k", [8, 24, 40, 64])
def test_contracted_runs_beside_odd_rows(k):
    # bf16 with an odd number of columns: element loads on one side only
    check("ik,kn->in", "ik", {"i": 4 * 40, "k": 6 * k, "n": 47}, {"i": 40, "k": k}, "bf16", seed=k)
    check("kn,ik->in", "ik", {"i": 4 * 40, "k": 6 * k, "n": 47}, {"i": 40, "k": k}, "bf16", seed=k)
