"""Vector-class contractions over consecutive elements (one output element per
group of lanes), at and around the groups' spans, and joins whose pairs come
out grouped because W's key is U's followed by V's other labels."""
import numpy as np
import pytest

import workloads
from _parity import check, gpu_run

pytestmark = pytest.mark.gpu


def run(orc, e, upper, ext, til, dtype, seed=0, keep=0.7, **plan_kw):
    import torch  # noqa: F401  (before the library: both then use one HIP runtime)

    rng = np.random.default_rng(seed)
    la, lb = e.split("->")[0].split(",")
    U = workloads.random_relation(rng, la, upper, ext, til, dtype, keep)
    V = workloads.random_relation(rng, lb, upper, ext, til, dtype, keep)
    spec = workloads.spec(e, upper, ext, til, dtype)
    plan, out = gpu_run(spec, U, V, **plan_kw)
    check(out, orc.run(orc.Plan(e, upper, ext, til), U, V), dtype)
    return plan, out


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k", [15, 16, 17, 63, 64, 65, 128, 256, 257, 260, 512, 520, 1000, 1024])
def test_dot(orc, k, dtype):
    # one element per key; several (odd) elements per tile, several pairs per key; keys cut into units
    plan, _ = run(orc, "ijk,jk->ij", "ij", {"i": 9, "j": 11, "k": k}, {"i": 1, "j": 1}, dtype, seed=k)
    assert plan.kernel_class == "vec"
    run(orc, "mak,nk->man", "a", {"m": 5, "a": 6, "n": 3, "k": k}, {"a": 2}, dtype, seed=k + 1)
    run(orc, "jmk,jk->m", "j", {"j": 40, "m": 7, "k": k}, {"j": 1}, dtype, seed=k + 2, max_pairs_per_unit=5)


@pytest.mark.parametrize("e,upper", [
    ("ik,ij->ijk", "ij"),    # rows scaled by an edge list sorted by the row
    ("ix,jiy->ijxy", "ij"),  # V in another order than its joined label first
    ("abx,bcdy->abcxy", "abcd"),  # not all of V's other labels
    ("ax,by->abxy", "ab"),   # nothing joined
    ("x,by->bxy", "b"),      # U without promoted labels
])
@pytest.mark.parametrize("keep", [1.0, 0.5])
def test_grouped_by_u_then_v(orc, e, upper, keep):
    ext = {c: (6 if c in upper else 3) for c in set(e) if c.isalpha()}
    for small in (0, -1):
        plan, _ = run(orc, e, upper, ext, {c: 2 if c == "a" else 1 for c in upper}, "f32", seed=3, keep=keep, small_join=small)
        assert not plan.group_needs_sort
    ext = {c: (40 if c in "bij" else 8 if c in upper else 3) for c in ext}  # more pairs than one workgroup joins
    run(orc, e, upper, ext, {c: 1 for c in upper}, "f32", seed=4, keep=keep)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [256, 129, 40])
def test_dot_many_elements(n, dtype):
    """Enough sums to fill the chip with 4 lanes each (65,536), with 16 each
    (16,384) and fewer, at and around the lengths where more lanes are taken,
    against float64."""
    import torch

    import paper_2603_08957_amd as tre

    g = torch.Generator(device="cuda").manual_seed(n)
    keys = torch.cartesian_prod(torch.arange(n), torch.arange(n)).to(torch.int32).cuda()
    vk = torch.arange(n, dtype=torch.int32, device="cuda").reshape(n, 1)
    for k in (16, 17, 20, 31, 32, 33, 63, 64, 65, 127, 128, 129, 136, 255, 256, 257, 264, 512, 516, 520, 1024, 1032):
        u, v = (torch.randn((m, k), generator=g, device="cuda") for m in (n * n, n))
        if dtype == "bf16":
            u, v = u.to(torch.bfloat16), v.to(torch.bfloat16)
        plan = tre.Plan("ijk,jk->ij", "ij", {"i": n, "j": n, "k": k}, {"i": 1, "j": 1}, dtype)
        assert plan.kernel_class == "vec"
        o = tre.einsum(plan, keys, u, vk, v)
        x = u.reshape(n, n, k).double() * v.double()[None]
        err = (o.w_tiles.reshape(n, n).double() - x.sum(2)).abs() / x.abs().sum(2)
        # exact bf16 products, rounded fp32 ones; sums in fp32
        assert float(err.max()) <= 8 * 2.0 ** -24, k
