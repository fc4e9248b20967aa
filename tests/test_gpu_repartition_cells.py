"""Repartition of relations with most of their tuples there (the copy over the
cells of each target tile): complete, with tuples missing (cells of zeros),
tiles that nest and that do not, runs around the chunk widths, target lists of
one workgroup and of many -- bit-exact against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check(orc, labels, up_in, up_out, ext, tin, tout, dtype, keep, seed=0, offset=0):
    import torch

    import paper_2603_08957_amd as tre

    rng = np.random.default_rng(seed)
    grids = np.meshgrid(*[np.arange(ext[c] // tin[c], dtype=np.int32) for c in labels if c in up_in], indexing="ij")
    keys = np.stack([g.reshape(-1) for g in grids], 1) if grids else np.zeros((1, 0), np.int32)
    n_all = len(keys)
    if keep < 1.0:
        keys = keys[np.sort(rng.choice(n_all, max(1, int(np.ceil(keep * n_all))), replace=False))]
    te = int(np.prod([tin[c] if c in up_in else ext[c] for c in labels]))
    vals = rng.standard_normal((len(keys), te)).astype(np.float32)
    if dtype == "bf16":
        bits = orc.f32_to_bf16(vals)
        host, ref_vals = torch.from_numpy(bits.view(np.int16)), orc.bf16_to_f64(bits)
    else:
        host, ref_vals = torch.from_numpy(vals), vals.astype(np.float64)
    # tiles that start `offset` elements into an allocation
    buf = torch.zeros(host.numel() + offset, dtype=host.dtype, device="cuda")
    buf[offset:] = host.reshape(-1).cuda()
    dev = buf[offset:].view(host.shape)
    k2, t2 = tre.repartition(labels, up_in, up_out, ext, tin, tout, torch.from_numpy(np.ascontiguousarray(keys)).cuda(),
                             dev)
    rk, rt = orc.repartition(labels, up_in, up_out, ext, tin, tout, np.ascontiguousarray(keys), ref_vals)
    assert np.array_equal(k2.cpu().numpy().reshape(rk.shape), rk)
    got = t2.cpu().numpy()
    got = orc.bf16_to_f64(got.view(np.uint16)) if dtype == "bf16" else got.astype(np.float64)
    assert np.array_equal(got.reshape(rt.shape), rt)


@pytest.fixture(scope="module")
def orc():
    import oracle

    oracle.build()
    return oracle


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("keep", [1.0, 0.75, 0.5])
def test_cells(orc, keep, dtype):
    # source / target columns whose common runs are 1 .. 17 elements, nested and not
    for a, b in [(1, 3), (2, 5), (3, 4), (4, 8), (5, 7), (7, 8), (8, 9), (9, 16), (16, 17), (6, 64)]:
        ext = {"i": 12, "j": 2 * a * b}
        check(orc, "ij", "ij", "ij", ext, {"i": 3, "j": a}, {"i": 4, "j": b}, dtype, keep, a)
        check(orc, "ij", "ij", "ij", ext, {"i": 4, "j": b}, {"i": 6, "j": a}, dtype, keep, b, offset=1)
    # labels promoted on one side only, three labels, one tuple without keys
    check(orc, "ij", "i", "j", {"i": 36, "j": 40}, {"i": 6}, {"j": 5}, dtype, keep)
    check(orc, "abc", "ab", "bc", {"a": 6, "b": 20, "c": 24}, {"a": 2, "b": 4}, {"b": 10, "c": 8}, dtype, keep)
    check(orc, "abc", "abc", "abc", {"a": 12, "b": 30, "c": 36}, {"a": 4, "b": 3, "c": 6}, {"a": 6, "b": 5, "c": 9},
          dtype, keep)
    check(orc, "ij", "", "ij", {"i": 30, "j": 33}, {}, {"i": 5, "j": 11}, dtype, 1.0)
    check(orc, "ij", "ij", "", {"i": 30, "j": 33}, {"i": 5, "j": 11}, {}, dtype, keep)


@pytest.mark.parametrize("n_out", [255, 4095, 4096, 4097, 16383, 16384, 16385, 40000])
def test_target_lists(orc, n_out):
    check(orc, "k", "k", "k", {"k": 2 * n_out}, {"k": 1}, {"k": 2}, "f32", 0.6, n_out)
    check(orc, "k", "k", "k", {"k": 2 * n_out}, {"k": 2 * n_out}, {"k": 2}, "bf16", 1.0)


def test_cells_larger_than_a_batch(orc):
    check(orc, "ij", "ij", "ij", {"i": 768, "j": 520}, {"i": 256, "j": 260}, {"i": 384, "j": 104}, "f32", 0.9)
    check(orc, "ij", "i", "i", {"i": 900, "j": 301}, {"i": 300}, {"i": 450}, "bf16", 1.0)


def test_bad_keys():
    import torch

    import paper_2603_08957_amd as tre

    t = torch.zeros((4, 2)).cuda()
    for keys, status in (([0, 2, 1, 3], "TRE_E_UNSORTED"), ([0, 1, 1, 3], "TRE_E_DUPKEY"),
                         ([0, 1, 2, 4], "TRE_E_KEYRANGE"), ([-1, 1, 2, 3], "TRE_E_KEYRANGE")):
        with pytest.raises(tre.TreError) as ei:
            tre.repartition("ij", "i", "i", {"i": 4, "j": 2}, {"i": 1}, {"i": 2},
                            torch.tensor(keys, dtype=torch.int32).reshape(4, 1).cuda(), t)
        assert ei.value.status == status
