"""Joins whose U key lists the joined labels in another order than V's, with
radices that differ and U complete: U is then not indexed by V's join key."""
import numpy as np
import pytest

import workloads
from _parity import check, gpu_run

pytestmark = pytest.mark.gpu

PLANS = [
    # (einsum, promoted, radices of the promoted labels)
    ("ijx,jix->ijx", "ij", {"i": 64, "j": 48}),
    ("ijx,jikx->ijkx", "ijk", {"i": 40, "j": 30, "k": 3}),
    ("jix,ijky->jikxy", "ijk", {"i": 30, "j": 40, "k": 3}),
    ("ijx,jix->jx", "ij", {"i": 64, "j": 48}),  # grouped by a label of V's order: sorted
    ("hijx,jhix->hix", "hij", {"h": 8, "i": 14, "j": 12}),  # three joined labels, none in its place
]


@pytest.mark.parametrize("small", [0, -1])
@pytest.mark.parametrize("keep_v", [1.0, 0.6])
@pytest.mark.parametrize("idx", range(len(PLANS)))
def test_joined_labels_in_another_order(orc, idx, keep_v, small):
    import torch  # noqa: F401  (before the library: both then use one HIP runtime)

    e, upper, radix = PLANS[idx]
    ext = {**radix, "x": 2, "y": 3}
    ext = {c: n for c, n in ext.items() if c in e}
    til = {c: 1 for c in upper}
    rng = np.random.default_rng(90 + idx)
    la, lb = e.split("->")[0].split(",")
    U = workloads.random_relation(rng, la, upper, ext, til, "f32", 1.0)
    V = workloads.random_relation(rng, lb, upper, ext, til, "f32", keep_v)
    assert len(U["keys"]) > 1024  # more than one workgroup joins
    spec = workloads.spec(e, upper, ext, til, "f32")
    _, out = gpu_run(spec, U, V, small_join=small)
    check(out, orc.run(orc.Plan(e, upper, ext, til), U, V), "f32")


@pytest.mark.parametrize("small", [0, -1])
@pytest.mark.parametrize("e,upper", [
    ("jx,jx->jx", "j"),      # one attribute on the driving side
    ("jx,jabx->ax", "jab"),  # three, V drives
    ("abjx,jx->ax", "jab"),  # three and four, U drives
    ("abcjx,jx->ax", "jabc"),
    ("bjx,bx->jx", "jb"),    # grouped by the attribute that is not first: sorted
])
def test_dense_join_by_arity(orc, e, upper, small):
    """One join label, W keyed by one label of the driving relation."""
    import torch

    import paper_2603_08957_amd as tre
    from _parity import to_dev

    ext = {"j": 9, "a": 7, "b": 6, "c": 5, "x": 2} if len(upper) > 2 else {"j": 40, "b": 37, "x": 2}
    if e == "jx,jx->jx":
        ext["j"] = 2000
    ext, til = {c: n for c, n in ext.items() if c in e}, {c: 1 for c in upper}
    la, lb = e.split("->")[0].split(",")
    whole = "u" if la == "jx" else "v"  # the relation that holds every key
    rng = np.random.default_rng(len(e))
    U = workloads.random_relation(rng, la, upper, ext, til, "f32", 1.0 if whole == "u" else 0.7)
    V = workloads.random_relation(rng, lb, upper, ext, til, "f32", 1.0 if whole == "v" else 0.7)
    spec = workloads.spec(e, upper, ext, til, "f32")
    plan, out = gpu_run(spec, U, V, small_join=small)
    check(out, orc.run(orc.Plan(e, upper, ext, til), U, V), "f32")
    # the driving relation's keys are checked on the way
    drives = V if whole == "u" else U
    for status, edit in (("TRE_E_KEYRANGE", lambda k: k[len(k) // 2].__setitem__(0, 10 ** 6)),
                         ("TRE_E_DUPKEY", lambda k: k.__setitem__(5, k[4])),
                         ("TRE_E_UNSORTED", lambda k: k.__setitem__([5, 6], k[[6, 5]]))):
        bad = dict(drives, keys=drives["keys"].copy())
        edit(bad["keys"])
        a, b = (to_dev(U), to_dev(bad)) if whole == "u" else (to_dev(bad), to_dev(V))
        with pytest.raises(tre.TreError) as err:
            tre.einsum(plan, *a, *b)
        assert err.value.status == status
    torch.cuda.synchronize()
