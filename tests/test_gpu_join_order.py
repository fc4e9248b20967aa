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
