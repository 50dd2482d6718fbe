"""Planning kernels where their forms change over: the one-block sort (and its
centroid update) against the three-kernel sort, the one-block selection against
the multi-launch one, and the row chunks of the projection and the correction.
Every stage is compared with the oracle as in the parity tests (labels,
centroids, permutations, group means, routes and probes bit-exact)."""
import pytest

from tests._common import medium, rel_l2
from tests.test_gpu_parity import _replay, _run, _stagewise

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


# rows: below one wave, a wave's slice and its edges, the most the one-block
# sort takes and one more; groups: one, two per wave (the most whose update is
# fused) and one more, one per row, more than the one-block sort's LDS holds;
# cells: the one-block selection's most (128 x 128) and one column more
@pytest.mark.parametrize("grid,ck,cq,dtype,d", [
    ((1, 5, 7), 1, 1, "f32", 64),
    ((1, 9, 7), 63, 5, "bf16", 64),
    ((2, 16, 31), 32, 33, "bf16", 128),
    ((1, 41, 25), 17, 64, "f32", 128),
    ((8, 32, 32), 128, 128, "bf16", 64),
    ((1, 3, 2731), 129, 128, "bf16", 64),
    ((2, 32, 32), 900, 831, "bf16", 64),
])
def test_plan_stages_at_changeovers(orc, grid, ck, cq, dtype, d):
    wl = medium(grid=grid, heads=2, dtype=dtype, d=d, n_kv_groups=ck, n_q_groups=cq, n_probes=8,
                resid_rank=4, density=0.4)
    r = _run(wl)
    for h in range(2):
        ex = _stagewise(orc, r, 0, h)
        ref, _ = _replay(orc, r, ex, 0, h)
        assert rel_l2(r["out"][0, h], ref) < (1e-5 if dtype == "f32" else 2e-2)


# budgets of the one-block selection: below the forced cells, exactly nothing
# more, and everything
@pytest.mark.parametrize("density", [1e-3, 0.07, 1.0])
def test_small_selection_budgets(orc, density):
    wl = medium(grid=(2, 17, 23), heads=2, n_probes=4, resid_rank=4, density=density)
    r = _run(wl)
    for h in range(2):
        _stagewise(orc, r, 0, h)
