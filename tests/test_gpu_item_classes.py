"""Sparse attention in two classes of work items (blocks of three and of two
waves), which only launches of many rows take, on imported plans: one, three and
eight K/V heads (both block orders) shared by several query heads, several key
segments, query groups of every split into 32-row sets, one K/V head without an
item of the first class.  Rows are compared with float64 rows on the CPU, and
bit by bit with the same plans in a launch too small for classes: an item's
waves compute the same in blocks of either size."""
import math

import numpy as np
import pytest

from tests._common import rel_l2

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 28032
# rows of the query groups (repeated to N): one to four sets and their edges
SIZES = [64, 65, 96, 97, 128, 129, 1, 32, 33, 160, 161, 192, 193, 63, 31, 256, 300]


def _sizes(sizes, n):
    out = []
    while sum(out) < n:
        out.append(min(sizes[len(out) % len(sizes)], n - sum(out)))
    return np.array(out)


def _plan(rng, sizes, c):
    """Labels in random row order, a third of the cells, and a group routed to
    every key beside one routed to a single key group."""
    lab_q = np.repeat(np.arange(len(sizes)), sizes)
    lab_k = np.sort(rng.integers(0, c, N))
    lab_q, lab_k = rng.permutation(lab_q), rng.permutation(lab_k)
    z = (rng.random((c, c)) < 0.3).astype(np.uint8)
    z[3] = 1
    z[5] = 0
    z[np.arange(c), rng.integers(0, c, c)] = 1
    z[:, np.bincount(lab_k, minlength=c) == 0] = 0
    z[np.arange(c), lab_k[rng.integers(0, N, c)]] = 1
    return lab_q.astype(np.int32), lab_k.astype(np.int32), z


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kv,group", [(1, 32), (3, 11), (8, 4)])
def test_item_classes(monkeypatch, d, kv, group):
    from paper_2608_18484_amd import sparsepr as S
    monkeypatch.setenv("SPARSEPR_SEG_KB", str(N * d * 4 // 1024 // 3 + 1))  # three segments
    rng = np.random.default_rng(d + kv)
    g = torch.Generator(device="cuda").manual_seed(d + kv)
    q = torch.randn(1, kv * group, N, d, generator=g, device="cuda").bfloat16()
    k, v = (torch.randn(1, kv, N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    c = -(-N // 64)
    # the last K/V head of several has no group of more than two sets
    plans = [_plan(rng, _sizes([64] if kv > 1 and h == kv - 1 else SIZES, N), c) for h in range(kv)]
    p = S.default_params(n_kv_groups=c, n_q_groups=c, n_probes=0, target_exec_density=1.0)

    def run(q, k, v, plans):
        per = q.shape[1] // k.shape[1]
        op = S.SparsePR(S.shape_of(q, kv=k if per > 1 else None), p)
        for h, (lq, lk, z) in enumerate(plans):
            op.import_plan(h * per, lq, lk, z, np.zeros(0, np.int32))
        out = torch.empty_like(q)
        op.attend(q, k, v, out)
        return op

    assert q.shape[1] * N >= 14000 * 64  # takes classes
    op = run(q, k, v, plans)
    heads = [0, kv * group - 1] if kv == 1 else [0, group + group // 2, kv * group - 1]
    for bh in heads:
        h = bh // group
        got = op.export(bh, fields=["o_sparse"])["o_sparse"]
        one = run(q[:, bh:bh + 1].contiguous(), k[:, h:h + 1].contiguous(),
                  v[:, h:h + 1].contiguous(), [plans[h]])
        assert np.array_equal(got, one.export(0, fields=["o_sparse"])["o_sparse"])
        lq, lk, z = plans[h]
        rows = np.sort(rng.choice(N, 400, replace=False))
        s = (q[0, bh].double().cpu()[torch.from_numpy(rows)] @ k[0, h].double().cpu().T) / math.sqrt(d)
        mask = torch.from_numpy(z[lq[rows]][:, lk] != 0)
        ref = torch.softmax(s.masked_fill(~mask, -math.inf), -1) @ v[0, h].double().cpu()
        assert rel_l2(got[rows], ref) < 1e-2  # 2^-9 of the rounded probabilities
