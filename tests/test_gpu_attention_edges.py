"""Attention kernels at the edges of their tiles, key parts and key splits,
against float64 rows on the CPU.  Tolerances are the parity tests': rel-L2
1e-5 in fp32 (sums of d and n terms of 2^-24 each stay far below it) and 2e-2
in bf16 (2^-9 of the rounded probabilities and output)."""
import math

import numpy as np
import pytest

from tests._common import medium, rel_l2
from tests.test_gpu_parity import _replay, _run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dense64(q, k, v):
    s = (q.double() @ k.double().transpose(-1, -2)) / math.sqrt(q.shape[-1])
    return torch.softmax(s, -1) @ v.double()


# one key; fewer keys than one tile, than one tile per key part; one and two
# 32-row sets; ragged last tiles on either side of a tile edge
@pytest.mark.parametrize("n", [1, 31, 33, 64, 97, 129, 256, 321, 1000])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("heads,kv", [(2, 2), (3, 1)])
def test_dense_attention_edges(n, dtype, d, heads, kv):
    from paper_2608_18484_amd import sparsepr as S
    g = torch.Generator().manual_seed(n * 7 + d)
    q, k, v = (torch.randn(2, h, n, d, generator=g) for h in (heads, kv, kv))
    if dtype == "bf16":
        q, k, v = (x.bfloat16() for x in (q, k, v))
    got = S.dense_attention(q.cuda(), k.cuda(), v.cuda()).cpu().double()
    rep = heads // kv
    ref = _dense64(q, k.repeat_interleave(rep, 1), v.repeat_interleave(rep, 1))
    assert rel_l2(got, ref) < (1e-5 if dtype == "f32" else 2e-2)


# the block orders of the bf16 kernel (head counts divisible by 8 and not) at
# both of its block sizes, with a short last tile of rows and of keys; launches
# of many heads with one to seven 64-row tiles, where the block size changes
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("batch,heads,kv,n", [(1, 8, 8, 77), (3, 5, 5, 4400), (2, 12, 3, 2800),
                                              (40, 16, 8, 33), (40, 16, 16, 65), (24, 16, 2, 130),
                                              (24, 13, 13, 256), (12, 16, 4, 300), (9, 16, 16, 400)])
def test_dense_attention_block_orders(d, batch, heads, kv, n):
    from paper_2608_18484_amd import sparsepr as S
    g = torch.Generator().manual_seed(n + d)
    q, k, v = (torch.randn(batch, h, n, d, generator=g).bfloat16() for h in (heads, kv, kv))
    got = S.dense_attention(q.cuda(), k.cuda(), v.cuda()).cpu().double()
    rows = torch.tensor([0, 31, min(63, n - 1), n // 2, n - 1])
    rep = heads // kv
    ref = _dense64(q[:, :, rows], k.repeat_interleave(rep, 1), v.repeat_interleave(rep, 1))
    assert rel_l2(got[:, :, rows], ref) < 2e-2


# base pointers aligned only to an element: fp32 Q, K, V and output, and a bf16
# output, one element into their allocation
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_attention_one_element_into_an_allocation(dtype, d):
    from paper_2608_18484_amd import sparsepr as S
    g = torch.Generator().manual_seed(d)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v = (torch.randn(1, 2, 513, d, generator=g).to(dt).cuda() for _ in range(3))

    def shifted(t):
        return torch.empty(t.numel() + 1, dtype=dt, device="cuda")[1:].view(t.shape).copy_(t)

    inputs = [shifted(x) for x in (q, k, v)] if dtype == "f32" else (q, k, v)
    assert torch.equal(S.dense_attention(*inputs, out=shifted(q)), S.dense_attention(q, k, v))
    if dtype == "f32":
        p = S.default_params(n_kv_groups=9, n_q_groups=9, n_probes=70, target_exec_density=0.5)
        outs = []
        for x in (inputs, (q, k, v)):
            op = S.SparsePR(S.shape_of(q), p)
            outs.append(op(*x, out=torch.empty_like(q)))
        assert torch.equal(*outs)


# probe rows over key splits: the last split short, one and two tiles of
# probes, more splits than the shortest split allows at this length
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("grid,m", [((1, 11, 13), 5), ((2, 23, 29), 33), ((3, 24, 31), 70)])
def test_probe_rows_and_output_over_short_splits(orc, dtype, grid, m):
    wl = medium(grid=grid, heads=2, dtype=dtype, n_probes=m)
    r = _run(wl)
    tol = 1e-5 if dtype == "f32" else 2e-2
    for h in range(2):
        ex = r["op"].export(h, fields=["labels_q", "labels_kv", "routes", "probes", "probe_weights",
                                       "o_dense_probes", "o_sparse"])
        q, k, v = (torch.from_numpy(r[x][0, h]) for x in "qkv")
        ref = _dense64(q[ex["probes"].astype(np.int64)], k, v)
        assert rel_l2(ex["o_dense_probes"], ref) < tol
        out, _ = _replay(orc, r, ex, 0, h)
        assert rel_l2(r["out"][0, h], out) < tol


# a bf16 launch of 384 blocks or more keeps whole 2,048-key splits: with one
# split a probe row is the dense kernel's row (the same key tiles, maxima and
# rounded probabilities) up to the division's last float bit, which rarely
# shows in bf16, while shorter splits round the probabilities against other
# maxima and move about half of the elements
def test_probe_rows_of_a_full_launch_are_not_split():
    from paper_2608_18484_amd import sparsepr as S
    g = torch.Generator().manual_seed(5)
    q, k, v = (torch.randn(16, 24, 1024, 128, generator=g).bfloat16().cuda() for _ in range(3))
    op = S.SparsePR(S.shape_of(q), S.default_params(n_kv_groups=16, n_q_groups=16, n_probes=32,
                                                    target_exec_density=0.25))
    op(q, k, v)
    dense = S.dense_attention(q, k, v)
    same = total = 0
    for bh in (0, 100, 383):
        ex = op.export(bh, fields=["probes", "o_dense_probes"])
        rows = dense[bh // 24, bh % 24].cpu()[torch.from_numpy(ex["probes"].astype(np.int64))]
        eq = torch.from_numpy(ex["o_dense_probes"]).bfloat16() == rows
        same, total = same + int(eq.sum()), total + eq.numel()
    assert same >= 0.999 * total


# keys whose scores are all -inf (a channel that no query leaves out) add
# nothing wherever they lie: the first, a later and the last tile, whole key
# parts and whole key splits
def _masked(n, lo, hi, dtype, d, heads):
    g = torch.Generator().manual_seed(n + d)
    q, k, v = (torch.randn(1, heads, n, d, generator=g) for _ in range(3))
    q[..., 0] = q[..., 0].abs() + 0.1
    k[:, :, lo:hi, 0] = -math.inf
    return (x.bfloat16() for x in (q, k, v)) if dtype == "bf16" else (q, k, v)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,lo,hi", [(256, 0, 32), (256, 32, 64), (256, 96, 128), (700, 640, 700)])
def test_dense_attention_with_keys_at_minus_infinity(dtype, d, n, lo, hi):
    from paper_2608_18484_amd import sparsepr as S
    q, k, v = _masked(n, lo, hi, dtype, d, 2)
    got = S.dense_attention(q.cuda(), k.cuda(), v.cuda()).cpu().double()
    assert rel_l2(got, _dense64(q, k, v)) < (1e-5 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lo", [0, 256])
def test_attend_with_keys_at_minus_infinity(dtype, d, lo):
    from paper_2608_18484_amd import sparsepr as S
    n, c = 1024, 16
    q, k, v = _masked(n, lo, lo + 256, dtype, d, 1)
    op = S.SparsePR(S.shape_of(q), S.default_params(n_kv_groups=c, n_q_groups=c, n_probes=32,
                                                    resid_rank=4, target_exec_density=1.0))
    lab = (np.arange(n) // 64).astype(np.int32)
    op.import_plan(0, lab, lab, np.ones((c, c), np.uint8), np.arange(16, n, 32, dtype=np.int32))
    out = torch.empty_like(q, device="cuda")
    op.attend(q.cuda(), k.cuda(), v.cuda(), out)
    ref = _dense64(q, k, v)[0, 0]
    ex = op.export(0, fields=["o_sparse", "o_dense_probes", "probes"])
    tol = 1e-5 if dtype == "f32" else 2e-2
    assert rel_l2(ex["o_dense_probes"], ref[ex["probes"].astype(np.int64)]) < tol
    assert rel_l2(ex["o_sparse"], ref) < tol


# the eigensolver's own convergence: a basis of every dimension (d = 64 keeps
# r_Q = d directions, down to the noise floor's close eigenvalues) comes from
# the tridiagonal solver, in both precisions, and the fit from few and many
# directions (1, one past a lane group's 16, d).  Ranks that reach eigenvalues
# below 1e-5 of the largest are left to Jacobi in double by design.
@pytest.mark.parametrize("dtype,d,rank", [("f32", 64, 1), ("bf16", 64, 17), ("f32", 128, 17),
                                          ("bf16", 128, 1), ("f32", 128, 100), ("bf16", 128, 100),
                                          ("f32", 64, 64)])
def test_eigensolver_without_jacobi_and_fit_ranks(orc, dtype, d, rank):
    from paper_2608_18484_amd import sparsepr as S
    wl = medium(grid=(3, 16, 24), heads=2, dtype=dtype, d=d, n_probes=140, resid_rank=rank)
    r = _run(wl)
    if rank <= 17:
        assert not r["op"].stats()["status_flags"] & S.FLAG_EIG_JACOBI
    for h in range(2):
        ex = r["op"].export(h, fields=["labels_q", "labels_kv", "routes", "probes", "probe_weights",
                                       "fit_bpsi", "fit_psi"])
        out, fit = _replay(orc, r, ex, 0, h)
        g = ex["fit_bpsi"].astype(np.float64) @ ex["fit_psi"].T.astype(np.float64)
        assert rel_l2(r["out"][0, h], out) < (1e-5 if dtype == "f32" else 2e-2)
        if dtype == "f32":
            assert rel_l2(g, fit["g"]) < 1e-4


# residuals far from 1: the float solver of the bf16 d = 128 basis squares the
# entries of Rbar^T W Rbar and of its rounding noise, so V near 1e-5 (noise
# below the float range) or 1e10 (squares above it) shows whether the matrix is
# brought into range first; the double ones only meet their float eigenvalue
# search there
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("rank", [1, 16])
@pytest.mark.parametrize("e", [-40, -30, -20, -17, 31, 36, 45])
def test_fit_of_small_and_large_values(orc, dtype, d, rank, e):
    from paper_2608_18484_amd import sparsepr as S
    from paper_2608_18484_amd import workloads as W
    wl = medium(grid=(3, 16, 24), heads=1, dtype=dtype, d=d, n_probes=64, resid_rank=rank)
    q, k, v, _ = W.make_inputs(wl)
    r = _run(wl, inputs=(q, k, v * np.float32(2.0) ** e))
    ex = r["op"].export(0)
    assert ex["fit_rank"] == rank
    assert not r["op"].stats()["status_flags"] & S.FLAG_EIG_JACOBI
    ref, _ = _replay(orc, r, ex, 0, 0)
    # bf16: 2^-9 of the rounded probabilities and as much of the output, where
    # the correction is 1.4e-2 of it
    assert rel_l2(r["out"][0, 0], ref) < (1e-5 if dtype == "f32" else 2.0 ** -8)


# the fit's map keeps the double basis up to its only rounding: Y is the float
# nearest to the fp64 solution on the same sparse and probe rows (a basis
# rounded to float first moves a fifth of the elements by a float step)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rank", [1, 8])
def test_fit_map_is_rounded_once(d, rank):
    from paper_2608_18484_amd import workloads as W
    wl = medium(grid=(4, 16, 24), heads=1, dtype="f32", d=d, n_probes=300, resid_rank=rank,
                density=0.4)
    q, k, v, _ = W.make_inputs(wl)
    v = np.random.default_rng(1).standard_normal(v.shape).astype(np.float32)
    r = _run(wl, inputs=(q, k, v))
    ex = r["op"].export(0)
    x = ex["o_sparse"].astype(np.float64)[ex["probes"]]
    res = ex["o_dense_probes"].astype(np.float64) - x
    w = ex["probe_weights"].astype(np.float64)
    m, al = len(w), (w / w.sum())[:, None]
    mx = (al * x).sum(0)
    xb = (x - mx) / np.sqrt((al * (x - mx) ** 2).sum(0) + float(np.float32(1e-6)))
    rb = res - (al * res).sum(0)
    psi = np.linalg.eigh(rb.T @ (m * al * rb))[1][:, ::-1][:, :rank]
    y = np.linalg.solve(xb.T @ (m * al * xb) + float(np.float32(wl.ridge)) * np.eye(d),
                        xb.T @ (m * al * (rb @ psi)))
    y *= np.sign((psi * ex["fit_psi"]).sum(0))
    assert np.mean(ex["fit_bpsi"] == y.astype(np.float32)) > 0.99


# one probe leaves no residual about the mean: the basis has rank 0, without the
# Jacobi solver, and the correction is the probe's residual
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("rank", [1, 16])
def test_fit_of_one_probe(orc, dtype, d, rank):
    from paper_2608_18484_amd import sparsepr as S
    wl = medium(grid=(3, 16, 24), heads=1, dtype=dtype, d=d, n_probes=1, resid_rank=rank)
    r = _run(wl)
    ex = r["op"].export(0)
    assert not r["op"].stats()["status_flags"] & S.FLAG_EIG_JACOBI
    assert ex["fit_rank"] == 0
    assert np.all(ex["fit_psi"] == 0.0) and np.all(ex["fit_bpsi"] == 0.0)
    ref, _ = _replay(orc, r, ex, 0, 0)
    assert rel_l2(r["out"][0, 0], ref) < (1e-5 if dtype == "f32" else 2e-2)


# a ridge matrix that is not positive definite: a channel of V that is zero
# leaves its row and column of the unregularised matrix exactly zero, whatever
# the other pivots are (noise with fewer probes than dimensions, positive with
# more).  The flag is raised and the correction is the mean residual.
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("probes,channel", [(9, 0), (200, 0), (200, 37), (200, -1)])
def test_fit_not_positive_definite(dtype, d, probes, channel):
    from paper_2608_18484_amd import sparsepr as S
    from paper_2608_18484_amd import workloads as W
    wl = medium(grid=(2, 16, 24), heads=1, dtype=dtype, d=d, n_probes=probes, resid_rank=4,
                density=0.5, ridge=0.0)
    q, k, v, _ = W.make_inputs(wl)
    v[..., channel] = 0.0
    r = _run(wl, inputs=(q, k, v))
    assert r["op"].stats()["status_flags"] & S.FLAG_FIT_NOT_PD
    ex = r["op"].export(0)
    assert np.all(ex["fit_bpsi"] == 0.0)
    out = r["out"][0, 0]
    assert np.isfinite(out).all()
    ref = ex["o_sparse"] + ex["fit_mu_r"]
    ref[ex["probes"]] = ex["o_dense_probes"]
    if dtype == "bf16":
        ref = torch.from_numpy(ref).bfloat16().float().numpy()
    assert np.array_equal(out, ref)
