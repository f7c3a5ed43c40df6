"""GPU parity of the building blocks against the oracle, through the C ABI.

Tolerances (FP64, u = 2^-53):
* random matrices: the same Philox words on both sides; the Box-Muller
  log/sqrt/cos/sin may differ by a few ulps -> |diff| <= 1e-14 max(1, |z|);
* sampling: a dot product of length K has error <= gamma_K |A||R| with
  gamma_K = K u / (1 - K u) in any summation order, so two correct
  implementations differ by at most 2 gamma_K (|A||R|) entrywise;
* ID: inputs with well separated column norms have unique pivots -> J and k
  equal exactly; E = (R1^{-1} R2)^T agrees to 1e-10 relative (the QR
  factors differ by rounding, amplified by cond(R1)).
"""
import os
import re

import numpy as np
import pytest
import torch

import paper_1503_05464_amd as P
import workloads as W
from oracle import hss as ohss
from oracle import interp, philox
from oracle.tree import bisection_tree

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _gamma(k):
    return k * U / (1 - k * U)


@pytest.mark.parametrize("n,c0,c1", [(1, 0, 1), (1001, 3, 70), (4096, 0, 128), (777, 64, 96)])
def test_random_normal_matches_oracle(n, c0, c1):
    print(f"random_normal n={n} cols=[{c0},{c1})", flush=True)
    for which in (0, 1):
        g = P.hss_random_normal(7, which, n, c0, c1).cpu().numpy()
        ref = philox.gaussian_columns(7, which, n, c0, c1)
        assert np.all(np.abs(g - ref) <= 1e-14 * np.maximum(1.0, np.abs(ref)))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n,ncols,masked", [(1000, 64, False), (1000, 100, True), (2048, 128, True),
                                            (300, 7, True), (4500, 64, False)])
def test_sample_matches_oracle(dtype, n, ncols, masked):
    print(f"sample n={n} ncols={ncols} masked={masked} dtype={dtype}", flush=True)
    g = np.random.default_rng(n + ncols)
    A = W.toeplitz_inverse_distance(n) + 0.3 * g.standard_normal((n, n)) / np.sqrt(n)
    A = A.astype(np.float32 if dtype == torch.float32 else np.float64)
    A64 = A.astype(np.float64)
    Rr = g.standard_normal((n, ncols))
    Rc = g.standard_normal((n, ncols))
    Ad = torch.from_numpy(A).cuda()
    tree = bisection_tree(n, 64)
    leaf_of = None
    if masked:
        lo = np.zeros(n, dtype=np.int32)
        for q, t in enumerate(sorted(tree.leaves(), key=lambda t: tree.lo[t])):
            lo[tree.lo[t]:tree.hi[t]] = q
        leaf_of = torch.from_numpy(lo).cuda()
    Sr, Sc = P.hss_sample(Ad, torch.from_numpy(Rr).cuda(), torch.from_numpy(Rc).cuda(), leaf_of)
    torch.cuda.synchronize()
    ref_r, ref_c = ohss.sample(A64, Rr, Rc)
    absA = np.abs(A64)
    if masked:
        ref_r, ref_c = ohss.leaf_local_samples(A64, tree, ref_r, ref_c, Rr, Rc)
    bound_r = 2 * _gamma(n) * (absA @ np.abs(Rr)) + 1e-300
    bound_c = 2 * _gamma(n) * (absA.T @ np.abs(Rc)) + 1e-300
    # the masked oracle subtracts D R afterwards: add that product's error too
    if masked:
        bound_r *= 2
        bound_c *= 2
    assert np.all(np.abs(Sr.cpu().numpy() - ref_r) <= bound_r)
    assert np.all(np.abs(Sc.cpu().numpy() - ref_c) <= bound_c)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n,ncols", [(511, 64), (512, 1), (513, 65), (1025, 64), (2047, 130), (8191, 3)])
def test_sample_split_edges(dtype, n, ncols):
    """Sizes at the edges of the rule that splits K over workgroups, against
    the product in FP64 on the host (bound as above), and the same bits from
    a second call."""
    g = np.random.default_rng(n + ncols)
    A = g.standard_normal((n, n)).astype(np.float32 if dtype == torch.float32 else np.float64)
    Rr, Rc = g.standard_normal((2, n, ncols))
    args = [torch.from_numpy(a).cuda() for a in (A, Rr, Rc)]
    print(f"sample split: n={n} ncols={ncols} {dtype}", flush=True)
    Sr, Sc = P.hss_sample(*args)
    again = P.hss_sample(*args)
    assert torch.equal(Sr, again[0]) and torch.equal(Sc, again[1])
    A64 = A.astype(np.float64)
    assert np.all(np.abs(Sr.cpu().numpy() - A64 @ Rr) <= 2 * _gamma(n) * (np.abs(A64) @ np.abs(Rr)))
    assert np.all(np.abs(Sc.cpu().numpy() - A64.T @ Rc) <= 2 * _gamma(n) * (np.abs(A64).T @ np.abs(Rc)))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [1, 3, 7, 15, 17, 33, 127, 129, 255, 383, 510])
def test_sample_small_matrices(dtype, n):
    """Matrices below the line of the K split, around the pieces of 16 and 64
    bytes, the slices and the tiles, rows on any entry, NaN beside and below
    the matrix: against the product in FP64 on the host (bound as above)."""
    g = np.random.default_rng(n)
    pad = np.full((n + 1, n + 3), np.nan, dtype=np.float32 if dtype == torch.float32 else np.float64)
    pad[:n, :n] = g.standard_normal((n, n))
    A64 = pad[:n, :n].astype(np.float64)
    lo = np.arange(n, dtype=np.int32) // 20
    A64[lo[:, None] == lo[None, :]] = 0.0
    Rr, Rc = g.standard_normal((2, n, 5))
    print(f"small sample: n={n} {dtype}", flush=True)
    Sr, Sc = P.hss_sample(torch.from_numpy(pad).cuda()[:n, :n], torch.from_numpy(Rr).cuda(),
                          torch.from_numpy(Rc).cuda(), leaf_of=torch.from_numpy(lo).cuda())
    assert np.all(np.abs(Sr.cpu().numpy() - A64 @ Rr) <= 2 * _gamma(n) * (np.abs(A64) @ np.abs(Rr)))
    assert np.all(np.abs(Sc.cpu().numpy() - A64.T @ Rc) <= 2 * _gamma(n) * (np.abs(A64).T @ np.abs(Rc)))


@pytest.mark.parametrize("prec,terms", [("f32", 1), ("bf16x3", 3)])
@pytest.mark.parametrize("n,ncols", [(767, 64), (768, 1), (1025, 65), (4097, 64)])
def test_sample_mixed_split_edges(prec, terms, n, ncols):
    """The reduced modes at the edges of their rule for splitting K: FP32
    sums over at most 256 values of k (three exact terms each in BF16x3),
    carried in FP64, so an entry errs by at most (256 terms + 8) 2^-24 of
    |A||R|; a second call gives the same bits."""
    A = torch.randn(n, n, dtype=torch.float32, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    Rr = P.hss_random_normal(3, 0, n, 0, ncols, sample_prec=prec)
    Rc = P.hss_random_normal(3, 1, n, 0, ncols, sample_prec=prec)
    print(f"sample split: n={n} ncols={ncols} {prec}", flush=True)
    got = P.hss_sample(A, Rr, Rc, sample_prec=prec)
    again = P.hss_sample(A, Rr, Rc, sample_prec=prec)
    for S, S2, B, R in zip(got, again, (A, A.T), (Rr, Rc)):
        assert torch.equal(S, S2)
        B, R = B.double().cpu(), R.cpu()
        assert torch.all((S.cpu() - B @ R).abs() <= (256 * terms + 8) * 2.0 ** -24 * (B.abs() @ R.abs()))


@pytest.mark.parametrize("n", [127, 260, 1157, 2309])
@pytest.mark.parametrize("dtype,prec", [(torch.float64, "f64"), (torch.float32, "f64"), (torch.float32, "f32"),
                                        (torch.float32, "bf16x3")])
def test_sample_any_row_alignment(dtype, prec, n):
    """Rows of A on any entry (odd leading dimensions, a base off the 16-byte
    grid) give the samples of an aligned copy, bit for bit: the same products
    summed in the same order."""
    kw = {} if prec == "f64" else {"sample_prec": prec}
    big = torch.randn(n, n + 9, dtype=dtype, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    lo = torch.arange(n, dtype=torch.int32, device="cuda") // 60
    Rr = P.hss_random_normal(5, 0, n, 0, 70, **kw)
    Rc = P.hss_random_normal(5, 1, n, 0, 70, **kw)
    for off, lda in ((0, n + 9), (1, n + 9), (3, n + 8), (2, n + 7)):
        A = torch.as_strided(big, (n, n), (lda, 1), off)
        pad = torch.zeros(n, (n + 15) // 4 * 4, dtype=dtype, device="cuda")
        pad[:, :n] = A
        print(f"sample alignment: n={n} lda={lda} offset={off} {dtype} {prec}", flush=True)
        got = P.hss_sample(A, Rr, Rc, leaf_of=lo, **kw)
        ref = P.hss_sample(pad[:, :n], Rr, Rc, leaf_of=lo, **kw)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def _separated(d, m, seed, rank=None):
    g = np.random.default_rng(seed)
    y = g.standard_normal((d, m))
    if rank is not None:
        y = g.standard_normal((d, rank)) @ g.standard_normal((rank, m))
    scale = 2.0 ** (-np.arange(m) * 0.37)
    return y * scale[g.permutation(m)]


@pytest.mark.parametrize("rtol", [1e-2, 1e-6, 1e-12])
def test_id_batched_matches_oracle(rtol):
    cases = [(12, 8, None), (8, 12, None), (64, 300, None), (130, 257, None), (1, 5, None),
             (5, 1, None), (40, 25, 6), (200, 64, None), (3, 3, 0)]
    Ys, refs = [], []
    for q, (d, m, rank) in enumerate(cases):
        y = _separated(d, m, 100 + q, rank) if rank != 0 else np.zeros((d, m))
        refs.append(interp.interpolative_decomposition(y, rtol))
        Ys.append(torch.from_numpy(np.ascontiguousarray(y.T)).cuda())  # rows = columns of Y
    print(f"id_batched rtol={rtol} problems={len(cases)}", flush=True)
    got = P.hss_id_batched(Ys, rtol)
    for (k, perm, E), ref, (d, m, rank) in zip(got, refs, cases):
        assert k == ref.k, (d, m, rank)
        assert list(perm[:k]) == list(ref.J)
        assert list(perm[k:]) == list(ref.rest)
        if E.size:
            assert np.allclose(E, ref.E, rtol=1e-10, atol=1e-10 * max(1.0, np.abs(ref.E).max()))


def test_id_ties_take_lowest_index():
    y = np.eye(6)[:, [3, 1, 5, 0, 2, 4]] * 2.0
    got = P.hss_id_batched([torch.from_numpy(np.ascontiguousarray(y.T)).cuda()], 1e-8)[0]
    ref = interp.interpolative_decomposition(y, 1e-8)
    assert got[0] == ref.k == 6 and list(got[1]) == list(ref.J) == [0, 1, 2, 3, 4, 5]


def _slow_decay(d, m, seed, rate):
    g = np.random.default_rng(seed)
    return g.standard_normal((d, m)) * (2.0 ** (-rate * np.arange(m)))[g.permutation(m)]


@pytest.mark.parametrize("cases", [[(2400, 700, 0.37, 11), (2350, 500, 0.0, 12)],
                                   [(900, 1100, 0.37, 15), (1000, 700, 0.0, 16)],
                                   [(700, 900, 0.37, 13), (650, 600, 0.0, 14)]], ids=["d2400", "d1000", "d700"])
@pytest.mark.parametrize("path", ["auto", "persistent"])
def test_id_batched_variant_problems(path, cases, monkeypatch, capfd):
    """The batch's largest d picks the persistent variant: above 2304 rows
    the one with the most rows per lane, at 1000 rows the 16-rows-per-lane
    one, at 700 rows the 12-rows-per-lane one.  Same checks as below, and
    no bounded wait of a persistent launch gave up (the results would then
    come from the per-step rerun)."""
    if path != "auto":
        monkeypatch.setenv("HSS_QRCP_PATH", path)
    monkeypatch.setenv("HSS_VERBOSE", "1")
    rtol = 1e-6
    Ys, refs, mats = [], [], []
    for d, m, rate, seed in cases:
        y = _slow_decay(d, m, seed, rate)
        mats.append(y)
        refs.append(interp.interpolative_decomposition(y, rtol))
        Ys.append(torch.from_numpy(np.ascontiguousarray(y.T)).cuda())
    print(f"id_batched variant: {len(cases)} problems, d max {max(c[0] for c in cases)}, path {path}", flush=True)
    capfd.readouterr()
    got = P.hss_id_batched(Ys, rtol)
    assert "persistent wait gave up" not in capfd.readouterr().err
    for (k, perm, E), ref, y, (d, m, rate, seed) in zip(got, refs, mats, cases):
        assert abs(k - ref.k) <= 1, (d, m, rate, k, ref.k)
        if rate >= 0.3:
            assert k == ref.k and list(perm[:k]) == list(ref.J)
            assert np.allclose(E, ref.E, rtol=1e-8, atol=1e-8 * max(1.0, np.abs(ref.E).max()))
        J, rest = perm[:k], perm[k:]
        X = np.zeros((k, m))
        X[:, J] = np.eye(k)
        if len(rest):
            X[:, rest] = E.T
        nu1 = np.linalg.norm(y, axis=0).max()
        err = np.linalg.norm(y - y[:, J] @ X, 2)
        assert err <= 10 * np.sqrt(max(1, m - k)) * rtol * nu1, (d, m, err)


_TALL_CASES = [(3300, 600, 0.37, 21), (4300, 400, 0.0, 22), (2700, 600, 0.02, 23)]


@pytest.fixture(scope="module")
def tall_refs():
    mats = [_slow_decay(d, m, seed, rate) for d, m, rate, seed in _TALL_CASES]
    return mats, [interp.interpolative_decomposition(y, 1e-6) for y in mats]


@pytest.mark.parametrize("path", ["auto", "step"])
def test_id_batched_tall_problems(path, tall_refs, monkeypatch):
    """Problems taller than the persistent kernel holds (d above 2560 rows)
    run one launch per pivot step.  While more than 4096 rows are active
    the general loop runs, after that the register variants up to 64 rows
    per lane; the 4300-row full-rank case crosses from one to the other.
    Same checks as above."""
    if path != "auto":
        monkeypatch.setenv("HSS_QRCP_PATH", path)
    rtol = 1e-6
    mats, refs = tall_refs
    Ys = [torch.from_numpy(np.ascontiguousarray(y.T)).cuda() for y in mats]
    print(f"id_batched tall: {len(mats)} problems, path {path}", flush=True)
    got = P.hss_id_batched(Ys, rtol)
    for (k, perm, E), ref, y, (d, m, rate, seed) in zip(got, refs, mats, _TALL_CASES):
        assert abs(k - ref.k) <= 1, (d, m, rate, k, ref.k)
        if rate >= 0.3:  # separated norms: the same pivots and interpolation matrix
            assert k == ref.k and list(perm[:k]) == list(ref.J)
            assert np.allclose(E, ref.E, rtol=1e-8, atol=1e-8 * max(1.0, np.abs(ref.E).max()))
        J, rest = perm[:k], perm[k:]
        X = np.zeros((k, m))
        X[:, J] = np.eye(k)
        if len(rest):
            X[:, rest] = E.T
        nu1 = np.linalg.norm(y, axis=0).max()
        err = np.linalg.norm(y - y[:, J] @ X, 2)
        assert err <= 10 * np.sqrt(max(1, m - k)) * rtol * nu1, (d, m, err)


@pytest.mark.parametrize("path", ["auto", "step", "persistent"])
def test_id_batched_large_problems(path, monkeypatch, capfd):
    """Problems on the large-problem paths (one launch per pivot step, or
    persistent launches with the columns in registers; "auto" lets the cost
    model choose): d up to 2100 rows, several workgroups per problem, more
    problems than are resident at once, and one full-rank factorization of 900
    pivot steps.  Pivots agree with the oracle while the norms are well
    separated; everywhere the rank agrees and the ID reproduces Y to its
    tolerance; no bounded wait of a persistent launch gave up."""
    if path != "auto":
        monkeypatch.setenv("HSS_QRCP_PATH", path)
    monkeypatch.setenv("HSS_VERBOSE", "1")
    rtol = 1e-6
    cases = [(2100, 1100, 0.37, 1), (2100, 1100, 0.37, 2), (2100, 1100, 0.37, 3),
             (2100, 1100, 0.37, 4), (2100, 1100, 0.37, 5), (1000, 900, 0.0, 6),
             (700, 1500, 0.02, 7)]
    Ys, refs, mats = [], [], []
    for d, m, rate, seed in cases:
        y = _slow_decay(d, m, seed, rate)
        mats.append(y)
        refs.append(interp.interpolative_decomposition(y, rtol))
        Ys.append(torch.from_numpy(np.ascontiguousarray(y.T)).cuda())
    print(f"id_batched large: {len(cases)} problems, path {path}", flush=True)
    capfd.readouterr()
    got = P.hss_id_batched(Ys, rtol)
    assert "persistent wait gave up" not in capfd.readouterr().err
    for (k, perm, E), ref, y, (d, m, rate, seed) in zip(got, refs, mats, cases):
        assert abs(k - ref.k) <= 1, (d, m, rate, k, ref.k)
        if rate >= 0.3:  # separated norms: the same pivots and interpolation matrix
            assert k == ref.k and list(perm[:k]) == list(ref.J)
            assert np.allclose(E, ref.E, rtol=1e-8, atol=1e-8 * max(1.0, np.abs(ref.E).max()))
        J, rest = perm[:k], perm[k:]
        X = np.zeros((k, m))
        X[:, J] = np.eye(k)
        if len(rest):
            X[:, rest] = E.T
        nu1 = np.linalg.norm(y, axis=0).max()
        err = np.linalg.norm(y - y[:, J] @ X, 2)
        assert err <= 10 * np.sqrt(max(1, m - k)) * rtol * nu1, (d, m, err)


def test_persistent_give_up_reruns_on_step_path(monkeypatch, capfd):
    """When a persistent launch's bounded wait gives up (forced here from the
    host: every workgroup leaves at its first wait, so every kernel exits
    normally), the problems are factored again on the per-step path from
    their untouched inputs: the IDs equal those of the step path itself,
    exactly, and match the oracle as above."""
    rtol = 1e-6
    cases = [(2100, 1100, 0.37, 11), (2100, 1100, 0.37, 12), (1000, 900, 0.0, 13)]
    mats = [_slow_decay(d, m, seed, rate) for d, m, rate, seed in cases]
    Ys = [torch.from_numpy(np.ascontiguousarray(y.T)).cuda() for y in mats]
    monkeypatch.setenv("HSS_QRCP_PATH", "step")
    print("id_batched give-up: step path reference", flush=True)
    ref_step = P.hss_id_batched(Ys, rtol)
    monkeypatch.setenv("HSS_QRCP_PATH", "persistent")
    monkeypatch.setenv("HSS_QRCP_GIVE_UP", "1")
    monkeypatch.setenv("HSS_VERBOSE", "1")
    capfd.readouterr()
    print("id_batched give-up: persistent launch that gives up", flush=True)
    got = P.hss_id_batched(Ys, rtol)
    err = capfd.readouterr().err
    assert "persistent wait gave up" in err, err
    for (k, perm, E), (k0, perm0, E0), y, (d, m, rate, seed) in zip(got, ref_step, mats, cases):
        assert k == k0 and np.array_equal(perm, perm0) and np.array_equal(E, E0)
        ref = interp.interpolative_decomposition(y, rtol)
        assert abs(k - ref.k) <= 1
        if rate >= 0.3:
            assert k == ref.k and list(perm[:k]) == list(ref.J)


@pytest.mark.parametrize("d,m", [(65, 129), (128, 256), (127, 255), (129, 129), (192, 256), (130, 161)])
def test_id_largest_register_classes(d, m):
    """The one-workgroup classes that hold a column in 64 lanes, at the edges
    of their rows and columns: the oracle's pivots where the norms are well
    separated, and the lowest index at exact ties (every column twice)."""
    y = _slow_decay(d, m, d + m, 0.37)
    twice = 2.0 * np.eye(d)[:, np.arange(m) % d]
    got = P.hss_id_batched([torch.from_numpy(np.ascontiguousarray(a.T)).cuda() for a in (y, twice)], 1e-6)
    k, perm, E = got[0]
    ref = interp.interpolative_decomposition(y, 1e-6)
    assert k == ref.k and list(perm[:k]) == list(ref.J)
    assert np.allclose(E, ref.E, rtol=1e-8, atol=1e-8 * max(1.0, np.abs(ref.E).max()))
    k, perm, E = got[1]
    assert k == d and list(perm[:k]) == list(range(d)) and list(perm[k:]) == list(range(d, m))
    assert np.array_equal(E, np.eye(d)[np.arange(d, m) % d])


@pytest.mark.parametrize("k,nrest", [(1, 1), (2, 33), (63, 31), (64, 32), (65, 9), (129, 100)])
def test_id_block_solve_edges(k, nrest):
    """E = (R1^{-1} R2)^T at the edges of the solve's 64-row blocks and of its
    column groups, against a dense solve with the chosen columns (full rank,
    condition below 1e4: 1e-10 relative), and the same entries bit for bit
    when every norm is scaled by 2^505, where the plain division runs."""
    y = _slow_decay(k, k + nrest, 7 * k + nrest, 0.02)
    one, big = P.hss_id_batched([torch.from_numpy(np.ascontiguousarray(y.T) * f).cuda() for f in (1.0, 2.0 ** 505)],
                                1e-14)
    assert one[0] == k
    J, rest = one[1][:k], one[1][k:]
    ref = np.linalg.solve(y[:, J], y[:, rest]).T
    assert np.linalg.norm(one[2] - ref) <= 1e-10 * np.linalg.norm(ref)
    assert big[0] == k and np.array_equal(big[1], one[1]) and np.array_equal(big[2], one[2])


@pytest.mark.parametrize("lo,hi", [(-1074, -1010), (-1010, -940), (-60, -20)])
def test_id_quotients_over_the_exponent_range(lo, hi):
    """Y = [diag(v), T] with v falling and T small: step i's pivot is column
    i, its reflector changes the sign of row i, so that R1 = -diag(v), R2 =
    -T, and E = (R1^{-1} R2)^T holds one correctly rounded quotient per entry,
    whatever its size."""
    g = np.random.default_rng(2000 + lo)
    d, rest = 64, 40
    v = np.linspace(1.9, 1.0, d)
    T = np.ldexp(g.uniform(1.0, 2.0, (d, rest)) * g.choice([-1.0, 1.0], (d, rest)), g.integers(lo, hi, (d, rest)))
    y = np.concatenate([np.diag(v), T], axis=1)
    print(f"ID quotients: 2^{lo} .. 2^{hi}", flush=True)
    k, perm, E = P.hss_id_batched([torch.from_numpy(np.ascontiguousarray(y.T)).cuda()], 1e-14)[0]
    assert k == d and np.array_equal(perm, np.arange(d + rest))
    assert np.array_equal(E, (T / v[:, None]).T)


@pytest.mark.parametrize("d,widest", [(250, 16), (384, 12), (500, 10), (760, 7), (1000, 6), (1270, 4),
                                      (1500, 4), (1790, 3), (2040, 3), (2300, 3), (2500, 2)])
def test_persistent_widths_agree(d, widest, monkeypatch, capfd):
    """Every width (columns per wavefront) of a persistent variant gives the
    same factorization, bit for bit: the width decides only which workgroup
    holds a column.  The cap on workgroups per launch forces each width; the
    ID reproduces Y to its tolerance, as above."""
    m, rtol = 300, 1e-6
    y = _slow_decay(d, m, d, 0.1)
    Y = torch.from_numpy(np.ascontiguousarray(y.T)).cuda()
    monkeypatch.setenv("HSS_QRCP_PATH", "persistent")
    monkeypatch.setenv("HSS_VERBOSE", "2")
    first, seen = None, set()
    for cap in (3, 4, 5, 6, 7, 8, 10, 13, 19, 38):  # ceil(300 / (8 C)) for every C
        monkeypatch.setenv("HSS_QRCP_PERSIST_WG", str(cap))
        capfd.readouterr()
        print(f"persistent widths: d={d}, at most {cap} workgroups", flush=True)
        k, perm, E = P.hss_id_batched([Y], rtol)[0]
        err = capfd.readouterr().err
        assert "persistent wait gave up" not in err
        got = re.findall(r"persistent launch: 1 problems, (\d+) workgroups", err)
        if not got:  # fewer workgroups than the widest needs: the step path
            assert cap < -(-m // (8 * widest))
            continue
        assert int(got[0]) <= cap
        seen.add(int(got[0]))
        if first is None:
            first = (k, perm, E)
        assert k == first[0] and np.array_equal(perm, first[1]) and np.array_equal(E, first[2])
    assert len(seen) >= 2
    k, perm, E = first
    ref = interp.interpolative_decomposition(y, rtol)
    assert abs(k - ref.k) <= 1
    X = np.zeros((k, m))
    X[:, perm[:k]] = np.eye(k)
    X[:, perm[k:]] = E.T
    res = np.linalg.norm(y - y[:, perm[:k]] @ X, 2)
    assert res <= 10 * np.sqrt(max(1, m - k)) * rtol * np.linalg.norm(y, axis=0).max()


def _persistent_widths():
    """{rows per lane: columns per wavefront} of the persistent instantiations."""
    path = os.path.join(os.path.dirname(P.__file__), "csrc", "kernels_qrcp.hip")
    widths = {}
    for t, c in re.findall(r"PV\((\d+), (\d+)\)", open(path).read()):
        widths.setdefault(int(t), []).append(int(c))
    return widths


@pytest.mark.parametrize("T", [4, 6, 8, 12, 16, 20, 24, 28, 32, 36, 40])
def test_persistent_widths_all_run(T, monkeypatch, capfd):
    """Each instantiation of the persistent kernel, by the workgroups that its
    launch reports: a cap of ceil(m / (8 C)) rules out narrower columns than C,
    and wider ones cost more by the model.  m is such that no two widths take
    the same number.  All give the same ID."""
    widths = _persistent_widths()
    assert sorted(widths) == [4, 6, 8, 12, 16, 20, 24, 28, 32, 36, 40]
    m = 300 if T == 4 else 280
    d = 64 * T - 20
    want = [-(-m // (8 * c)) for c in widths[T]]
    assert len(set(want)) == len(want)
    Y = torch.from_numpy(np.ascontiguousarray(_slow_decay(d, m, d, 0.1).T)).cuda()
    monkeypatch.setenv("HSS_QRCP_PATH", "persistent")
    monkeypatch.setenv("HSS_VERBOSE", "2")
    first, seen = None, []
    for cap in want:
        monkeypatch.setenv("HSS_QRCP_PERSIST_WG", str(cap))
        capfd.readouterr()
        k, perm, E = P.hss_id_batched([Y], 1e-6)[0]
        err = capfd.readouterr().err
        assert "persistent wait gave up" not in err
        seen += [int(g) for g in re.findall(r"persistent launch: 1 problems, (\d+) workgroups", err)]
        first = first or (k, perm, E)
        assert k == first[0] and np.array_equal(perm, first[1]) and np.array_equal(E, first[2])
    assert seen == want


@pytest.mark.parametrize("variant", list(range(-1, 7)))
def test_gemm_batched_tile_shapes(variant):
    """The batched FP64 GEMM of every per-node product (Alg. 1-4), in each
    of its tile shapes (variant -1: the tuning table's choice), against the
    FP64 product on the host: a dot product of length K differs from another
    correct one by at most 2 gamma_K |A||B| entrywise; problems cover empty
    K, single rows and columns, ragged edges of every tile and transposed A;
    every shape gives the same bits (the k order of each entry is the same)."""
    if variant >= P.hss_gemm_variants():
        pytest.skip("no such tile shape")
    g = np.random.default_rng(40)
    sizes = [(1, 1, 1, 0), (17, 5, 33, 1), (64, 64, 64, 0), (100, 130, 70, 1), (257, 3, 300, 0),
             (33, 200, 0, 0), (129, 17, 16, 1), (15, 65, 129, 0)]
    As, Bs, Cs, tr, ref, bnd = [], [], [], [], [], []
    alpha, beta = -1.5, 0.5
    for M, N, K, t in sizes:
        A = g.standard_normal((K, M) if t else (M, K))
        B = g.standard_normal((K, N))
        C = g.standard_normal((M, N))
        opA = A.T if t else A
        ref.append(alpha * (opA @ B) + beta * C)
        gam = 2 * K * U / (1 - K * U) if K else 0.0
        bnd.append(gam * abs(alpha) * (np.abs(opA) @ np.abs(B)) + 4 * U * (np.abs(alpha * (opA @ B)) + np.abs(beta * C)))
        As.append(torch.from_numpy(A).cuda())
        Bs.append(torch.from_numpy(B).cuda())
        Cs.append(torch.from_numpy(C).cuda())
        tr.append(bool(t))
    print(f"gemm_batched variant {variant}: {len(sizes)} problems", flush=True)
    out = P.hss_gemm_batched(As, Bs, [c.clone() for c in Cs], tr, alpha, beta, variant)
    base = P.hss_gemm_batched(As, Bs, [c.clone() for c in Cs], tr, alpha, beta, 0)
    torch.cuda.synchronize()
    for o, b0, r, bd in zip(out, base, ref, bnd):
        assert np.all(np.abs(o.cpu().numpy() - r) <= bd + 1e-300)
        assert torch.equal(o, b0)


@pytest.mark.parametrize("K", [15, 511, 512, 513, 1041])
def test_gemm_batched_long_inner_dimensions(K):
    """Inner dimensions around the kernel's chunks of 512 k and its slices of
    16, with leading dimensions beyond the rows and NaN just past every row
    and column that belongs to the product: within 2 gamma_K |A||B| of the
    host's product, and the same bits in every tile shape and in the shape the
    library picks by itself."""
    g = np.random.default_rng(K)
    As, Bs, Cs, tr, ref, bnd = [], [], [], [], [], []
    for M, N, t in [(33, 17, 0), (70, 65, 1), (1, 1, 0), (130, 5, 1)]:
        A = g.standard_normal((K, M) if t else (M, K))
        B, C = g.standard_normal((K, N)), g.standard_normal((M, N))
        opA = A.T if t else A
        ref.append(opA @ B - C)
        bnd.append(2 * _gamma(K) * (np.abs(opA) @ np.abs(B)) + 4 * U * (np.abs(opA @ B) + np.abs(C)))
        pads = [np.full((x.shape[0] + 1, x.shape[1] + 3), np.nan) for x in (A, B, C)]
        views = []
        for pad, x in zip(pads, (A, B, C)):
            pad[:-1, :-3] = x
            views.append(torch.from_numpy(pad).cuda()[:-1, :-3])
        As.append(views[0])
        Bs.append(views[1])
        Cs.append(views[2])
        tr.append(bool(t))
    print(f"gemm_batched K={K}", flush=True)
    first = None
    for v in range(-1, P.hss_gemm_variants()):
        out = P.hss_gemm_batched(As, Bs, [c.clone() for c in Cs], tr, 1.0, -1.0, v)
        torch.cuda.synchronize()
        first = first or out
        for o, f, r, bd in zip(out, first, ref, bnd):
            assert np.all(np.abs(o.cpu().numpy() - r) <= bd)
            assert torch.equal(o, f)


@pytest.mark.parametrize("K", [0, 1, 16, 17, 33, 64])
def test_gemm_batched_short_inner_dimensions(K):
    """Launches of few slices run on kernels with one slice ahead: the same
    bits in every shape as in a launch that one longer product (200 k) sends
    to the others, and within 2 gamma_K |A||B| of the host's product."""
    g = np.random.default_rng(1000 + K)
    As, Bs, Cs, tr, ref, bnd = [], [], [], [], [], []
    for M, N, k, t in [(33, 17, K, 0), (70, 65, K, 1), (1, 1, K // 2, 0), (130, 5, K, 1), (16, 64, 200, 0)]:
        A, B, C = g.standard_normal((k, M) if t else (M, k)), g.standard_normal((k, N)), g.standard_normal((M, N))
        opA = A.T if t else A
        ref.append(0.5 * (opA @ B) - C)
        bnd.append(2 * _gamma(max(k, 1)) * (np.abs(opA) @ np.abs(B)) + 4 * U * (np.abs(opA @ B) + np.abs(C)))
        for xs, x in zip((As, Bs, Cs), (A, B, C)):
            xs.append(torch.from_numpy(x).cuda())
        tr.append(bool(t))
    print(f"gemm_batched short: K={K}", flush=True)
    for v in range(-1, P.hss_gemm_variants()):
        short = P.hss_gemm_batched(As[:4], Bs[:4], [c.clone() for c in Cs[:4]], tr[:4], 0.5, -1.0, v)
        deep = P.hss_gemm_batched(As, Bs, [c.clone() for c in Cs], tr, 0.5, -1.0, v)
        for s, d, r, b in zip(short, deep, ref, bnd):
            assert torch.equal(s, d) and np.all(np.abs(s.cpu().numpy() - r) <= b)


@pytest.mark.parametrize("M,N,K,t,lda", [
    (70, 40, 520, 1, 1_048_000),   # offsets reach almost 2^32 bytes
    (70, 40, 520, 1, 1_100_000),   # the last slices of a chunk lie beyond
    (70, 40, 1041, 1, 540_000),    # three chunks, each within
    (3, 5, 40, 1, 16_000_000),     # a few rows far apart
    (130, 17, 37, 0, 4_150_000),   # without transposition: a tile of 128 rows almost there
    (130, 17, 37, 0, 4_250_000),   # and beyond
])
def test_gemm_batched_far_apart_rows(M, N, K, t, lda):
    """Rows of A so far apart that 32-bit offsets reach, or no longer reach,
    the last of a tile: the same bits as from a compact copy of A, in the
    shape the library picks and in one that is asked for."""
    g = torch.Generator("cuda").manual_seed(lda)
    rows, cols = (K, M) if t else (M, K)
    print(f"gemm_batched lda={lda} trans={t}", flush=True)
    A = torch.empty((rows - 1) * lda + cols, dtype=torch.float64, device="cuda").as_strided((rows, cols), (lda, 1))
    A.copy_(torch.randn(rows, cols, dtype=torch.float64, device="cuda", generator=g))
    B = torch.randn(K, N, dtype=torch.float64, device="cuda", generator=g)
    C = torch.empty(M, N, dtype=torch.float64, device="cuda")
    ref = P.hss_gemm_batched([A.contiguous()], [B], [C.clone()], [t])[0]
    for v in (-1, 2):
        assert torch.equal(P.hss_gemm_batched([A], [B], [C.clone()], [t], variant=v)[0], ref)
    exact = (A.T if t else A).cpu() @ B.cpu()
    assert torch.allclose(ref.cpu(), exact, rtol=0, atol=2 * _gamma(K) * float((A.abs().max() * B.abs().max())) * K)
