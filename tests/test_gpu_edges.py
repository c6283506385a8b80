"""Kernels at the sizes where their tilings change: edges of tiles, remainders,
the smallest and largest of a range.  References are LAPACK and the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import require_gpu
from paper_1708_00744_amd import dsu, inputs

pytestmark = pytest.mark.gpu


def well_conditioned(seed, n, complex_=False):
    """2 I + (entries uniform in [-1, 1]) / (2 sqrt(n)): singular values within
    about [1, 3], so FP64 ratios are good to ~n 2^-53 and FP32 ones to ~n 2^-24
    of the terms' size (bounded by 4)."""
    a = inputs.dense_matrix(seed, n) / (2.0 * np.sqrt(n))
    if complex_:
        a = a + 1j * inputs.dense_matrix(seed + 1, n) / (2.0 * np.sqrt(n))
    return a + 2.0 * np.eye(n)


# Look-ahead launches: 64 real columns a block up to 2048, more from there
# (2049 real: 128 with a half last block; complex from 1025); 2 k + 1 rows in
# tiles of 16 over 8 waves (k = 7, 8: one and two tiles; k = 63, 64: one and
# two rounds of the waves); k = 65 and 130: second and third 64 entries of t.
@pytest.mark.parametrize("n,K,moves,kind", [
    (1, 1, 1, "fp64"), (64, 9, 10, "fp64"), (65, 66, 65, "fp64"), (200, 131, 131, "fp64"),
    (2049, 10, 12, "fp64"), (130, 66, 70, "fp32"), (2113, 9, 12, "fp32"), (2113, 9, 12, "fp32_dev"),
    (67, 66, 67, "complex"), (1030, 9, 12, "complex")])
def test_lookahead_edges(n, K, moves, kind):
    require_gpu()
    import torch
    cplx = kind == "complex"
    a = well_conditioned(11 + n, n, cplx)
    inv = np.linalg.inv(a)
    noise = inputs.rows(5, moves, n) + (1j * inputs.rows(6, moves, n) if cplx else 0.0)
    f32 = kind.startswith("fp32")
    # FP32: N-term dot products of terms bounded by 4, unit roundoff 2^-24, x 4 for the pending moves' solve
    tol = 16.0 * np.sqrt(n) * 2.0**-24 if f32 else 1e-10
    w = dsu.ZWalker(a, K) if cplx else dsu.Walker(a, K, precision=dsu.FP32_MIXED if f32 else dsu.FP64)
    with w:
        for m in range(moves):
            e = (7 * m) % n if n > moves else m
            row = 0.9 * a[e] + 0.1 * noise[m] / np.sqrt(n)
            if kind == "fp32_dev":
                dev = torch.tensor(row, dtype=torch.float32, device="cuda")
                torch.cuda.synchronize()
                row = dev.cpu().numpy().astype(np.float64)
                r = w.propose_dev(e, dev.data_ptr())
            else:
                r = w.propose(e, row)
            exact = row @ inv[:, e]
            assert abs(r - exact) <= tol * max(1.0, abs(exact)), (m, e, r, exact)
            w.accept()
            inv = inv - np.outer(inv[:, e], row @ inv - np.eye(n)[e]) / exact
        got = w.inverse()
    assert np.abs(got - inv).max() <= (1e-9 if not f32 else 16.0 * np.sqrt(n) * 2.0**-24)


# Gauss-Jordan groups: 256 threads up to a padded 256 and 512 rows, 512 threads
# up to 1024, 2048, 4096 and 8192; the last panel and its last group narrower
# than their tiles (4 pivots a loop body, 32 .. 4 columns a group).
@pytest.mark.parametrize("n", [3, 67, 255, 257, 511, 513, 1027, 2051, 4101])
def test_inverse_edges(n):
    require_gpu()
    a = well_conditioned(31 + n, n)
    with dsu.Walker(a, 4) as w:
        got, (sg, ld) = w.inverse(), w.logdet()
    s_np, l_np = np.linalg.slogdet(a)
    # well conditioned: backward-stable elimination, growth far below sqrt(n)
    assert np.abs(got @ a - np.eye(n)).max() <= 64 * n * 2.0**-53 * 4
    assert sg == s_np and abs(ld - l_np) <= 64 * n * 2.0**-53 * max(1.0, abs(l_np))


# Every pivot column full of ties and every pivot off the diagonal: a signed
# permutation matrix, whose inverse (its transpose) has no rounding at all.
@pytest.mark.parametrize("n", [2, 70, 300, 1100])
def test_inverse_of_signed_permutation_is_exact(n):
    require_gpu()
    rng = np.random.default_rng(n)
    a = np.zeros((n, n))
    a[np.arange(n), rng.permutation(n)] = rng.choice([-1.0, 1.0], n)
    with dsu.Walker(a, 4) as w:
        assert np.array_equal(w.inverse(), a.T)
        sg, ld = w.logdet()
    assert ld == 0.0 and sg == round(np.linalg.slogdet(a)[0])


# The flush's launches: 16, 32 .. slots (one or two tiles), 64-row blocks with
# and without padding, FP64 columns in 1, 2, 4 or 8 parts, k at and beside the
# tile widths; the vector-ALU kernel as the other path.  Complex: 2 k real
# slots, and k = 130 beyond the embedding's width.
@pytest.mark.parametrize("n,k,kind", [
    (5, 5, "fp64"), (64, 16, "fp64"), (65, 17, "fp64"), (300, 33, "fp64"), (1100, 64, "fp64"), (2100, 7, "fp64"),
    (260, 129, "fp64"), (200, 33, "fp32"), (700, 128, "fp32"), (3, 3, "complex"), (70, 8, "complex"),
    (70, 9, "complex"), (300, 65, "complex"), (600, 32, "complex"), (140, 130, "complex")])
def test_flush_edges(n, k, kind):
    require_gpu()
    cplx, f32 = kind == "complex", kind == "fp32"
    a = well_conditioned(51 + n, n, cplx)
    noise = inputs.rows(7, k, n) + (1j * inputs.rows(8, k, n) if cplx else 0.0)
    order = [(5 * m + 1) % n if n % 5 else m for m in range(k)]
    rows = [0.9 * a[e] + 0.1 * noise[m] / np.sqrt(n) for m, e in enumerate(order)]
    b = a.copy()
    b[order] = rows
    K, got = min(256, k + 1), []
    for mode in (dsu.FLUSH_MFMA, dsu.FLUSH_VALU):
        if mode == dsu.FLUSH_VALU and K > 64 and not cplx:
            continue  # refused: the vector-ALU kernel holds up to 64 slots
        with (dsu.ZWalker(a, K) if cplx else
              dsu.Walker(a, K, precision=dsu.FP32_MIXED if f32 else dsu.FP64)) as w:
            w.set_flush_kernel(mode)
            for e, row in zip(order, rows):
                w.propose(e, row)
                w.accept()
            assert w.pending() == k
            w.flush()
            got.append(w.inverse())
    exact = np.linalg.inv(b)
    tol = 64.0 * np.sqrt(n) * 2.0**-24 if f32 else 1e-10
    for inv in got:
        assert np.abs(inv - exact).max() <= tol


# Fresh inverses.  Complex: groups of 16 columns (15, 16, 17: a short, a full and
# a short second group), 8 above n = 1024, 4 above 2048; rows in permuted order
# make every pivot leave its place.  Real: a ragged matrix goes up unpadded.
@pytest.mark.parametrize("n,cplx", [(1, True), (15, True), (16, True), (17, True), (64, True), (513, True),
                                    (1024, True), (1025, True), (2049, True), (1, False), (65, False), (200, False)])
def test_fresh_inverse_edges(n, cplx):
    require_gpu()
    a = [well_conditioned(40 + n + q, n, cplx)[np.random.default_rng(n + q).permutation(n)] for q in range(2)]
    # singular values within about [1, 3]: backward error of order n 2^-53, times the condition and the pivot growth
    tol = 64.0 * n * 2.0**-53 + 2.0**-52
    with (dsu.ZWalker(a[0], 4) if cplx else dsu.Walker(a[0], 4)) as w:
        for m in (None, a[1], None):
            if m is not None or n > 1:
                w.recompute(m)
            ref = a[0] if m is None else m
            assert np.abs(w.inverse() - np.linalg.inv(ref)).max() <= tol
            s, ld = np.linalg.slogdet(ref)
            got = w.logdet()
            phase = np.exp(1j * got[1]) if cplx else got[0]
            assert abs(phase - s) <= n * tol and abs((got[0] if cplx else got[1]) - ld) <= n * tol
            a[0] = ref


@pytest.mark.parametrize("n", [3, 40])
def test_complex_singular_and_nan(n):
    require_gpu()
    a = well_conditioned(70 + n, n, True)
    for bad in ("zero column", "nan"):
        b = a.copy()
        if bad == "zero column":
            b[:, n // 2] = 0.0
        else:
            b[n // 2, :] = np.nan
        with dsu.ZWalker(a, 4) as w:
            with pytest.raises(dsu.DsuError):
                w.recompute(b)


# FP32 sweeps at K = 64 and 128: up to 256 blocks of 64 rows take the split flush,
# more the 128-row one (257 blocks of n = 64; 129 determinants of two blocks); n <=
# K is one window, without a next one.  A determinant's trajectory depends on its
# own seed alone, and both forms do the same operations in the same order.
@pytest.mark.parametrize("n,K,walkers", [(64, 64, 257), (50, 128, 257), (128, 64, 129), (100, 64, 129),
                                         (128, 128, 129), (65, 50, 129), (300, 100, 52)])
def test_flush_forms_agree(n, K, walkers):
    require_gpu()
    pos = np.stack([inputs.positions(9, w, n, 10.0) for w in range(walkers)])

    def run(sel):
        with dsu.Batch(n, pos[sel], [9] * len(sel), sel, 0.3, K, precision=dsu.FP32_MIXED, box_l=10.0) as b:
            b.sweep(2)
            st = b.stats()
            return [(st["logdet"][q], st["sign"][q], st["accepted"][q], b.positions(q)) for q in range(3)]

    many, few = run(list(range(walkers))), run([0, 1, 2])
    for a, b in zip(many, few):
        assert a[:3] == b[:3] and np.array_equal(a[3], b[3])


# Recomputes: the update's column parts by the number of determinants (np = 256, 320
# ragged in thirds, 512, 1024: 2 to 8 parts for one determinant, one part from 512
# workgroups on); a determinant's inverse does not depend on its company.
@pytest.mark.parametrize("n,many", [(250, 128), (300, 103), (512, 64), (1024, 32)])
def test_recompute_parts_agree(n, many):
    require_gpu()
    pos = np.stack([inputs.positions(21, w, n, 10.0) for w in range(many)])

    def run(count):
        with dsu.Batch(n, pos[:count], [21] * count, list(range(count)), 0.1, 16, precision=dsu.FP64, box_l=10.0) as b:
            st = b.stats()
            return st["logdet"][0], st["sign"][0], b.inverse(0)

    one, all_ = run(1), run(many)
    assert one[:2] == all_[:2] and np.array_equal(one[2], all_[2])
    kv = dsu.plane_wave_rows(n, 10.0, pos[0])
    assert np.abs(one[2] @ kv - np.eye(n)).max() <= 1e-16 * n * np.linalg.cond(kv)


# Proposal rows: column groups of 64 over the blocks and waves (np = 192: three groups
# on four waves; 320: five; 576: two blocks of four and five), short last windows.
@pytest.mark.parametrize("n,K", [(130, 16), (300, 32), (520, 64)])
def test_rows_splits_match_oracle(n, K):
    require_gpu()
    pos = inputs.positions(31, 0, n, 10.0)
    with dsu.Batch(n, pos[None], [31], [0], 0.3, K, precision=dsu.FP64, box_l=10.0) as b:
        b.set_trace(1)
        b.sweep(1)
        r, acc = b.trace(0)
    t = oracle.walker_run(n, 10.0, 31, 0, 0, 0.3, pos, 1)
    assert np.array_equal(acc, t.accepted)
    # ratios: FP64 sums of n terms through an inverse of condition ~1e4 at most, absolute below 1e-2
    assert (np.abs(r - t.ratio) / np.maximum(np.abs(t.ratio), 1e-2)).max() < 1e-8
