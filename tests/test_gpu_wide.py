"""The host-driven kernels beyond one block and one tile, and the inverses
beyond the register groups: expansions with more than one tile of virtual
orbitals over many column blocks, gradients on blocks wider than 64 columns,
matrices of more than 4096 and 8192 rows.  References are LAPACK's solves of the
dense matrices, and permutations, whose inverses have no rounding."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_1708_00744_amd import dsu, inputs
from test_gpu_edges import well_conditioned

pytestmark = pytest.mark.gpu


def expansion(n, m):
    """Orders 0 .. 4 over the first, middle and last occupied and virtual
    orbitals; the reference dominates, so Psi stays near 1."""
    o, v = [n - 1, 0, n // 2, 64 % n], [m - 1, 0, m // 2, 15 % m]
    dets = [(1.0, [])] + [(0.05 / (1 + a + b), [(o[a], v[b])]) for a in range(4) for b in range(4)]
    return dets + [(0.03 * (-1) ** q, [(o[(q + a) % 4], v[a]) for a in range(q)]) for q in (2, 3, 4)]


def psi(a, v, dets):
    """sum_I c_I det(A_I) / det(A), sign and log|det| of A."""
    t = np.linalg.solve(a, v)
    q = sum(c * (np.linalg.det(t[np.ix_([j for j, _ in sub], [x for _, x in sub])]) if sub else 1.0)
            for c, sub in dets)
    return (q,) + tuple(np.linalg.slogdet(a))


# 130: three column blocks, one tile and one orbital of a second; 1030: 17 blocks,
# more virtuals than eight waves take at once; 2113: 128 columns a block, the last half full
@pytest.mark.parametrize("n,m,K", [(130, 17, 5), (1030, 130, 9), (2113, 17, 4)])
def test_multidet_over_blocks_and_tiles(n, m, K):
    require_gpu()
    a, v = well_conditioned(90 + n, n), inputs.rows(91, n, m) / np.sqrt(n)
    dets, moves = expansion(n, m), 8
    noise, vrows = inputs.rows(92, moves, n), inputs.rows(93, moves, m) / np.sqrt(n)
    # singular values of A within about [1, 3], T and Psi near 1: as for the look-ahead ratios
    tol = 1e-10
    with dsu.Walker(a, K) as w:
        w.set_multidet(v, dets)
        q0, s0, l0 = psi(a, v, dets)
        for e, row, vrow in zip([0, n - 1, 70, 0, n // 2, 70, 5, 64], noise, vrows):
            row = 0.9 * a[e] + 0.1 * row / np.sqrt(n)
            b, vb = a.copy(), v.copy()
            b[e], vb[e] = row, vrow
            q1, s1, l1 = psi(b, vb, dets)
            ref = s1 * s0 * np.exp(l1 - l0)
            total, r = w.propose_md(e, row, vrow)
            assert abs(r - ref) <= tol * max(1.0, abs(ref))
            assert abs(total - ref * q1 / q0) <= tol * max(1.0, abs(total))
            if e == 5:
                w.reject()
                continue
            w.accept()
            a, v, q0, s0, l0 = b, vb, q1, s1, l1
        for _ in range(2):
            sg, la = w.md_value()
            assert sg == np.sign(q0) * s0 and abs(la - (l0 + np.log(abs(q0)))) <= n * tol
            w.recompute()


# Five columns of the product in LDS; the electron asked for holds no pending
# move, then one.  128 and 64 columns a block.
@pytest.mark.parametrize("n,prec", [(2113, dsu.FP64), (2113, dsu.FP32_MIXED), (1025, dsu.FP64)])
def test_gradients_on_wide_blocks(n, prec):
    require_gpu()
    a = well_conditioned(95 + n, n)
    inv = np.linalg.inv(a)
    noise = inputs.rows(96, 12, n)
    # N-term dot products of terms bounded by 4 (FP32: unit roundoff 2^-24), x 4 for the pending moves' solve
    tol = 16.0 * np.sqrt(n) * 2.0**-24 if prec == dsu.FP32_MIXED else 1e-10
    mix = lambda e, x: 0.9 * a[e] + 0.1 * x / np.sqrt(n)
    near = lambda got, exact: np.all(np.abs(np.asarray(got) - exact) <= tol * np.maximum(1.0, np.abs(exact)))
    with dsu.Walker(a, 6, precision=prec) as w:
        for q, e in enumerate([3, n - 1, 3, 64]):
            row, drow = mix(e, noise[q]), np.stack([mix(e, noise[4 + q + x]) for x in range(3)])
            assert near(w.grad(e, drow), drow @ inv[:, e])
            exact = row @ inv[:, e]
            r, g = w.propose_grad(e, row, drow)
            assert near(r, exact) and near(g, drow @ inv[:, e])
            assert near(w.grad(7, drow), drow @ inv[:, 7])  # the proposal stays pending
            w.accept()
            inv = inv - np.outer(inv[:, e], row @ inv - np.eye(n)[e]) / exact
            a[e] = row
            assert w.pending() > 0 and near(w.grad(e, drow), drow @ inv[:, e])


# Real: one column at a time above 8192 rows.  Complex: groups of two columns
# above 4096, one above 8192.  Every pivot leaves its place.
@pytest.mark.parametrize("n,cplx", [(8257, False), (4100, True), (8257, True)])
def test_large_permutation_inverse_is_exact(n, cplx):
    require_gpu()
    rng = np.random.default_rng(n)
    to, unit = rng.permutation(n), rng.choice(np.array([1, -1, 1j, -1j] if cplx else [1, -1]), n)
    a = np.zeros((n, n), np.complex128 if cplx else np.float64)
    a[np.arange(n), to] = unit
    with (dsu.ZWalker(a, 4) if cplx else dsu.Walker(a, 4)) as w:
        x = w.inverse()
        got = w.logdet()
    assert np.array_equal(x[to, np.arange(n)], unit.conj())
    x[to, np.arange(n)] = 0
    assert not x.any()
    odd, seen = 0, np.zeros(n, bool)
    for i in range(n):
        length = 0
        while not seen[i]:
            seen[i] = True
            i, length = to[i], length + 1
        odd ^= length > 0 and length % 2 == 0
    sign = (-1) ** odd * np.round(np.exp(1j * np.angle(unit).sum()))
    if cplx:
        assert got[0] == 0.0 and abs(np.exp(1j * got[1]) - sign) <= 8 * n * 2.0**-53
    else:
        assert got == (int(sign.real), 0.0)


def test_multidet_replaced_by_another_size():
    """A larger, then a smaller expansion on one walker: the ratios of a walker
    that had the smaller one alone, bit for bit."""
    require_gpu()
    n, moves = 200, 6
    a = well_conditioned(98, n)
    rows, v = inputs.rows(99, moves, n) / np.sqrt(n), inputs.rows(97, n, 130) / np.sqrt(n)
    seen = []
    for sizes in ((130, 17), (17,), (1, 17)):
        with dsu.Walker(a, 4) as w:
            for m in sizes:
                w.set_multidet(np.ascontiguousarray(v[:, :m]), expansion(n, m) if m > 1 else [(1.0, []), (0.1, [(3, 0)])])
                got = []
                for e, row in enumerate(rows):
                    got.append(w.propose_md(e, 0.9 * a[e] + 0.1 * row, v[e, :m]))
                    w.reject()
            seen.append((got, w.md_value()))
    assert seen[0] == seen[1] == seen[2]
