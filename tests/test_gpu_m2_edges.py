"""The FP64 second-moment operator at the edges of its dispatch: column counts on
both sides of the two- and four-columns-per-lane kernels, even and odd, rows of
C^T short (one wave per row) and long (entries split over waves), with empty
rows and rows that end inside, at and across the shares of 256 entries; against the dense expression in float64.

Bar: 1e-12 relative (Frobenius): sums of at most 3e4 terms of mixed sign in
float64 differ by their order in about sqrt(3e4) 2^-53 = 2e-14 of the terms' norm,
and O takes differences of two such sums up to 10 times their size."""
import numpy as np
import pytest
import torch

from gpu_util import dev, rel

from paper_1309_0787_amd import otm

pytestmark = pytest.mark.gpu


def _csr(dense):
    rp = np.concatenate([[0], np.cumsum((dense != 0).sum(1))]).astype(np.int32)
    r, c = np.nonzero(dense)
    return rp, c.astype(np.int32), dense[r, c].astype(np.float32)


def _dev_csr(rp, ci, v, n_cols):
    t = [torch.from_numpy(x).to(dev()) for x in (rp, ci, v)]
    return otm.DeviceCSR(len(rp) - 1, n_cols, t[0], t[1], t[2])


@pytest.mark.parametrize("m", [1, 2, 63, 64, 100, 127, 128, 130, 200, 255, 256])
@pytest.mark.parametrize("n,d,heavy", [(300, 200, False), (2500, 9, False), (2048, 20, True), (700, 1, False)])
@pytest.mark.parametrize("normalize", [False, True])
def test_m2_apply(m, n, d, heavy, normalize):
    g = np.random.default_rng(m * 7 + n + d)
    C = g.integers(1, 4, (n, d)).astype(np.float64)
    if d == 200:
        C *= g.random((n, d)) < 0.1          # short rows of C^T
        C[:, 5] = 0                          # an empty one
        C[:, 1:3] += 1
    elif heavy:
        C *= g.random((n, d)) < np.linspace(0.05, 1.0, d)   # from 100 entries to 2048
        C[:, 3] = 0
        C[:, 0:2] += 1
    if d == 1:
        C += 1
    S = g.standard_normal((d, m))
    alpha0 = 0.7
    rs = C.sum(1)
    a1, a2 = (1 / rs, 1 / (rs * (rs - 1))) if normalize else (np.ones(n), np.ones(n))
    M1 = C.T @ a1 / n
    ref = (alpha0 + 1) / n * (C.T @ (a2[:, None] * (C @ S)) - (C.T @ a2)[:, None] * S) - alpha0 * np.outer(M1, M1 @ S)
    A, AT = _dev_csr(*_csr(C), d), _dev_csr(*_csr(C.T.copy()), n)
    St = torch.from_numpy(S).to(dev())
    O = otm.m2_apply(A, AT, normalize, alpha0, St)
    again = otm.m2_apply(A, AT, normalize, alpha0, St)
    torch.cuda.synchronize()
    assert rel(O.cpu().numpy(), ref) < 1e-12
    assert torch.equal(O, again)             # fixed order of every sum


@pytest.mark.parametrize("n,d,m,per_row,normalize",
                         [(41000, 40500, 50, 6, False), (41000, 40500, 51, 6, True), (42000, 1000, 48, 8, True),
                          (42000, 40000, 62, 5, True), (64000, 90, 32, 4, True), (20000, 100, 128, 40, False),
                          (42000, 8000, 48, 5, False)])
def test_m2_apply_panels(n, d, m, per_row, normalize):
    """Matrices past 16 MB: both passes by panels, the second alone, rows of C^T
    short and long (a workgroup each), m at the ends of a panel with and without room
    for the two weight columns, empty rows of C^T."""
    import scipy.sparse as sp

    g = np.random.default_rng(n + m)
    cols = g.integers(0, d - 1, (n, per_row))         # column d - 1 stays empty
    C = sp.csr_matrix((g.integers(1, 4, n * per_row).astype(np.float64),
                       (np.repeat(np.arange(n), per_row), cols.reshape(-1))), shape=(n, d))
    C.sum_duplicates()
    S = g.standard_normal((d, m))
    rs = np.asarray(C.sum(1)).ravel()
    a1, a2 = (1 / rs, 1 / (rs * (rs - 1))) if normalize else (np.ones(n), np.ones(n))
    M1 = C.T @ a1 / n
    ref = 1.7 / n * (C.T @ (a2[:, None] * (C @ S)) - (C.T @ a2)[:, None] * S) - 0.7 * np.outer(M1, M1 @ S)
    CT = C.T.tocsr()
    dc = lambda M: _dev_csr(M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data.astype(np.float32), M.shape[1])
    A, AT, St = dc(C), dc(CT), torch.from_numpy(S).to(dev())
    O = otm.m2_apply(A, AT, normalize, 0.7, St)
    again = otm.m2_apply(A, AT, normalize, 0.7, St)
    torch.cuda.synchronize()
    assert rel(O.cpu().numpy(), ref) < 1e-12
    assert torch.equal(O, again)


@pytest.mark.parametrize("m", [7, 40, 128, 130, 200])
def test_columns_out_of_range_are_skipped(m):
    """Entries with a column outside the matrix count for nothing, in short rows and long ones,
    by rows and by panels; a matrix without columns leaves nothing of X to read."""
    g = np.random.default_rng(m)
    n, d = 60000 if m >= 40 else 700, 300
    per = 12
    cols = g.integers(0, d, (n, per)).astype(np.int64)
    bad = g.random((n, per)) < 0.2
    ci = np.where(bad, np.where(g.random((n, per)) < 0.5, -1 - cols, d + cols), cols).astype(np.int32)
    rp = np.arange(0, n * per + 1, per, dtype=np.int32)
    A = _dev_csr(rp, ci.reshape(-1), np.ones(n * per, np.float32), d)
    # its transpose, with bad columns put among the good ones of every row
    r, c = np.repeat(np.arange(n), per)[~bad.reshape(-1)], cols.reshape(-1)[~bad.reshape(-1)]
    extra = int(bad.sum())
    rows = np.concatenate([c, g.integers(0, d, extra)])
    cc = np.concatenate([r, np.where(g.random(extra) < 0.5, -7, n + 3)])
    o = np.argsort(rows, kind="stable")
    rpt = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=d))]).astype(np.int32)
    AT = _dev_csr(rpt, cc[o].astype(np.int32), np.ones(n * per, np.float32), n)
    S = g.standard_normal((d, m))
    C = np.zeros((n, d))
    np.add.at(C, (r, c), 1.0)
    M1 = C.sum(0) / n
    ref = 1.7 / n * (C.T @ (C @ S) - C.sum(0)[:, None] * S) - 0.7 * np.outer(M1, M1 @ S)
    O = otm.m2_apply(A, AT, False, 0.7, torch.from_numpy(S).to(dev()))
    assert rel(O.cpu().numpy(), ref) < 1e-12
    # Pairs V = (1/n) G1T (G2 V) with G2 of no columns
    E = otm.DeviceCSR(n, 0, A.rowptr, A.colidx, None).c()
    G = AT.c()
    V = torch.ones(8, dtype=torch.float64, device=dev())
    out = torch.full((d, m), 5.0, dtype=torch.float64, device=dev())
    ws = torch.empty(otm.lib().otm_pairs_apply_workspace(n, m), dtype=torch.uint8, device=dev())
    otm._check(otm.lib().otm_pairs_apply(G, E, V.data_ptr(), m, out.data_ptr(), ws.data_ptr(), ws.numel(), otm._stream()))
    assert torch.equal(out, torch.zeros_like(out))


def test_many_long_rows():
    """A million rows of C^T of 256 entries, 256 columns: a workgroup to each row and
    panel would be more threads than a launch holds.  The matrix is circulant, so rows of
    the result follow from 256 x 256 rows of S; entries agree within 1e-12 of the row's largest
    (sums of 65536 terms)."""
    d = m = 256
    n = 1_000_000
    o = torch.from_numpy(np.random.default_rng(0).permutation(n)[:d].astype(np.int32)).to(dev())
    t = torch.arange(n, dtype=torch.int32, device=dev())
    rp = torch.arange(0, n * d + 1, d, dtype=torch.int32, device=dev())
    A = otm.DeviceCSR(n, n, rp, ((t[:, None] + o) % n).reshape(-1))
    AT = otm.DeviceCSR(n, n, rp, ((t[:, None] - o + n) % n).reshape(-1))
    S = torch.randn((n, m), dtype=torch.float64, device=dev(), generator=torch.Generator(device=dev()).manual_seed(1))
    O = otm.m2_apply(A, AT, False, 0.7, S)
    v = d * S.sum(0) / n
    for a in (0, 1, 63, 64, 500_001, n - 1):
        rows = (a - o[:, None].long() + o[None].long()) % n
        ref = 1.7 / n * (S[rows.reshape(-1)].sum(0) - d * S[a]) - 0.7 * d / n * v
        assert (O[a] - ref).abs().max() <= 1e-12 * ref.abs().max(), a


@pytest.mark.parametrize("n,d,m,per", [(300, 200, 40, 5), (20000, 70, 20, 40), (3000, 9, 256, 6), (42000, 41000, 50, 4),
                                       (64000, 90, 32, 6), (42000, 41000, 49, 5),
                                       (42000, 41000, 50, 24), (42000, 41000, 49, 25), (110000, 5000, 60, 6)])
def test_workspace_is_all_that_is_written(n, d, m, per):
    """The layout of every path stays inside the size that the workspace function gives: bytes past
    it keep their value, and the result is that of a roomier one."""
    g = np.random.default_rng(n + m)
    key = np.unique(g.integers(0, n, n * per).astype(np.int64) * d + g.integers(0, d, n * per))
    r, c = key // d, key % d
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32)
    o = np.argsort(c, kind="stable")
    rpt = np.concatenate([[0], np.cumsum(np.bincount(c, minlength=d))]).astype(np.int32)
    one = np.ones(len(r), np.float32)
    A, AT = _dev_csr(rp, c.astype(np.int32), one, d), _dev_csr(rpt, r[o].astype(np.int32), one, n)
    S = torch.from_numpy(g.standard_normal((d, m))).to(dev())
    size, guard = otm.lib().otm_m2_apply_workspace(n, d, m), 1 << 20
    ws = torch.full((size + guard,), 0xA5, dtype=torch.uint8, device=dev())
    O = torch.empty((d, m), dtype=torch.float64, device=dev())
    info = torch.zeros(1, dtype=torch.int32, device=dev())
    otm._check(otm.lib().otm_m2_apply(A.c(), AT.c(), 0, 0.7, S.data_ptr(), m, O.data_ptr(), info.data_ptr(),
                                      ws.data_ptr(), size, otm._stream()))
    kept = int((ws[size:] == 0xA5).sum().item())
    assert kept == guard
    assert torch.equal(O, otm.m2_apply(A, AT, False, 0.7, S))
    assert otm.lib().otm_m2_apply(A.c(), AT.c(), 0, 0.7, S.data_ptr(), m, O.data_ptr(), info.data_ptr(),
                                  ws.data_ptr(), size - 1, otm._stream()) == -7


@pytest.mark.parametrize("n2,m,per", [(9000, 140, 33), (9000, 139, 33), (9000, 138, 32), (9000, 140, 31), (25000, 100, 40),
                                      (25000, 99, 40), (12000, 256, 70), (20000, 128, 35)])
@pytest.mark.parametrize("weighted", [False, True])
def test_pairs_apply_both_loops(n2, m, per, weighted):
    """Pairs V on both sides of the rule between the two loops of the plain product (size
    of V, its width, entries per row; rows of every length mod 4), with columns out of range,
    against dense float64."""
    g = np.random.default_rng(n2 + m)
    n = 400
    ln = np.full(n, per)
    ln[:8] += np.arange(8) - 4                        # rows that end inside a group of four
    ln[8] = 0
    ln[9] += 4 + per
    r = np.repeat(np.arange(n), ln)
    c = g.integers(0, n2, len(r)).astype(np.int32)
    bad = g.random(len(r)) < 0.05
    v = g.integers(1, 4, len(r)).astype(np.float32) if weighted else None
    rp = np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)
    ci = np.where(bad, n2 + 5, c).astype(np.int32)
    t = lambda x: None if x is None else torch.from_numpy(x).to(dev())
    G2 = otm.DeviceCSR(n, n2, t(rp), t(ci), t(v))
    eye = np.arange(n, dtype=np.int32)
    G1T = otm.DeviceCSR(n, n, t(np.arange(n + 1, dtype=np.int32)), t(eye), None)
    V = g.standard_normal((n2, m))
    ref = np.zeros((n, m))
    w = (np.ones(len(r)) if v is None else v.astype(np.float64)) * ~bad
    np.add.at(ref, r, w[:, None] * V[c])
    out = otm.pairs_apply(G1T, G2, torch.from_numpy(V).to(dev()))
    assert rel(out.cpu().numpy(), ref / n) < 1e-14    # sums of at most 150 terms


@pytest.mark.parametrize("n,d,m,per_row,normalize",
                         [(41000, 40500, 50, 24, False), (41000, 40500, 51, 24, True), (42000, 40000, 62, 21, True),
                          (42000, 40000, 62, 20, False), (42000, 40000, 62, 19, True), (30000, 60000, 80, 45, False),
                          (60000, 30000, 80, 15, True), (63000, 12000, 100, 5, False), (63000, 12000, 100, 3, True)])
def test_m2_apply_row_lengths(n, d, m, per_row, normalize):
    """Both sides of the rules that take rows by panels: 20 entries a row of C^T for the
    second pass and of C for the first, and workgroups enough."""
    test_m2_apply_panels(n, d, m, per_row, normalize)
