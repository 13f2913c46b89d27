"""GPU parity: every format conversion, feature and SpMM of the HIP library
against the CPU oracle, on the same seeded inputs.

Bar: conversions and integer features bit-exact; feature doubles bitwise
equal; SpMM within |Y - Y_ref| <= 1e-5 (|A||X|) + 1e-6 elementwise.
"""
import ctypes

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2111_00352_amd as gs

pytestmark = pytest.mark.gpu

FMTS = ["csr", "coo", "ell", "dia", "bsr", "csc"]
DEV = "cuda"


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _host(t):
    return t.cpu().numpy()


class Case:
    def __init__(self, R, C, row, col, val, X=None):
        self.R, self.C = R, C
        self.row, self.col, self.val = row, col, val
        self.X = X
        self.d_row, self.d_col, self.d_val = _dev(row), _dev(col), _dev(val)
        orow, ocol, oval = oracle.canon(R, C, row, col, val)
        self.crow, self.ccol, self.cval = orow, ocol, oval
        self.rp = oracle.csr(R, orow)

    def build(self, fmt, b=16, **kw):
        return gs.build_format(self.d_row, self.d_col, self.d_val, (self.R, self.C), fmt,
                               bsr_block=b, **kw)


def _case_from_graph(g, shuffle_seed=None):
    row, col, val = g.row, g.col, g.val
    if shuffle_seed is not None:
        row, col, val = graphgen.shuffled(row, col, val, shuffle_seed)
    return Case(g.R, g.C, row, col, val, g.X)


def _random_case(R, C, nnz, seed, empty=0.1, shuffle=True):
    row, col, val = graphgen.random_coo(R, C, nnz, seed, empty_rows=empty)
    if shuffle:
        row, col, val = graphgen.shuffled(row, col, val, seed + 1)
    return Case(R, C, row, col, val)


def _bits(a):
    a = np.ascontiguousarray(a)
    return a.view(np.uint32) if a.dtype == np.float32 else a


def check_layout(case, fmt, b=16):
    m = case.build(fmt, b)
    R, C = case.R, case.C
    if fmt == "csr":
        exp = [case.rp, case.ccol, case.cval]
    elif fmt == "coo":
        exp = [case.crow, case.ccol, case.cval]
    elif fmt == "csc":
        exp = list(oracle.csc(R, C, case.crow, case.ccol, case.cval))
    elif fmt == "ell":
        K, ec, ev = oracle.ell(R, case.rp, case.ccol, case.cval)
        assert m.param == K
        exp = [ec, ev]
    elif fmt == "dia":
        off, data = oracle.dia(R, C, case.crow, case.ccol, case.cval)
        assert m.param == off.size
        exp = [off, data]
    else:
        bp, bc, bv = oracle.bsr(R, C, b, case.crow, case.ccol, case.cval)
        assert m.param == bc.size
        exp = [bp, bc, bv]
    for which, e in enumerate(exp):
        got = _host(m.array(which))
        assert got.size == e.size, (fmt, which)
        assert (_bits(got) == _bits(e.astype(got.dtype))).all(), (fmt, which)
    r, c, v = (_host(t) for t in m.to_coo())
    assert (r == case.crow).all() and (c == case.ccol).all()
    assert (_bits(v) == _bits(case.cval)).all()
    return m


def check_spmm(case, m, X, rows=None, ldx_pad=0, ldy_pad=0):
    F = X.shape[1]
    Xd = torch.zeros((case.C, F + ldx_pad), dtype=torch.float32, device=DEV)
    Xd[:, :F] = _dev(X)
    Xv = Xd[:, :F]
    out = torch.full((case.R, F + ldy_pad), 7.0, dtype=torch.float32, device=DEV)
    Y = m.spmm(Xv, out=out[:, :F])
    Y2 = m.spmm(Xv)
    torch.cuda.synchronize()
    Yh = _host(Y)
    assert (_bits(Yh) == _bits(_host(Y2))).all(), "SpMM not deterministic"
    if ldy_pad:
        assert (_host(out[:, F:]) == 7.0).all(), "columns beyond F were written"
    if rows is None:
        Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
        ok, worst = oracle.check_spmm(Yh, Yref, M)
    else:
        Yref, M = oracle.spmm_rows(rows, case.rp, case.ccol, case.cval, X)
        ok, worst = oracle.check_spmm(Yh[rows], Yref, M)
    assert ok, f"{m.format}: worst |err|/bound = {worst}"
    return worst


def check_features(case):
    ints, f = oracle.features(case.R, case.C, case.crow, case.ccol)
    got = gs.extract_features(case.d_row, case.d_col, case.d_val, (case.R, case.C))
    for k, v in ints.items():
        assert got[k] == v, k
    assert got["f"] == f.tolist()


# ------------------------------------------------------------ scaled workloads

@pytest.mark.parametrize("k", [1, 2, 3, 4, 5])
def test_scaled_workload_all_formats(k):
    g = graphgen.scaled(k)
    case = _case_from_graph(g)
    check_features(case)
    for fmt in FMTS:
        m = check_layout(case, fmt)
        check_spmm(case, m, g.X)


def test_unsorted_input_is_canonicalised():
    case = _case_from_graph(graphgen.scaled(2), shuffle_seed=9)
    for fmt in FMTS:
        check_layout(case, fmt)
    check_features(case)


# -------------------------------------------------------- property cases

PROPS = [
    (1, 1, 1, 0), (5, 7, 9, 1), (33, 17, 100, 2), (100, 100, 0, 3), (257, 129, 3000, 4),
    (16, 16, 256, 5), (31, 64, 400, 6), (1000, 999, 8000, 7), (3000, 40, 20000, 8),
    (40, 3000, 20000, 9),
]


@pytest.mark.parametrize("R,C,nnz,seed", PROPS)
def test_random_matrix_layouts_features(R, C, nnz, seed):
    case = _random_case(R, C, nnz, seed)
    for fmt in FMTS:
        for b in ((1, 3, 16, 64) if fmt == "bsr" else (16,)):
            check_layout(case, fmt, b)
    check_features(case)


@pytest.mark.parametrize("F", [1, 3, 6, 64, 100, 128, 300])
@pytest.mark.parametrize("fmt", FMTS)
def test_spmm_widths(fmt, F):
    case = _random_case(523, 411, 6000, 11, empty=0.2)
    X = graphgen.features_x(case.C, F, 12, "normal")
    m = case.build(fmt)
    check_spmm(case, m, X)


@pytest.mark.parametrize("fmt", FMTS)
def test_spmm_strided_operands(fmt):
    case = _random_case(300, 280, 3000, 13)
    X = graphgen.features_x(case.C, 64, 14, "normal")
    m = case.build(fmt)
    check_spmm(case, m, X, ldx_pad=4, ldy_pad=8)
    check_spmm(case, m, graphgen.features_x(case.C, 20, 15), ldx_pad=1, ldy_pad=3)


@pytest.mark.parametrize("fmt", FMTS)
def test_long_and_dense_rows(fmt):
    # rows far longer than one chunk and one dense column block
    R, C = 700, 5000
    row, col, val = graphgen.dense_rows_coo(R, C, [0, 3, 350, 699], seed=21, base_nnz=8000)
    case = Case(R, C, row, col, val)
    X = graphgen.features_x(C, 32, 22, "normal")
    try:
        m = case.build(fmt)
    except gs.GnnSpmmError as e:  # padded formats may be over the default cap: not here
        raise AssertionError(str(e))
    check_spmm(case, m, X)


@pytest.mark.parametrize("F", [4, 5, 7, 15, 17, 31, 33, 61, 66, 127, 131, 257])
@pytest.mark.parametrize("fmt", FMTS)
def test_spmm_any_width_and_alignment(fmt, F):
    # widths around the column quads, lanes and slices of every kernel, with
    # operands at every 4-byte alignment (columns cut out of wider tensors);
    # rows of 0..40, 300 and 2,100 entries.  X rows that no entry references
    # hold NaN and must not leak in through the tails of batches.
    case = _uniform_long_rows(230, 2300, 0, 40, 60 + F, hubs=(3,))
    keep = (case.crow != 7) | (np.cumsum(case.crow == 7) <= 15)  # and one row cut short
    keep &= ~((case.crow == 3) & (case.ccol >= 2100))
    case = Case(case.R, case.C, case.crow[keep], case.ccol[keep], case.cval[keep])
    used = np.zeros(case.C, bool)
    used[case.ccol] = True
    X = graphgen.features_x(case.C, F, 61, "normal")
    m = case.build(fmt)
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    X[~used] = np.nan
    for off in range(4):
        Xd = torch.full((case.C, F + 5), float("inf"), dtype=torch.float32, device=DEV)
        Xd[:, off:off + F] = _dev(X)
        out = torch.full((case.R, F + 7), 7.0, dtype=torch.float32, device=DEV)
        m.spmm(Xd[:, off:off + F], out=out[:, 3 - off:3 - off + F])
        got = _host(out)
        ok, worst = oracle.check_spmm(got[:, 3 - off:3 - off + F], Yref, M)
        assert ok, (off, worst)
        assert (got[:, :3 - off] == 7.0).all() and (got[:, 3 - off + F:] == 7.0).all(), "wrote outside Y"


@pytest.mark.parametrize("F", [16, 48, 64, 256, 320])
def test_bsr16_remainder_rows(F):
    # 16 x 16 blocks too sparse for the matrix cores run as rows: full batches
    # and tails of every length (rows of 0..40 entries, a hub), one slice and
    # four slices of columns to a workgroup.  X rows that no entry references
    # hold NaN.
    case = _uniform_long_rows(230, 2300, 0, 40, 60 + F, hubs=(3,))
    keep = ~((case.crow == 3) & (case.ccol >= 2100))
    case = Case(case.R, case.C, case.crow[keep], case.ccol[keep], case.cval[keep])
    used = np.zeros(case.C, bool)
    used[case.ccol] = True
    X = graphgen.features_x(case.C, F, 62, "normal")
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    X[~used] = np.nan
    ok, worst = oracle.check_spmm(_host(case.build("bsr").spmm(_dev(X))), Yref, M)
    assert ok, worst


def _chained_sums(case, X, chains):
    # A.X in fp32 with `chains` running sums per row and column, entry k of a row
    # in chain k % chains (a remainder in the first), added pairwise at the end
    n = np.diff(case.rp)
    acc = np.zeros((chains, case.R, X.shape[1]), np.float32)
    for k in range(int(n.max())):
        r = np.nonzero(n > k)[0]
        e = case.rp[r] + k
        c = np.where(k < n[r] // chains * chains, k % chains, 0)
        prod = case.cval[e].astype(np.float64)[:, None] * X[case.ccol[e]]
        acc[c, r] = (prod + acc[c, r]).astype(np.float32)
    while len(acc) > 1:
        acc = acc[0::2] + acc[1::2]
    return acc[0]


@pytest.mark.parametrize("lo,hi", [(0, 9), (10, 20), (100, 128)])
@pytest.mark.parametrize("fmt,F,off,chains", [("csr", 47, 0, 4), ("csr", 64, 1, 4), ("csr", 131, 0, 4), ("csr", 257, 0, 4),
                                              ("csr", 18, 2, 4), ("csr", 6, 0, 4), ("coo", 64, 0, 4), ("coo", 47, 3, 4),
                                              ("ell", 47, 0, 2), ("ell", 128, 1, 2), ("dia", 47, 0, 2)])
def test_odd_operands_and_coo_keep_short_chains(fmt, F, off, chains, lo, hi):
    # operands that are no 16-byte quads, and COO, are summed no less exactly
    # than in four (ELL and DIA two) chains: the 2-norm of the error is at most
    # that of such sums, up to 4% for the other order (at 10,000 sums and more the
    # spread of a 2-norm is under 1%).  One chain has 1.8 (1.4) times as much over
    # rows of 100 to 128 entries.
    # (DIA folds its chains every 128 of the 1,899 diagonals, which rounds rows of
    # a few entries once more, as it always did: not the first row lengths.)
    if fmt == "dia" and hi == 9:
        lo, hi = 30, 40
    case = _uniform_long_rows(1500, 400, lo, hi, 700 + hi)
    X = graphgen.features_x(case.C, F, 701, "normal").astype(np.float32)
    exact, _ = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    Xd = torch.zeros((case.C, F + off), device=DEV)
    Xd[:, off:] = _dev(X)
    got = _host(case.build(fmt).spmm(Xd[:, off:]))
    want = np.linalg.norm(_chained_sums(case, X, chains) - exact)
    assert np.linalg.norm(got - exact) <= 1.04 * want


@pytest.mark.parametrize("F", [1, 2, 3, 4, 50, 260])
@pytest.mark.parametrize("noalloc", [False, True])
def test_csc_row_sums_in_fp64(F, noalloc):
    # the row form behind a CSC handle: short rows, rows of one workgroup
    # (129..1,024 entries), chunked rows.  For noalloc at F = 260 the chunks'
    # partial sums (8 F bytes each) exceed the fixed scratch while the refusal
    # rule (8 R F bytes) does not apply, so the long rows take a workgroup
    # each; every width equals the oracle's fp64 sum rounded once, up to one
    # fp32 step where a sum sits on a rounding boundary.
    n_long = 40_000 if noalloc and F == 260 else 3_000
    case = _uniform_long_rows(130, n_long, 0, 400, 70, hubs=range(0, 130, 1 if n_long > 3000 else 40))
    X = graphgen.features_x(case.C, F, 71, "normal")
    m = case.build("csc")
    Xd = _dev(X)
    out = torch.full((case.R, F), 7.0, dtype=torch.float32, device=DEV)
    (m.spmm_noalloc if noalloc else m.spmm)(Xd, out)
    Yref, _ = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    want = Yref.astype(np.float32)
    assert np.all(np.abs(_host(out) - want) <= np.spacing(np.abs(want)))


def _uniform_long_rows(R, C, lo, hi, seed, hubs=()):
    # every row holds lo..hi entries at uniformly drawn columns, plus dense hub rows
    rng = np.random.default_rng(seed)
    keys = []
    for r in range(R):
        n = C if r in hubs else int(rng.integers(lo, hi + 1))
        keys.append(r * C + np.sort(rng.choice(C, size=n, replace=False)).astype(np.int64))
    keys = np.concatenate(keys)
    row, col = (keys // C).astype(np.int32), (keys % C).astype(np.int32)
    val = rng.standard_normal(row.size).astype(np.float32)
    val[val == 0] = 0.5
    return Case(R, C, row, col, val)


@pytest.mark.parametrize("group_row", ["", "128", "300"])
@pytest.mark.parametrize("sort", ["1", "2"])
def test_csr_group_tier(monkeypatch, group_row, sort):
    # more medium rows (129..1024 entries) than resident workgroups: rows up
    # to the group limit take one lane group each and are summed chunk by
    # chunk; longer rows (hubs of 6,000) are cut into chunk items.  128 gives
    # the chunk-items-only plan, 300 a limit between the row lengths.
    if group_row:
        monkeypatch.setenv("GS_CSR_GROUP_ROW", group_row)
    monkeypatch.setenv("GS_CSR_GROUP_MIN", "1000")  # the tier's default needs 8 medium rows per resident workgroup
    monkeypatch.setenv("GS_CSR_SORT", sort)
    case = _uniform_long_rows(2600, 6000, 150, 700, 95, hubs=(0, 1300, 2599))
    m = case.build("csr")
    for F, seed in ((64, 96), (36, 97), (132, 98)):
        check_spmm(case, m, graphgen.features_x(case.C, F, seed, "normal"))
    for fmt in ("ell", "dia", "bsr", "coo"):  # the same long rows through the folded chains of every format
        check_spmm(case, case.build(fmt), graphgen.features_x(case.C, 64, 99, "normal"))


@pytest.mark.parametrize("F", [250, 256])
def test_csr_many_long_rows_few_in_flight(F):
    # 2^28 gathered floats in rows of 128 entries and more on average: the row
    # kernel's variant with 4 X rows in flight (full and ragged widths)
    case = _uniform_long_rows(2600, 6000, 150, 700, 93)
    assert case.crow.size * F >= 1 << 28
    check_spmm(case, case.build("csr"), graphgen.features_x(case.C, F, 94, "normal"))


@pytest.mark.parametrize("n", [13, 14, 31, 32, 33, 64, 65])
@pytest.mark.parametrize("F", [67, 100, 128])
def test_csr_two_registers_of_entries(n, F):
    # groups of 32 lanes around the average row length from which they hold 32
    # entries in two registers (14), rows of 0 to 2 n entries with n of them
    # on average: batches that end in either register, empty rows, a hub
    case = _uniform_long_rows(400, 3000, 0, 2 * n, 400 + n, hubs=(7,) if n == 33 else ())
    check_spmm(case, case.build("csr"), graphgen.features_x(case.C, F, 401, "normal"))


@pytest.mark.parametrize("cpl", ["", "4", "8", "16"])
@pytest.mark.parametrize("thr,chunk,wg", [(128, 128, 1024), (32, 32, 64), (16, 8, 100000), (200, 64, 201)])
def test_coo_row_plan(monkeypatch, thr, chunk, wg, cpl):
    # the row plan that a COO handle keeps, under different long-row, chunk and
    # workgroup thresholds and lane layouts: rows at and around 32 and 128
    # entries (the chunk length), short, workgroup-wide and chunked rows back to
    # back, at the first and last row, with empty rows between them
    monkeypatch.setenv("GS_CSR_LONG_ROW", str(thr))
    monkeypatch.setenv("GS_CSR_CHUNK", str(chunk))
    monkeypatch.setenv("GS_CSR_WG_ROW", str(wg))
    if cpl:
        monkeypatch.setenv("GS_CSR_CPL", cpl)
    _check_coo_row_mix()


def _check_coo_row_mix():
    lens = [300, 0, 127, 128, 129, 0, 256, 257, 1000, 1, 0, 0, 5, 128, 16, 17, 15, 640, 0, 3, 31, 32, 33, 0,
            64, 129]
    C = 2000
    rng = np.random.default_rng(77)
    rows, cols = [], []
    for i, n in enumerate(lens):
        rows.append(np.full(n, i, np.int32))
        cols.append(np.sort(rng.choice(C, n, replace=False)).astype(np.int32))
    row, col = np.concatenate(rows), np.concatenate(cols)
    val = rng.uniform(-1, 1, row.size).astype(np.float32)
    val[val == 0] = 0.5
    row, col, val = graphgen.shuffled(row, col, val, 78)
    case = Case(len(lens), C, row, col, val)
    m = case.build("coo")
    for F in (4, 64, 132, 256):
        X = graphgen.features_x(C, F, 79 + F, "normal")
        check_spmm(case, m, X)


def test_empty_and_degenerate_matrices():
    for R, C in ((0, 0), (0, 5), (5, 0), (7, 9)):
        case = Case(R, C, np.zeros(0, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
        for fmt in FMTS:
            m = case.build(fmt)
            assert m.nnz == 0
            if R and C:
                Y = m.spmm(_dev(np.ones((C, 4), np.float32)))
                assert (_host(Y) == 0).all()
        if R and C:
            check_features(case)


def test_one_row_holds_most_entries():
    # a single row of 300,000 entries among short and empty rows: CSR and COO
    # split it into chunks combined in order, CSC does in fp64
    R, C = 5000, 400_000
    rng = np.random.default_rng(131)
    hub = np.sort(rng.choice(C, 300_000, replace=False)).astype(np.int32)
    rows = [np.full(hub.size, 2500, np.int32)]
    cols = [hub]
    for i in range(0, R, 7):
        if i == 2500:
            continue
        n = int(rng.integers(0, 40))
        rows.append(np.full(n, i, np.int32))
        cols.append(np.sort(rng.choice(C, n, replace=False)).astype(np.int32))
    row, col = np.concatenate(rows), np.concatenate(cols)
    val = rng.uniform(0.5, 1.5, row.size).astype(np.float32)
    row, col, val = graphgen.shuffled(row, col, val, 132)
    case = Case(R, C, row, col, val)
    for fmt in ("csr", "coo", "csc"):
        m = case.build(fmt)
        for F in (4, 64):
            check_spmm(case, m, graphgen.features_x(C, F, 133 + F, "normal"))


def test_identity_spmm_is_exact():
    n = 4097
    idx = np.arange(n, dtype=np.int32)
    case = Case(n, n, idx, idx, np.ones(n, np.float32))
    X = graphgen.features_x(n, 64, 3, "normal")
    for fmt in FMTS:
        Y = _host(case.build(fmt).spmm(_dev(X)))
        assert (_bits(Y) == _bits(X)).all(), fmt


# ------------------------------------------------------------ error paths

def test_invalid_coo_errors():
    R = C = 8
    def build(r, c, v):
        return gs.build_format(_dev(np.array(r, np.int32)), _dev(np.array(c, np.int32)),
                               _dev(np.array(v, np.float32)), (R, C), "csr")
    for (r, c, v), code in [
        (([0, 8], [0, 0], [1, 1]), gs.ERR_INDEX),
        (([0, 1], [0, -1], [1, 1]), gs.ERR_INDEX),
        (([0, 1], [0, 1], [1, -0.0]), gs.ERR_EXPLICIT_ZERO),
        (([1, 0, 1], [2, 0, 2], [1, 1, 2]), gs.ERR_DUPLICATE),
        (([1, 1, 9], [2, 2, 0], [0, 1, 1]), gs.ERR_INDEX),
        (([1, 1], [2, 2], [0, 1]), gs.ERR_EXPLICIT_ZERO),
    ]:
        with pytest.raises(gs.GnnSpmmError) as e:
            build(r, c, v)
        assert e.value.code == code
        with pytest.raises(oracle.OracleError) as eo:  # the oracle agrees
            oracle.canon(R, C, r, c, v)
        assert eo.value.code == code


def _offset_dev(a, off):
    # a on the device, starting `off` elements into its allocation
    t = torch.from_numpy(np.ascontiguousarray(a))
    buf = torch.empty(a.size + off, dtype=t.dtype, device=DEV)
    buf[off:] = t.to(DEV)
    return buf[off:]


@pytest.mark.parametrize("off", [0, 1])
def test_validation_at_every_quad_position(off):
    # the validation reads four entries per thread through 16-byte loads when
    # the three arrays are 16-byte aligned (off = 0), one at a time otherwise
    # (off = 1): an error at any position of a quad, across a quad boundary
    # or in the ragged tail is found, with the oracle's code
    n = 4099
    R = C = n
    base_r = np.arange(n, dtype=np.int32)
    base_c = np.arange(n, dtype=np.int32)
    base_v = np.ones(n, np.float32)
    for pos in (0, 1, 2, 3, 4, 7, 2048, 4096, 4098):
        for kind in ("index", "zero", "order"):
            r, c, v = base_r.copy(), base_c.copy(), base_v.copy()
            if kind == "index":
                c[pos] = C
            elif kind == "zero":
                v[pos] = 0.0
            else:  # entry pos repeats its predecessor's (row, col): unsorted / duplicate
                q = pos if pos > 0 else 1
                r[q], c[q] = r[q - 1], c[q - 1]
            with pytest.raises(oracle.OracleError) as eo:
                oracle.canon(R, C, r, c, v)
            d = [_offset_dev(x, off) for x in (r, c, v)]
            assert (d[0].data_ptr() % 16 == 0) == (off == 0)
            with pytest.raises(gs.GnnSpmmError) as e:
                gs.build_format(*d, (R, C), "csr")
            assert e.value.code == eo.value.code, (pos, kind)
            if kind == "order":  # sorted input promised, then broken
                with pytest.raises(gs.GnnSpmmError):
                    gs.build_format(*d, (R, C), "csr", assume_canonical=True)


@pytest.mark.parametrize("shuffle", [False, True])
def test_unaligned_coo_arrays_build_the_same_matrix(shuffle):
    g = graphgen.scaled(2)
    case = _case_from_graph(g, shuffle_seed=12 if shuffle else None)
    case.d_row, case.d_col, case.d_val = (_offset_dev(x, 1) for x in (case.row, case.col, case.val))
    for fmt in ("csr", "coo", "ell", "bsr"):
        check_layout(case, fmt)
    check_features(case)


def test_infeasible_padded_format_reports_bytes():
    R, C = 2000, 2000
    row, col, val = graphgen.dense_rows_coo(R, C, [5], seed=4, base_nnz=4000)
    case = Case(R, C, row, col, val)
    with pytest.raises(gs.GnnSpmmError) as e:
        case.build("ell", max_bytes=1 << 20)
    assert e.value.code == gs.ERR_INFEASIBLE
    assert e.value.bytes_required == 8 * R * C  # K = C (row 5 is dense)


def test_spmm_argument_errors():
    case = _random_case(50, 40, 200, 5)
    m = case.build("csr")
    X = torch.zeros((40, 8), device=DEV)
    with pytest.raises(ValueError):
        m.spmm(torch.zeros((39, 8), device=DEV))
    Y = torch.zeros((50, 8), device=DEV)
    rc = gs.lib().gs_spmm(m.handle, X.data_ptr(), 8, Y.data_ptr(), 4, 8, None)
    assert rc == gs.ERR_INVALID_ARG  # ldy < F
    big = torch.zeros((100, 8), device=DEV)
    rc = gs.lib().gs_spmm(m.handle, big.data_ptr(), 8, big[10:].data_ptr(), 8, 8, None)
    assert rc == gs.ERR_INVALID_ARG  # X and Y overlap
    # rejected before any device access: a width past 2^24 columns, and a
    # leading dimension whose span overflows 64-bit byte offsets
    F = (1 << 24) + 1
    rc = gs.lib().gs_spmm(m.handle, X.data_ptr(), F, Y.data_ptr(), F, F, None)
    assert rc == gs.ERR_UNSUPPORTED
    rc = gs.lib().gs_spmm(m.handle, X.data_ptr(), 1 << 61, Y.data_ptr(), 8, 8, None)
    assert rc == gs.ERR_INVALID_ARG


def test_buffers_return_to_the_hooks_that_allocated_them():
    # a handle built (and given a workspace) under one set of allocator hooks
    # and destroyed after the hooks changed returns every buffer to the hooks
    # that allocated it
    live, errors = {}, []

    def _alloc(n, stream, _ctx):
        p = torch.cuda.caching_allocator_alloc(int(n), stream=int(stream or 0))
        live[p] = n
        return p

    def _free(p, _stream, _ctx):
        if p not in live:
            errors.append(p)
            return
        del live[p]
        torch.cuda.caching_allocator_delete(int(p))

    gs._require_gpu()  # the binding installs its own hooks on first use: do that before replacing them
    hooks = gs._Allocator(gs._ALLOC_FN(_alloc), gs._FREE_FN(_free), None)
    assert gs.lib().gs_set_allocator(ctypes.byref(hooks)) == 0
    try:
        case = _random_case(300, 310, 2500, 41)
        m = case.build("coo")
        check_spmm(case, m, graphgen.features_x(case.C, 64, 42, "normal"))
    finally:
        # the binding's own hooks, the same objects: buffers they allocated
        # earlier must find them alive when freed
        assert gs.lib().gs_set_allocator(ctypes.byref(gs._alloc_keep[0])) == 0
    assert live  # the handle holds its arrays and workspace
    m.close()
    torch.cuda.synchronize()
    assert not live and not errors
    check_spmm(case, case.build("csr"), graphgen.features_x(case.C, 8, 43, "normal"))


def test_allocation_failure_is_reported_and_recovers():
    # an allocator that returns NULL: the calls that need memory report
    # GS_ERR_OOM and leave no half-made buffer behind, so once allocation
    # works again the same handle builds its workspace and computes correctly
    gs._require_gpu()
    case = Case(3000, 2800, *graphgen.dense_rows_coo(3000, 2800, [5, 1700], seed=71, base_nnz=60000))
    m = case.build("coo")
    X = graphgen.features_x(case.C, 64, 72, "normal")
    Xd = _dev(X)
    refuse = {"on": True}

    def _alloc(n, stream, _ctx):
        if refuse["on"]:
            return None
        return torch.cuda.caching_allocator_alloc(int(n), stream=int(stream or 0))

    def _free(p, _stream, _ctx):
        torch.cuda.caching_allocator_delete(int(p))

    hooks = gs._Allocator(gs._ALLOC_FN(_alloc), gs._FREE_FN(_free), None)
    assert gs.lib().gs_set_allocator(ctypes.byref(hooks)) == 0
    m2 = None
    try:
        with pytest.raises(gs.GnnSpmmError) as e1:  # partial sums of the dense rows' chunks
            m.spmm(Xd)
        with pytest.raises(gs.GnnSpmmError) as e2:  # a whole build
            case.build("csr")
        assert e1.value.code == gs.ERR_OOM and e2.value.code == gs.ERR_OOM
        del e1, e2
        refuse["on"] = False
        check_spmm(case, m, X)
        m2 = case.build("csr")
        check_spmm(case, m2, X)
    finally:
        # buffers go back through the hooks that made them: every handle that
        # allocated through these hooks is destroyed while they still exist
        m.close()
        if m2 is not None:
            m2.close()
        torch.cuda.synchronize()
        # the binding's own hooks, the same objects: buffers they allocated
        # earlier must find them alive when freed
        assert gs.lib().gs_set_allocator(ctypes.byref(gs._alloc_keep[0])) == 0


def test_work_stays_on_the_callers_stream():
    # Everything on a second stream (default priority), queued behind an
    # asynchronous copy of X into a fresh buffer on that stream: builds,
    # SpMMs, a conversion, features and the selector.  A kernel launched on
    # another stream could read X before the copy lands.  Results are read
    # after synchronising that stream alone.
    case = _random_case(3000, 2800, 60000, 61)
    F = 64
    X = graphgen.features_x(case.C, F, 62, "normal")
    Xpin = torch.from_numpy(X).pin_memory()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())  # the case's arrays were copied on the default stream
    with torch.cuda.stream(s):
        Xd = torch.empty((case.C, F), device=DEV)
        Xd.copy_(Xpin, non_blocking=True)
        outs = []
        for fmt in FMTS:
            m = case.build(fmt)
            outs.append((fmt, m, m.spmm(Xd)))
        m2 = outs[0][1].convert("ell")
        outs.append(("csr->ell", m2, m2.spmm(Xd)))
        feats = gs.extract_features(case.d_row, case.d_col, case.d_val, (case.R, case.C))
        sel = []
        for mode in ("profile", "model"):
            ctx = gs.SelectContext(mode)
            sel.append((mode, ctx, *ctx.run(9, case.d_row, case.d_col, case.d_val, (case.R, case.C), Xd)))
    s.synchronize()
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    for name, _, Y in outs + [(f"select/{mode}/{fmt}", ctx, Y) for mode, ctx, Y, fmt in sel]:
        ok, worst = oracle.check_spmm(_host(Y), Yref, M)
        assert ok, f"{name}: worst |err|/bound {worst}"
    ints, f = oracle.features(case.R, case.C, case.crow, case.ccol)
    assert all(feats[k] == v for k, v in ints.items()) and feats["f"] == f.tolist()


def test_destroy_right_after_spmm_on_another_stream():
    # a handle built on the default stream, multiplied on a second stream and
    # destroyed at once: the destroy waits for that SpMM before its arrays go
    # back to the allocator, so the default stream's next allocations (which
    # may take the same memory) cannot overwrite them under the running SpMM
    gs._require_gpu()
    case = _random_case(20000, 20000, 600000, 91, empty=0.0)
    X = graphgen.features_x(case.C, 128, 92, "normal")
    Xd = _dev(X)
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    s2 = torch.cuda.Stream()
    for fmt in ("csc", "coo", "csr"):
        m = case.build(fmt)
        torch.cuda.synchronize()
        with torch.cuda.stream(s2):
            Y = m.spmm(Xd)
        m.close()
        junk = [torch.full((1 << 20,), float("nan"), device=DEV) for _ in range(16)]
        s2.synchronize()
        ok, worst = oracle.check_spmm(_host(Y), Yref, M)
        assert ok, f"{fmt}: worst |err|/bound {worst}"
        del junk


def _busy(stream):
    # tens of milliseconds of work that later calls on the stream queue behind
    with torch.cuda.stream(stream):
        torch.cuda._sleep(50_000_000)


@pytest.mark.parametrize("src", FMTS)
@pytest.mark.parametrize("dst", FMTS)
def test_destroy_waits_for_a_conversion_on_another_stream(src, dst):
    # a handle converted on a second stream behind other work, then destroyed:
    # whether or not the conversion waited for its copies, nothing of it is
    # outstanding once the source's arrays go back to the allocator
    case = _random_case(300, 310, 2500, 31)
    m = case.build(src)
    torch.cuda.synchronize()
    s2 = torch.cuda.Stream()
    _busy(s2)
    with torch.cuda.stream(s2):
        m2 = m.convert(dst)
    m.close()
    assert s2.query(), "destroyed under a conversion that still reads it"
    r, c, v = (_host(t) for t in m2.to_coo())
    assert (r == case.crow).all() and (c == case.ccol).all() and (_bits(v) == _bits(case.cval)).all()


@pytest.mark.parametrize("fmt", ["csr", "coo", "csc"])
def test_destroy_waits_for_every_stream_that_read(fmt):
    # reads on two other streams, then an SpMM on the handle's own: the
    # later record replaces neither of the earlier ones
    case = _random_case(300, 310, 2500, 32)
    m = case.build(fmt)
    Xd = _dev(graphgen.features_x(case.C, 16, 33, "normal"))
    torch.cuda.synchronize()
    others = [torch.cuda.Stream() for _ in range(2)]
    for s2 in others:
        _busy(s2)
        with torch.cuda.stream(s2):
            m.to_coo()
    m.spmm(Xd)
    m.close()
    assert all(s2.query() for s2 in others), "destroyed under a copy that still reads it"


@pytest.mark.parametrize("fmt,classes", [("coo", False), ("coo", True), ("csr", True), ("csc", False)])
def test_first_spmm_inside_a_capture(monkeypatch, fmt, classes):
    # nothing that a handle keeps may be left to the first replay: an eager
    # call between capture and replay, and every replay, give what a handle
    # that was never captured gives, bit for bit
    monkeypatch.setenv("GS_CSR_HOTCOLD", "on" if classes else "off")
    monkeypatch.setenv("GS_CSR_HOT_KB", "1")
    monkeypatch.setenv("GS_CSR_SORT", "2")
    case = Case(700, 5000, *graphgen.dense_rows_coo(700, 5000, [0, 3, 350, 699], seed=35, base_nnz=8000))
    Xd = _dev(graphgen.features_x(case.C, 64, 36, "normal"))
    X2 = _dev(graphgen.features_x(case.C, 64, 37, "normal"))
    plain = case.build(fmt)
    want, want2 = _bits(_host(plain.spmm(Xd))), _bits(_host(plain.spmm(X2)))
    m = case.build(fmt)
    Xs, out = Xd.clone(), torch.empty((case.R, 64), device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.spmm(Xs, out=out)
    assert (_bits(_host(m.spmm(Xd))) == want).all()
    for x, w in ((Xd, want), (X2, want2), (Xd, want)):
        Xs.copy_(x)
        out.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert (_bits(_host(out)) == w).all()
        assert (_bits(_host(m.spmm(X2))) == want2).all()


# -------------------------------------------------------------- conversion

@pytest.mark.parametrize("src", FMTS)
def test_convert_between_formats(src):
    case = _random_case(300, 310, 2500, 31)
    m = case.build(src)
    for dst in FMTS:
        m2 = m.convert(dst)
        r, c, v = (_host(t) for t in m2.to_coo())
        assert (r == case.crow).all() and (c == case.ccol).all()
        assert (_bits(v) == _bits(case.cval)).all()
    f = m.features()
    ints, fo = oracle.features(case.R, case.C, case.crow, case.ccol)
    assert f["f"] == fo.tolist()


@pytest.mark.parametrize("dst", ["csr", "coo"])
def test_rows_made_from_csc_gather_by_class(monkeypatch, dst):
    # the row form behind a CSC handle has no reference classes; CSR and COO
    # made from it do, like those built directly: their first SpMM allocates
    # the tagged copy of the columns, and the results agree bit for bit
    monkeypatch.setenv("GS_CSR_HOTCOLD", "on")
    monkeypatch.setenv("GS_CSR_HOT_KB", "1")
    case = _random_case(523, 411, 6000, 11)
    Xd = _dev(graphgen.features_x(case.C, 64, 12, "normal"))
    out = torch.empty((case.R, 64), device=DEV)
    src = case.build("csc")
    ys, made = [], []
    for m in (case.build(dst), src.convert(dst)):
        n0 = torch.cuda.memory_stats()["allocation.all.allocated"]
        ys.append(_bits(_host(m.spmm(Xd, out=out))))
        made.append(torch.cuda.memory_stats()["allocation.all.allocated"] - n0)
    assert made == [1, 1]
    assert (ys[0] == ys[1]).all()
    ints, fo = oracle.features(case.R, case.C, case.crow, case.ccol)
    assert src.features()["f"] == fo.tolist()


@pytest.mark.parametrize("cpl", [4, 8, 16])
@pytest.mark.parametrize("sort", [1, 2])
@pytest.mark.parametrize("F", [64, 128, 256])
def test_csr_lane_shapes(monkeypatch, cpl, sort, F):
    # columns per lane and row ordering are tunable; every shape must agree,
    # with long rows (workgroup-wide path) present in both orders
    monkeypatch.setenv("GS_CSR_CPL", str(cpl))
    monkeypatch.setenv("GS_CSR_SORT", str(sort))
    g = graphgen.scaled(2)
    case = _case_from_graph(g)
    X = graphgen.features_x(case.C, F, 50 + F, "normal")
    check_spmm(case, case.build("csr"), X)


@pytest.mark.parametrize("thr,chunk,wg", [(32, 32, 64), (16, 8, 100000), (200, 64, 201), (128, 128, 1024)])
@pytest.mark.parametrize("sort", ["1", "2"])
def test_csr_plan_thresholds(monkeypatch, thr, chunk, wg, sort):
    # the device-built work plan under different long-row / chunk / workgroup
    # thresholds: short, medium and huge rows in every mix, both row orders
    monkeypatch.setenv("GS_CSR_LONG_ROW", str(thr))
    monkeypatch.setenv("GS_CSR_CHUNK", str(chunk))
    monkeypatch.setenv("GS_CSR_WG_ROW", str(wg))
    monkeypatch.setenv("GS_CSR_SORT", sort)
    g = graphgen.scaled(2)
    case = _case_from_graph(g)
    check_spmm(case, case.build("csr"), g.X[:, :64])
    R, C = 700, 5000
    row, col, val = graphgen.dense_rows_coo(R, C, [0, 3, 350, 699], seed=23, base_nnz=8000)
    case = Case(R, C, row, col, val)
    m = case.build("csr")
    check_spmm(case, m, graphgen.features_x(C, 36, 24, "normal"))
    # several column slices (one completion count per huge row and slice),
    # then a narrower call on the same handle
    check_spmm(case, m, graphgen.features_x(C, 300, 25, "normal"))
    check_spmm(case, m, graphgen.features_x(C, 20, 26, "normal"))


@pytest.mark.parametrize("hot_kb", ["1", "16", "64"])
@pytest.mark.parametrize("sort", ["1", "2"])
def test_csr_reference_classes(monkeypatch, hot_kb, sort):
    # gathers chosen by the column's reference class: a small hot budget puts
    # most X rows on the non-temporal path.  The class tags live in a copy of
    # the column indices, so the handle's arrays stay canonical, and the load
    # kind changes no result: Y equals the untagged path's bit for bit.
    monkeypatch.setenv("GS_CSR_SORT", sort)
    monkeypatch.setenv("GS_CSR_HOTCOLD", "off")
    g = graphgen.scaled(2)
    case = _case_from_graph(g)
    plain = case.build("csr")
    monkeypatch.setenv("GS_CSR_HOTCOLD", "on")
    monkeypatch.setenv("GS_CSR_HOT_KB", hot_kb)
    m = check_layout(case, "csr")
    for F in (64, 128, 132):
        X = graphgen.features_x(case.C, F, 70 + F, "normal")
        check_spmm(case, m, X)
        Xd = _dev(X)
        assert (_bits(_host(m.spmm(Xd))) == _bits(_host(plain.spmm(Xd)))).all()
    # hub rows of every tier with the classes on
    R, C = 700, 5000
    row, col, val = graphgen.dense_rows_coo(R, C, [0, 3, 350, 699], seed=27, base_nnz=8000)
    case = Case(R, C, row, col, val)
    check_spmm(case, case.build("csr"), graphgen.features_x(C, 64, 28, "normal"))


@pytest.mark.parametrize("fmt,F,off", [("csr", 47, 0), ("csr", 64, 1), ("csr", 131, 0), ("csr", 7, 2), ("coo", 64, 0),
                                       ("coo", 128, 0), ("coo", 256, 0), ("coo", 130, 0)])
@pytest.mark.parametrize("group_min", ["100000", "100"])
def test_reference_classes_in_chains_of_four(monkeypatch, fmt, F, off, group_min):
    # gathers by class and the group tier where rows are summed in chains of
    # four: within the bound of the oracle, and bit for bit the sums of plain
    # gathers, which keep other numbers of X rows in flight
    monkeypatch.setenv("GS_CSR_SORT", "2")
    monkeypatch.setenv("GS_CSR_GROUP_MIN", group_min)
    case = _uniform_long_rows(500, 3000, 0, 300, 710 + F, hubs=(3, 499))
    X = graphgen.features_x(case.C, F, 711, "normal")
    Xd = torch.zeros((case.C, F + off), device=DEV)
    Xd[:, off:] = _dev(X)
    ys = []
    for classes in ("off", "on"):
        monkeypatch.setenv("GS_CSR_HOTCOLD", classes)
        monkeypatch.setenv("GS_CSR_HOT_KB", "16")
        ys.append(_host(case.build(fmt).spmm(Xd[:, off:])))
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    ok, worst = oracle.check_spmm(ys[0], Yref, M)
    assert ok, worst
    assert (_bits(ys[0]) == _bits(ys[1])).all()


@pytest.mark.parametrize("T,h", [("32", "0"), ("64", "1"), ("256", "1"), ("96", "0")])
def test_csr_lds_window_tiles(monkeypatch, T, h):
    # row tiles with their X window staged in LDS: communities of consecutive
    # nodes and a stencil (entries inside and outside the window), tiles cut
    # across communities (96 rows), ragged last tile, several column slices,
    # strided operands, rectangular matrices whose windows run past the last
    # column or are empty
    monkeypatch.setenv("GS_CSR_WIN_T", T)
    monkeypatch.setenv("GS_CSR_WIN_H", h)
    for k in (4, 3):
        g = graphgen.scaled(k)
        case = _case_from_graph(g)
        m = case.build("csr")
        check_spmm(case, m, g.X)
        check_spmm(case, m, graphgen.features_x(case.C, 36, 80 + k, "normal"), ldx_pad=4, ldy_pad=8)
        check_spmm(case, m, graphgen.features_x(case.C, 520, 90 + k, "normal"))
    for R, C, seed in ((1003, 517, 81), (517, 1003, 82), (2000, 2000, 83)):
        case = _random_case(R, C, 9000, seed, empty=0.2)
        m = case.build("csr")
        check_spmm(case, m, graphgen.features_x(C, 64, seed + 5, "normal"))
        check_spmm(case, m, graphgen.features_x(C, 132, seed + 6, "normal"))


@pytest.mark.parametrize("T,h", [("", ""), ("32", "0"), ("64", "1"), ("96", "0")])
def test_ell_lds_window_tiles(monkeypatch, T, h):
    # ELL rows of one tile with their X window staged in LDS (the tile the
    # counts pick, or a forced one): communities, a stencil, ragged tiles,
    # several column slices, strided operands, rectangular matrices
    if T:
        monkeypatch.setenv("GS_CSR_WIN_T", T)
        monkeypatch.setenv("GS_CSR_WIN_H", h)
    for k in (4, 3):
        g = graphgen.scaled(k)
        case = _case_from_graph(g)
        m = check_layout(case, "ell")
        check_spmm(case, m, g.X)
        check_spmm(case, m, graphgen.features_x(case.C, 36, 180 + k, "normal"), ldx_pad=4, ldy_pad=8)
        check_spmm(case, m, graphgen.features_x(case.C, 520, 190 + k, "normal"))
    for R, C, seed in ((1003, 517, 181), (517, 1003, 182)):
        case = _random_case(R, C, 9000, seed, empty=0.2)
        m = case.build("ell")
        check_spmm(case, m, graphgen.features_x(C, 64, seed + 5, "normal"))
        check_spmm(case, m, graphgen.features_x(C, 132, seed + 6, "normal"))


@pytest.mark.parametrize("P", [2, 5])
def test_column_panel_schedule_sums_to_the_product(P):
    # the column-panel schedule that bench.py --column-panels measures: one
    # CSR handle per column range, passes summed in panel order.  Rows are cut
    # across panels, and the first panel holds no entry.
    R, C = 1500, 2000
    row, col, val = graphgen.random_coo(R, C, 24000, 91, empty_rows=0.1)
    bounds = [C * p // P for p in range(P + 1)]
    keep = col >= bounds[1]
    case = Case(R, C, row[keep], col[keep], val[keep])
    X = graphgen.features_x(C, 64, 92, "normal")
    Xd = _dev(X)
    Y = torch.zeros((R, 64), dtype=torch.float32, device=DEV)
    for p in range(P):
        c0, c1 = bounds[p], bounds[p + 1]
        sel = (case.d_col >= c0) & (case.d_col < c1)
        assert p > 0 or int(sel.sum()) == 0
        m = gs.build_format(case.d_row[sel], case.d_col[sel] - c0, case.d_val[sel], (R, c1 - c0), "csr")
        Y += m.spmm(Xd[c0:c1])
        m.close()
    Yref, M = oracle.spmm(R, case.rp, case.ccol, case.cval, X)
    ok, worst = oracle.check_spmm(_host(Y), Yref, M)
    assert ok, f"panels: worst |err|/bound = {worst}"


@pytest.mark.parametrize("dense_min", ["1", "64", "256", "300"])
@pytest.mark.parametrize("ht", ["", "1", "8"])
def test_bsr16_hybrid_plan(monkeypatch, dense_min, ht):
    # dense 16x16 blocks on the matrix cores, every other block's entries as a
    # row list: block communities (dense and sparse blocks), a stencil, random
    # matrices with R, C not multiples of 16 and empty rows; every block dense
    # (1), the default cut (64), only full blocks (256) and none (300); tiles
    # per wave forced to 1 and 8; widths over one and several column groups.
    # The block arrays stay canonical.
    monkeypatch.setenv("GS_BSR_DENSE_MIN", dense_min)
    if ht:
        monkeypatch.setenv("GS_BSR_HT", ht)
    cases = [_case_from_graph(graphgen.scaled(4)), _case_from_graph(graphgen.scaled(3)),
             _random_case(1001, 997, 12000, 63, empty=0.1)]
    for i, case in enumerate(cases):
        m = check_layout(case, "bsr", 16)
        for F in (16, 48, 272):
            check_spmm(case, m, graphgen.features_x(case.C, F, 64 + F + i, "normal"), ldx_pad=4 * (i == 2))


@pytest.mark.parametrize("F", [16, 48, 80, 512, 1040])
def test_bsr16_matrix_core_widths(monkeypatch, F):
    # 16x16 blocks run on the matrix cores for F a multiple of 16 (wide F
    # spans several workgroup column groups); R, C not multiples of 16
    monkeypatch.setenv("GS_BSR_MFMA", "1")  # force the matrix-core kernel on sparse blocks too
    case = _random_case(1001, 997, 12000, 61, empty=0.1)
    X = graphgen.features_x(case.C, F, 62, "normal")
    check_spmm(case, case.build("bsr", 16), X)


def test_bsr16_dense_blocks_match_generic(monkeypatch):
    # block-community structure: full 16x16 diagonal blocks plus sparse ones
    g = graphgen.scaled(4)
    case = _case_from_graph(g)
    m = case.build("bsr", 16)
    monkeypatch.setenv("GS_BSR_MFMA", "1")
    w1 = check_spmm(case, m, g.X)
    monkeypatch.setenv("GS_BSR_GENERIC", "1")
    w2 = check_spmm(case, m, g.X)
    assert w1 <= 1.0 and w2 <= 1.0


# --------------------------------------------------------------- selection

@pytest.mark.parametrize("mode", ["model", "profile", "fixed"])
def test_select_and_run_modes(mode):
    # every selection mode must return A.X (in whatever format it picks),
    # convert at most once per key, and report what it chose
    g = graphgen.scaled(3)
    case = _case_from_graph(g)
    ctx = gs.SelectContext(mode, fixed="ell")
    shape = (case.R, case.C)
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, g.X)
    X = _dev(g.X)
    seen = set()
    for _ in range(3):
        Y, fmt = ctx.run(7, case.d_row, case.d_col, case.d_val, shape, X)
        ok, worst = oracle.check_spmm(_host(Y), Yref, M)
        assert ok, (mode, fmt, worst)
        seen.add(fmt)
    assert len(seen) == 1
    st = ctx.stats()
    assert st["chosen"] == fmt and st["feasible_mask"] & (1 << gs.FORMATS[fmt])
    if mode == "fixed":
        assert fmt == "ell"
    if mode == "profile":  # the reference selector keeps the fastest measured format
        times = {k: v for k, v in st["scores"].items() if v > 0}
        assert min(times.values()) * 1.0101 >= times[fmt]
    # a different width re-decides but reuses the cached features
    X2 = _dev(graphgen.features_x(case.C, 16, 5))
    Yref2, M2 = oracle.spmm(case.R, case.rp, case.ccol, case.cval, _host(X2))
    Y2, _ = ctx.run(7, case.d_row, case.d_col, case.d_val, shape, X2)
    assert oracle.check_spmm(_host(Y2), Yref2, M2)[0]


def _footprints(f, b=16):
    # device bytes of each candidate layout, the memory term M of Eq. 1
    R, C, Z = f["n_rows"], f["n_cols"], f["nnz"]
    return {"csr": 4 * (R + 1) + 8 * Z, "coo": 12 * Z, "ell": 8 * R * f["max_rd"],
            "dia": 4 * f["n_diags"] * (R + 1), "bsr": 4 * (-(-R // b) + 1) + (12 + 4 * b * b) * f["n_blocks16"],
            "csc": 4 * (C + 1) + 8 * Z}


@pytest.mark.parametrize("kind", ["mesh", "uniform"])
def test_profile_selection_trades_time_for_memory(kind):
    # Eq. 1 in the exhaustive mode: with mem_weight 1 (w = 0) the smallest
    # footprint wins (DIA on a stencil, ELL on rows of one length); with 0.5
    # the chosen format's objective, from the measured times and the
    # footprints, min-max scaled over the candidates, is within 1e-4 of the
    # smallest.  The result is A.X either way.
    if kind == "mesh":
        g = graphgen.scaled(3)
        case, X = _case_from_graph(g), g.X
    else:
        case = _uniform_long_rows(3000, 3000, 12, 12, 95)
        X = graphgen.features_x(case.C, 64, 96, "normal")
    shape = (case.R, case.C)
    foot = _footprints(gs.extract_features(case.d_row, case.d_col, case.d_val, shape))
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, X)
    order = ["csr", "coo", "ell", "dia", "bsr", "csc"]
    for mw in (1.0, 0.5):
        ctx = gs.SelectContext("profile", mem_weight=mw)
        Y, fmt = ctx.run(3, case.d_row, case.d_col, case.d_val, shape, _dev(X))
        assert oracle.check_spmm(_host(Y), Yref, M)[0]
        st = ctx.stats()
        cand = [f for f in order if st["feasible_mask"] & (1 << gs.FORMATS[f]) and st["scores"][f] > 0]
        t = {f: st["scores"][f] for f in cand}
        w = 1.0 - mw
        sc = lambda v, d: (v - min(d.values())) / (max(d.values()) - min(d.values()))  # noqa: E731
        O = {f: w * sc(t[f], t) + (1 - w) * sc(foot[f], {k: foot[k] for k in cand}) for f in cand}
        assert O[fmt] <= min(O.values()) + 1e-4, (mw, fmt, O)
        if mw == 1.0:
            assert fmt == {"mesh": "dia", "uniform": "ell"}[kind]
        ctx.close()


def test_fixed_selector_reports_an_infeasible_format():
    # the fixed mode extracts no features; the build itself reports the cap
    g = graphgen.scaled(2)
    case = _case_from_graph(g)
    ctx = gs.SelectContext("fixed", fixed="dia", max_bytes=1 << 20)
    with pytest.raises(gs.GnnSpmmError) as e:
        ctx.run(9, case.d_row, case.d_col, case.d_val, (case.R, case.C), _dev(g.X[:, :16]))
    assert e.value.code == gs.ERR_INFEASIBLE
    ctx.close()


@pytest.mark.parametrize("mode", ["model", "profile"])
def test_select_respects_candidate_formats(mode):
    g = graphgen.scaled(3)
    case = _case_from_graph(g)
    ctx = gs.SelectContext(mode, formats=["coo", "ell"])
    Y, chosen = ctx.run(5, case.d_row, case.d_col, case.d_val, (case.R, case.C), _dev(g.X))
    assert chosen in ("coo", "ell")
    Yref, M = oracle.spmm(case.R, case.rp, case.ccol, case.cval, g.X)
    assert oracle.check_spmm(_host(Y), Yref, M)[0]
    ctx.close()


def test_select_model_on_mesh_prefers_diagonals():
    g = graphgen.scaled(3)
    case = _case_from_graph(g)
    ctx = gs.SelectContext("model", model_path="builtin")  # the hand-set trees
    assert ctx.select(1, case.d_row, case.d_col, case.d_val, (case.R, case.C), 64) == "dia"


def test_library_predictor_matches_the_training_code():
    # the library's predictor (feature vector, fp32-rounded min-max scaling,
    # tree walk, tie order) against the training code's own definition of
    # each step, on the shipped model: equal scores, the same choice
    from paper_2111_00352_amd.selector import MODEL_PATH, train
    mn, mx, base, classes, trees = train.read_model(MODEL_PATH)
    names = {v: k for k, v in gs.FORMATS.items()}
    tie = ["csr", "coo", "ell", "dia", "bsr", "csc"]
    cases = [_case_from_graph(graphgen.scaled(k)) for k in (1, 2, 3, 4, 5)]
    cases += [_random_case(3000, 5000, 40000, 141), _random_case(20000, 20000, 9000, 142, empty=0.5)]
    key = 0
    for case in cases:
        feats = gs.extract_features(case.d_row, case.d_col, case.d_val, (case.R, case.C))
        for F in (8, 64, 128, 256):
            key += 1
            x = np.array([train.model_input(feats["f"], feats["n_blocks16"], F)])
            S = train.score_exported(trees, base, train.normalise(x, mn, mx))[0]
            ctx = gs.SelectContext("model")
            got = ctx.select(key, case.d_row, case.d_col, case.d_val, (case.R, case.C), F)
            st = ctx.stats()
            ctx.close()
            feasible = [n for n in tie if st["feasible_mask"] >> gs.FORMATS[n] & 1]
            score = {names[fmt]: S[k] for k, fmt in enumerate(classes)}
            for n in feasible:
                if n in score:
                    assert st["scores"][n] == score[n], (case.R, F, n)
            cand = [n for n in feasible if n in score]
            best = max(score[n] for n in cand)
            assert got == next(n for n in cand if score[n] == best), (case.R, F)


def test_trained_model_choice_is_near_the_profiled_best():
    # the shipped ensemble against the exhaustive selector (the paper's
    # oracle, Sec. 6.3) on inputs it was not trained on: the five scaled
    # workloads at their own widths.  The chosen format's time over the
    # fastest one's, geometric mean at least 0.9 and none below 0.75.
    ratios = []
    for k in (1, 2, 3, 4, 5):
        g = graphgen.scaled(k)
        case = _case_from_graph(g)
        X = _dev(g.X)
        shape = (case.R, case.C)
        prof = gs.SelectContext("profile", profile_reps=10)
        prof.run(1, case.d_row, case.d_col, case.d_val, shape, X)
        times = {f: t for f, t in prof.stats()["scores"].items() if t > 0}
        chosen = gs.SelectContext("model").select(1, case.d_row, case.d_col, case.d_val, shape, g.F)
        ratios.append(min(times.values()) / times[chosen])
    assert np.exp(np.mean(np.log(ratios))) >= 0.9, ratios
    assert min(ratios) >= 0.75, ratios


@pytest.mark.parametrize("path", ["lds", "global", "windows1", "windows64"])
def test_diagonal_bitmap_paths_agree(monkeypatch, path):
    # the per-workgroup LDS bitmap, the global-atomic bitmap and the bitmap in
    # LDS windows (forced here to windows of 1 and 64 words, many per matrix)
    # must give the same diagonal set (features N_diags and the DIA layout)
    if path == "global":
        monkeypatch.setenv("GS_DIAG_GLOBAL", "1")
    if path.startswith("windows"):
        monkeypatch.setenv("GS_DIAG_WIN_WORDS", path[len("windows"):])
    for case in (_random_case(3001, 2500, 20000, 91), _random_case(300, 7000, 9000, 92, empty=0.3),
                 _case_from_graph(graphgen.scaled(3), shuffle_seed=93)):
        check_features(case)
        check_layout(case, "dia")


@pytest.mark.parametrize("path", ["windows", "global"])
def test_wide_diagonal_bitmap(monkeypatch, path):
    # a span of 1.6 million diagonals and 700,001 rows is too wide for one
    # LDS bitmap: it is marked in LDS windows of the bitmap (default) or with
    # global atomics, each wave's batches of entries in flight
    if path == "global":
        monkeypatch.setenv("GS_DIAG_GLOBAL", "1")
    check_features(_random_case(700_001, 900_000, 1_100_000, 96, empty=0.1))


@pytest.mark.parametrize("path", ["bucketed", "atomic"])
def test_column_count_paths_agree(monkeypatch, path):
    # bucketed LDS counting (over a million entries, several 32k-column
    # windows, a ragged last window) and the atomic histogram give the same
    # column features
    if path == "atomic":
        monkeypatch.setenv("GS_COLHIST_ATOMIC", "1")
    check_features(_random_case(50_000, 70_001, 1_200_000, 95, empty=0.05))


@pytest.mark.parametrize("C,nnz", [(32_767, 16_384), (32_769, 16_383), (262_144, 70_000), (262_145, 70_000),
                                   (70_001, 4_300_000)])
def test_column_counts_by_windows(C, nnz):
    # the column counts around the limits of their three paths: one window
    # short of full, one column into the second, all eight, one over (atomics)
    # and more entries than are read once per window (bucketed)
    check_features(_random_case(20_000, C, nnz, 96))


@pytest.mark.parametrize("C", [1, 255, 256, 257, 70_000])
@pytest.mark.parametrize("n", [2_047, 2_048, 2_049, 20_000])
def test_sort_and_scan_at_tile_edges(n, C):
    # the radix sort's tiles hold 2,048 keys, the scan's 2,048 values: counts
    # around them, column indices around one digit, an unsorted input
    R = max(2 * n // C, 3)
    case = _random_case(R, C, min(n, R * C), 97)
    case.d_row, case.d_col, case.d_val = (_dev(a) for a in graphgen.shuffled(case.crow, case.ccol, case.cval, 98))
    for fmt in ("csr", "csc", "coo"):
        check_layout(case, fmt)


@pytest.mark.parametrize("merge", ["0", "1"])
def test_block_count_kernels_agree(monkeypatch, merge):
    # the 16x16 block count (features, BSR sizing) has an LDS-bitmap kernel and
    # a merge kernel for very wide matrices; both must give the oracle's count
    monkeypatch.setenv("GS_BLOCK_COUNT_MERGE", merge)
    for k in (2, 4):
        case = _case_from_graph(graphgen.scaled(k))
        check_features(case)
        check_layout(case, "bsr", 16)
    case = _random_case(777, 3001, 20000, 71)
    check_features(case)
    for b in (3, 16, 64):
        check_layout(case, "bsr", b)
    # wide and sparse: block rows hold fewer entries than the bitmap has
    # words, so the count clears only the words its entries touched
    case = _random_case(300, 200003, 3000, 72, empty=0.3)
    check_features(case)
    check_layout(case, "bsr", 16)
