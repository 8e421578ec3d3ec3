"""GPU solvers, searches and products at the sizes where their kernels change.

Blocks of every size class (four-lane, 4 x 4-grid, workgroup-inverse and FP64
solvers), the searches of distance 3 and more, chunks of small batches, the
compact adjacency's tiles, repeated calls whose sizes change under one shape,
and the transposes and products at their row-length limits.  All against the
oracle (or the exact transpose, or ``dense.product_reference``) with the gates
of tests/_util.py: pattern identical, row error <= 1e-10, constraint residual
<= 1e-12 of its terms.  The generated systems are strictly diagonally dominant
(condition numbers below 100), so FP64-refined rows are good to about 1e-14 and
1e-10 is a gate on the method, not on rounding.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
from oracle import dense
from paper_2307_00229_amd import problems as P

from ._util import ROW_TOL, assert_matches_oracle, gpu_build, row_errors, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2307_00229_amd import clair

    clair.load_library()


def _problem(name, M, cf, B, ell, **kw):
    M = sp.csr_matrix(M)
    M.sort_indices()
    return P.Problem(name, M.shape[0], M.indptr.astype(np.int32), M.indices.astype(np.int32),
                     M.data.astype(np.float64), cf.astype(np.int8), B, ell, **kw)


def _groups(sizes, seed, deg=4, ell=1, with_B=True):
    """One C-point per entry of ``sizes``, connected to that many F-points (so
    |N| = size at distance 1); consecutive groups share an F-point, and every
    F-point couples to up to ``deg`` others of its group."""
    rng = np.random.default_rng(seed)
    rows, cols, cf = [], [], []
    last = None
    for s in sizes:
        fresh = s - 1 if (last is not None and s > 1) else s
        base = len(cf)
        at_c = int(rng.integers(0, fresh + 1))  # the C-point lies anywhere in its group
        ids = list(range(base, base + fresh + 1))
        c = ids.pop(at_c)
        cf.extend([0] * (fresh + 1))
        cf[c] = 1
        if fresh < s:
            ids = [last] + ids
        for f in ids:
            rows += [c, f]
            cols += [f, c]
            others = [x for x in ids if x != f]
            for x in rng.permutation(others)[:deg]:
                rows.append(f)
                cols.append(int(x))
        if ids:
            last = ids[-1]
    n = len(cf)
    M = sp.coo_matrix((-rng.uniform(0.1, 1.0, len(rows)), (rows, cols)), shape=(n, n)).tocsr()
    M.sum_duplicates()
    off = np.asarray(abs(M).sum(axis=1)).ravel()
    M = (M + sp.diags(1.5 * off + 1.0)).tocsr()
    B = rng.uniform(0.5, 1.5, n) if with_B else None
    return _problem(f"groups_{min(sizes)}_{max(sizes)}_d{deg}", M, np.asarray(cf), B, ell)


def _check(ps, **kw):
    res, infos, st = gpu_build(ps, **kw)
    assert st == 0, infos
    for p, g, inf in zip(ps, res, infos):
        assert_matches_oracle(p, g, oracle.build_R_problem(p), inf)
    return infos


# rows of A of up to 3, exactly 5, 6 and more than 9 entries
@pytest.mark.parametrize("deg", [1, 3, 4, 12])
@pytest.mark.parametrize("group", [1, 4, 8])
def test_small_rows(group, deg):
    from paper_2307_00229_amd import clair

    ctx = clair.Context()
    ctx.set_tuning(group=group)
    _check([_groups([0, 1, 2, 3, 4, 5, 6, 7, 8] * 23 + [8, 0], 7 + deg, deg)], ctx=ctx)


@pytest.mark.parametrize("top", [9, 12, 13, 16, 17, 20, 21, 24, 25, 28, 29, 32])
@pytest.mark.parametrize("group", [4, 16, 32])
def test_tile_rows(group, top):
    """The largest block of a call picks the tile; smaller rows are padded."""
    from paper_2307_00229_amd import clair

    ctx = clair.Context()
    ctx.set_tuning(group=group)
    p = _groups([top, 0, 9, top - 1, 3, top, 10, 8, 1] * 7, 100 + top, deg=11 if top % 2 else 5)
    assert _check([p, p], ctx=ctx)[0]["max_block"] == max(top, 10)  # sizes read back
    _check([p], ctx=ctx)  # and known


@pytest.mark.parametrize("sizes,deg", [([33, 48, 49, 64], 6), ([65, 112, 113, 128], 6), ([129, 40, 150, 5], 6),
                                       ([127, 96, 33], 200)])
def test_wide_rows(sizes, deg):
    _check([_groups(sizes * 3, 11, deg), _groups(sizes[:1], 12, deg)])


def test_wide_rows_plan_twice():
    from paper_2307_00229_amd import clair

    p = _groups([33, 8, 64, 65, 20, 128, 130], 21, 6)
    As, cfs, Bs, ells = to_device([p])
    o0 = oracle.build_R_problem(p)
    ctx = clair.Context()
    plan = clair.Plan(ctx, As, cfs, ells, [clair.ROut(o0["n_c"], o0["nnz"])])
    for scale in (1.0, 3.0, 1.0):
        q = P.Problem(p.name, p.n, p.row_ptr, p.col_idx,
                      p.val * (1.0 + (scale - 1.0) * (np.arange(p.nnz) % 3 == 0) * 0.01), p.cf, p.B * scale, p.ell)
        A2, _, B2, _ = to_device([q])
        infos, st = plan.execute(A2, B2)
        rp, ci, va = (x.cpu().numpy() for x in plan.outs[0].trimmed())
        g = dict(row_ptr=rp, col_idx=ci, val=va, n_c=plan.outs[0].n_c, nnz=plan.outs[0].nnz)
        assert_matches_oracle(q, g, oracle.build_R_problem(q), infos[0])
    plan.close()


@pytest.mark.parametrize("mode", [0, 4, 8])
@pytest.mark.parametrize("ell", [3, 5])
def test_far_searches(ell, mode):
    from paper_2307_00229_amd import clair

    ctx = clair.Context()
    ctx.set_search_adjacency(mode)
    grid = P.small_2d(31, stencil=9, eps=0.05, angle=1.0, k=4, ell=ell)
    rnd = P.random_sparse(300, 0.012, 3, ell=ell, c_frac=0.4)  # points of more than 8 edges
    _check([grid, rnd], ctx=ctx)
    ctx.set_literal_pattern(True)
    res, infos, st = gpu_build([grid, rnd], ctx=ctx)
    assert st == 0
    for p, g, inf in zip([grid, rnd], res, infos):
        assert_matches_oracle(p, g, oracle.build_R_problem(p, literal=True), inf)


@pytest.mark.parametrize("ell", [1, 2])
def test_small_batches(ell):
    """Batches of fewer chunks than CUs use smaller chunks: matrices below, at
    and above a chunk, and of one point."""
    ps = []
    for n in (1, 2, 63, 64, 65, 127, 129, 1000, 4099):
        rng = np.random.default_rng(n)
        M = sp.diags([-rng.uniform(0.2, 1, n), np.full(n, 2.5), -rng.uniform(0.2, 1, n)], [-1, 0, 1], shape=(n, n))
        ps.append(_problem(f"line_{n}", M, (np.arange(n) % 3 == 1) | (n == 1), rng.uniform(0.5, 1.5, n), ell))
    _check(ps)
    for p in ps[1:6]:
        _check([p])


def test_adjacency_tiles():
    """Points whose entries span several LDS tiles, and one row longer than a
    tile (most of it C-points, so that no neighbourhood passes the limit)."""
    n = 5000
    rng = np.random.default_rng(5)
    M = sp.diags([-rng.uniform(0.2, 1, n), np.zeros(n), -rng.uniform(0.2, 1, n)], [-1, 0, 1], shape=(n, n)).tolil()
    hub = 701
    cf = np.arange(n) % 4 == 0
    cf[rng.choice(n, 300, replace=False)] = True
    cf[hub] = False
    M[hub, np.nonzero(cf)[0]] = -1e-4
    M[hub, rng.choice(n, 30, replace=False)] = -1e-4
    for r in range(1024, 1280):  # 9 to 12 entries: several tiles for 256 points
        M[r, rng.choice(n, 9, replace=False)] = -0.05
    M = M.tocsr()
    M.setdiag(0)
    M.eliminate_zeros()
    M = M + sp.diags(np.asarray(abs(M).sum(axis=1)).ravel() + 1.0)
    p = _problem("hub", M, cf, rng.uniform(0.5, 1.5, n), 2)
    _check([p])


@pytest.mark.parametrize("nx,theta", [(37, 0.25), (80, 0.5), (740, 0.25)])
def test_strength_runs(nx, theta):
    """Column maxima within, across and (740^2) with four rows a thread of the
    workgroups' runs of points."""
    from paper_2307_00229_amd import clair

    p = P.small_2d(nx, stencil=5, eps=0.01, angle=0.4, ell=2)
    p.theta = theta
    ps = [p] if nx > 100 else [p, p, p]
    ctx = clair.Context()
    ctx.set_strength(theta)
    _check(ps, ctx=ctx)


def test_same_shape_other_sizes():
    """Calls of one shape (points, entries, distance) whose block sizes, bins
    and queues change from call to call: each result is the call's own."""
    from paper_2307_00229_amd import clair

    base = _groups([20, 4, 60, 2, 8, 33, 9] * 9, 31, 7, ell=2)
    rng = np.random.default_rng(8)
    cfs = [base.cf, (np.arange(base.n) % 2).astype(np.int8), (rng.random(base.n) < 0.15).astype(np.int8),
           (rng.random(base.n) < 0.9).astype(np.int8), np.ones(base.n, np.int8)]
    ps = [P.Problem(f"cf{k}", base.n, base.row_ptr, base.col_idx, base.val, cf, base.B, 2)
          for k, cf in enumerate(cfs)]
    want = [oracle.build_R_problem(p) for p in ps]
    for first in range(len(ps)):
        ctx = clair.Context()
        for k in (first, first, 0, 1, 2, 2, 3, 4, first):
            As, cf, Bs, ells = to_device([ps[k]])
            outs = [clair.ROut(want[k]["n_c"], want[k]["nnz"])]
            outs, infos, st = clair.clair_build_R_batched(As, cf, Bs, ells, ctx=ctx, outs=outs)
            rp, ci, va = (x.cpu().numpy() for x in outs[0].trimmed())
            g = dict(row_ptr=rp, col_idx=ci, val=va, n_c=outs[0].n_c, nnz=outs[0].nnz)
            assert_matches_oracle(ps[k], g, want[k], infos[0])
        # a repeated shape with too little room still reports what it needs
        small = [clair.ROut(want[first]["n_c"], max(want[first]["nnz"] - 1, 0))]
        if want[first]["nnz"] > want[first]["n_c"]:
            As, cf, Bs, ells = to_device([ps[first]])
            _, infos, st = clair.clair_build_R_batched(As, cf, Bs, ells, ctx=ctx, outs=small, check=False)
            assert st == 2 and infos[0]["nnz"] == want[first]["nnz"]


@pytest.mark.parametrize("sizes", [[1, 8, 15, 16], [17, 31, 32, 33], [47, 48, 63, 64]])
def test_fp64_and_ilu_rows(sizes):
    p = _groups(sizes * 4, 41, 5)
    _check([p], precision=1)
    from paper_2307_00229_amd import clair

    As, cfs, Bs, ells = to_device([p])
    for inverse, code in (("ilu0", clair.CLAIR_INVERSE_ILU0), ("gmres", clair.CLAIR_INVERSE_GMRES)):
        for iters in (1, 3):
            kw = dict(krylov=4) if inverse == "gmres" else {}
            R, _, _ = clair.clair_build_R_approx(As[0], cfs[0], Bs[0], 1, iters, inverse=code, **kw)
            o = oracle.build_R_approx(p.n, p.row_ptr, p.col_idx, p.val, p.cf, p.B, 1, iters, inverse, **kw)
            rp, ci, va = (x.cpu().numpy() for x in R)
            assert np.array_equal(rp, o["row_ptr"]) and np.array_equal(ci, o["col_idx"])
            err, _, _ = row_errors(p, dict(val=va), o)
            assert err.max() <= ROW_TOL, (inverse, iters, err.max())


@pytest.mark.parametrize("widths", [[0, 1, 2, 7, 8], [9, 16, 31, 32], [33, 48, 63, 64, 65], [200, 3, 0]])
def test_products_and_transposes(widths):
    """Row lengths at the limits of the transposes' registers (8) and the
    products' hash tables."""
    from paper_2307_00229_amd import clair

    rng = np.random.default_rng(sum(widths))
    m, k = 7 * len(widths), 300
    rows, cols = [], []
    for r in range(m):
        w = widths[r % len(widths)]
        rows += [r] * w
        cols += rng.choice(k, w, replace=False).tolist()
    X = sp.csr_matrix((rng.uniform(-1, 1, len(rows)), (rows, cols)), shape=(m, k))
    Y = sp.random(k, 500, density=0.004, random_state=3, format="csr")
    Y.data -= 0.5

    def dev(M):
        M = sp.csr_matrix(M)
        M.sort_indices()
        return clair.CSR(torch.from_numpy(M.indptr.astype(np.int32)).cuda(),
                         torch.from_numpy(M.indices.astype(np.int32)).cuda(),
                         torch.from_numpy(M.data.astype(np.float64)).cuda(), n=M.shape[0])

    def host(t, shape):
        rp, ci, va = (x.cpu().numpy() for x in t)
        return sp.csr_matrix((va, ci, rp), shape=shape)

    for M in (X, Y):
        T = M.T.tocsr()
        T.sort_indices()
        G = host(clair.clair_transpose(dev(M), M.shape[1]), T.shape)
        assert np.array_equal(G.indptr, T.indptr) and np.array_equal(G.indices, T.indices)
        assert np.array_equal(G.data, T.data)
    G = host(clair.clair_spgemm(dev(X), k, dev(Y), 500), (m, 500))
    C, S = dense.product_reference(X, Y)
    assert np.array_equal(G.indptr, C.indptr) and np.array_equal(G.indices, C.indices)
    assert np.all(np.abs(G.data - C.data) <= 1e-13 * S.data + 1e-300)


def test_malformed_transpose_is_refused():
    """Row pointers that do not end at nnz, and a column out of range, are
    refused by every entry point that transposes, and outputs are left alone."""
    from paper_2307_00229_amd import clair

    p = P.small_2d(12, stencil=5, ell=1)
    A, cf, B, _ = to_device([p])
    bad_end = clair.CSR(A[0].row_ptr.clone(), A[0].col_idx, A[0].val, n=p.n)
    bad_end.row_ptr[p.n] -= 1
    bad_col = clair.CSR(A[0].row_ptr, A[0].col_idx.clone(), A[0].val, n=p.n)
    bad_col.col_idx[5] = p.n
    for M in (bad_end, bad_col):
        with pytest.raises(clair.ClairError) as e:
            clair.clair_transpose(M, p.n)
        assert e.value.status == 1
        with pytest.raises(clair.ClairError) as e:
            clair.clair_build_P(M, cf[0], B[0], 1)
        assert e.value.status == 1
        with pytest.raises(clair.ClairError) as e:
            clair.clair_smooth_B(M, cf[0], B[0], 1, 0.6, transpose=True)
        assert e.value.status == 1
    clair.clair_transpose(A[0], p.n)  # and the library goes on


@pytest.mark.parametrize("top,status", [(64, 0), (65, 5), (128, 5)])
def test_rows_beyond_the_lds_need_a_scratch(top, status):
    """Without an FP64 scratch (the fixed-memory entry point; an asynchronous
    call before any synchronous one) rows above 64 points are reported."""
    import ctypes

    from paper_2307_00229_amd import clair

    lib = clair.load_library()
    p = _groups([5, top, 33, 8], 61, 6)
    o = oracle.build_R_problem(p)
    (A,), (cf,), (B,), _ = to_device([p])
    first = int(np.nonzero(p.cf)[0][1])
    out, info, Ac = clair.ROut(o["n_c"], o["nnz"]), clair.Info(), A.c()
    Rc = out.c()
    st = lib.clair_build_R_noalloc(ctypes.byref(Ac), cf.data_ptr(), B.data_ptr(), 1, ctypes.byref(Rc), None,
                                   ctypes.byref(info))
    assert st == status and info.status == status
    assert info.first_bad_row == (first if status else -1)
    ctx = clair.Context()
    outs, _, _ = clair.clair_build_R_batched([A], [cf], [B], [1], ctx=ctx, outs=[clair.ROut(o["n_c"], o["nnz"])],
                                             async_=True)
    st, infos = ctx.info(1, outs)
    assert infos[0]["status"] == status and infos[0]["first_bad_row"] == (first if status else -1)
    _check([p], ctx=ctx)  # a synchronous call sizes the scratch


@pytest.mark.parametrize("deg", [2, 4, 5, 7, 8, 9])
@pytest.mark.parametrize("group", [4, 16, 32])
def test_width_8_adjacency_rows(group, deg):
    """Rows at distance 2 over a width-8 adjacency: points of up to four edges,
    of five to eight and beyond, neighbourhoods up to and above 32 points."""
    from paper_2307_00229_amd import clair

    ctx = clair.Context()
    ctx.set_tuning(group=group)
    ctx.set_search_adjacency(8)
    _check([_groups([0, 1, 3, 4, 5, 6, 7, 8, 2] * 29, 71 + deg, deg, ell=2), _groups([8, 4] * 3, 5, 2, ell=2),
            P.random_sparse(200, 0.02, deg, ell=2)], ctx=ctx)
