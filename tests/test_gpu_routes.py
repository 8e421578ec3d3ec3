"""GPU calls whose kernels are chosen from what earlier calls read back.

Blocks larger than the context has seen, rows and outputs at the choice's
edges.  Against the oracle with the gates of tests/_util.py (the generated
systems are the strictly dominant ones of tests/test_gpu_solvers.py).
"""
import numpy as np
import pytest

import oracle
from paper_2307_00229_amd import problems as P

from ._util import assert_matches_oracle, to_device
from .test_gpu_solvers import _groups, _need_gpu  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _host(out):
    rp, ci, va = (x.cpu().numpy() for x in out.trimmed())
    return dict(row_ptr=rp, col_idx=ci, val=va, n_c=out.n_c, nnz=out.nnz)


@pytest.mark.parametrize("group", [4, 8, 16, 32])
@pytest.mark.parametrize("seen,then", [(5, 9), (9, 13), (9, 16), (12, 16), (20, 20), (26, 29), (28, 32)])
def test_larger_blocks_in_an_asynchronous_call(group, seen, then):
    """An asynchronous call whose blocks outgrow the last synchronous call's,
    within the bin's bounds of 16, 20, 24 and 32 points (bin A: the group), is
    solved by the same solvers: no row falls to the one-workgroup FP64 solver."""
    from paper_2307_00229_amd import clair

    ctx = clair.Context()
    ctx.set_tuning(group=group)
    small, big = _groups([seen, 3, 8] * 5, 1, 5), _groups([then, then - 1, 3, 9, 8] * 11, 2, 6)
    for p in (small, big, small):  # (the larger blocks are never read back before their call)
        As, cfs, Bs, ells = to_device([p])
        o = oracle.build_R_problem(p)
        outs = [clair.ROut(o["n_c"], o["nnz"])]
        if p is small:
            clair.clair_build_R_batched(As, cfs, Bs, ells, ctx=ctx, outs=outs)
            continue
        for _ in range(2):
            clair.clair_build_R_batched(As, cfs, Bs, ells, ctx=ctx, outs=outs, async_=True)
            st, infos = ctx.info(1, outs)
            assert st == 0 and infos[0]["n_fp64_rows"] == 0
            assert_matches_oracle(p, _host(outs[0]), o, infos[0])


def _row_bounds(p, g):
    """(error, bound) of every non-empty row of an unconstrained g: the distance
    to the row's solution in extended precision, and the forward error that one
    FP64 residual's rounding allows, (s + 2) 2^-53 |K^-1| (|K| |z| + |f|)."""
    import scipy.sparse as sp

    M = sp.csr_matrix((p.val, p.col_idx, p.row_ptr), shape=(p.n, p.n))
    C = np.nonzero(p.cf)[0]
    err, bound = [], []
    for r in range(g["n_c"]):
        cols, z = (g[k][g["row_ptr"][r]:g["row_ptr"][r + 1]] for k in ("col_idx", "val"))
        N, z = cols[cols != C[r]], z[cols != C[r]]
        if not N.size:
            continue
        K, f = M[N][:, N].toarray().T, -M[C[r]][:, N].toarray().ravel()
        inv = np.linalg.inv(K)
        x = (inv @ f).astype(np.longdouble)
        for _ in range(4):
            x = x + inv @ (f - K.astype(np.longdouble) @ x).astype(np.float64)
        x64 = np.abs(x.astype(np.float64))
        err.append(float(np.abs(z - x).max()))
        bound.append((N.size + 2) * 2.0**-53 * (np.abs(inv) @ (np.abs(K) @ x64 + np.abs(f))).max())
    return np.array(err), np.array(bound)


@pytest.mark.parametrize("case", ["diffusive", "4", "8"])
def test_rows_of_the_default_group_to_a_residual_rounding(case):
    """Rows of up to 8 points with a bin-A bound of 8 (the default): off by no more
    than the rounding of one FP64 residual, whatever the residual that passed the
    stopping test was."""
    from paper_2307_00229_amd import clair

    p = P.small_2d(61, stencil=5, eps=1.0, ell=2) if case == "diffusive" else _groups([int(case)] * 200, 9, 4)
    p.B = None
    As, cfs, _, ells = to_device([p])
    outs, infos, st = clair.clair_build_R_batched(As, cfs, None, ells, ctx=clair.Context())
    assert st == 0 and infos[0]["n_fp64_rows"] == 0 and infos[0]["max_block"] <= 8
    err, bound = _row_bounds(p, _host(outs[0]))
    assert np.all(err <= bound), float((err / bound).max())


@pytest.mark.parametrize("extra", [0, 3, 40, 70, 150])
@pytest.mark.parametrize("top", [12, 16, 20, 24, 28, 32])
def test_tile_rows_of_long_rows(top, extra):
    """Blocks of the 4 x 4-grid solver whose rows of A hold up to `extra` entries
    outside the block, on both sides of it: below and above the nine of the first
    reads and the 64 that a marking word covers."""
    import scipy.sparse as sp

    from paper_2307_00229_amd import clair

    p = _groups([top, top - 2, 9, top] * 45, 31 + top, 31)
    rng = np.random.default_rng(extra)
    M = sp.csr_matrix((p.val, p.col_idx, p.row_ptr), shape=(p.n, p.n))
    F, C = np.nonzero(p.cf == 0)[0], np.nonzero(p.cf)[0]
    cols = np.concatenate([rng.choice(C, extra, replace=False) for _ in F]) if extra else np.zeros(0, int)
    X = sp.coo_matrix((-rng.uniform(0.01, 0.1, cols.size), (np.repeat(F, extra), cols)), shape=M.shape).tocsr()
    M = (M + X + sp.diags(np.asarray(abs(X).sum(axis=1)).ravel())).tocsr()
    M.sort_indices()
    p = P.Problem(f"long_{top}_{extra}", p.n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data, p.cf,
                  p.B, 1)
    As, cfs, Bs, ells = to_device([p])
    outs, infos, st = clair.clair_build_R_batched(As, cfs, Bs, ells, ctx=clair.Context())
    assert st == 0 and infos[0]["max_block"] == top
    assert_matches_oracle(p, _host(outs[0]), oracle.build_R_problem(p), infos[0])


@pytest.mark.parametrize("blocks,left", [(8191, 1), (8192, 0), (8192, 1), (8200, 1023)])
def test_scans_of_many_blocks(blocks, left):
    """Column pointers over as many blocks of 1,024 columns as one kernel sums
    for itself, and over more (the blocks' totals are then scanned in turn)."""
    from paper_2307_00229_amd import clair

    ncol, m, w = 1024 * blocks + left, 200, 5000
    rng = np.random.default_rng(blocks + left)
    cols = np.sort(rng.integers(0, ncol // w, (m, w)) + np.arange(w) * (ncol // w), axis=1).astype(np.int32)
    cols[-1, -1] = ncol - 1
    A = clair.CSR(torch.arange(0, m * w + 1, w, dtype=torch.int32).cuda(), torch.from_numpy(cols.ravel()).cuda(),
                  torch.from_numpy(rng.uniform(1, 2, m * w)).cuda())
    rp, ci, va = (x.cpu().numpy() for x in clair.clair_transpose(A, ncol))
    order = np.argsort(cols.ravel(), kind="stable")
    assert np.array_equal(rp, np.concatenate([[0], np.cumsum(np.bincount(cols.ravel(), minlength=ncol))]))
    assert np.array_equal(ci, (order // w).astype(np.int32)) and np.array_equal(va, A.val.cpu().numpy()[order])


@pytest.mark.parametrize("fault", ["start", "end", "column", "below", "no columns"])
def test_refused_transposes_leave_their_outputs(fault):
    """Row pointers that do not run from 0 to nnz, and a column out of range:
    refused, and no output array of the call is written."""
    import ctypes

    from paper_2307_00229_amd import clair

    lib = clair.load_library()
    p = P.small_2d(40, stencil=5, ell=1)
    (A,), (cf,), (B,), _ = to_device([p])
    M = clair.CSR(A.row_ptr.clone(), A.col_idx.clone(), A.val, n=p.n)
    if fault == "start":
        M.row_ptr[0] = 1
    elif fault == "end":
        M.row_ptr[p.n] -= 1
    elif fault != "no columns":
        M.col_idx[p.nnz // 2] = p.n if fault == "column" else -1
    ncol = 0 if fault == "no columns" else p.n
    ctx, mc = clair.Context(), M.c()

    def out():
        o = clair.ROut(p.n, 4 * p.nnz)
        for t in (o.row_ptr, o.col_idx, o.val):
            t.fill_(-7)
        return o, o.c()

    o, oc = out()
    assert lib.clair_transpose(ctx.handle, ctypes.byref(mc), ncol, ctypes.byref(oc), None) == 1
    q, qc = out()
    s = torch.full_like(B, -7)
    if fault != "no columns":
        opts, info = clair.Opts(), clair.Info()
        assert lib.clair_build_P(ctx.handle, ctypes.byref(mc), cf.data_ptr(), B.data_ptr(), 1, ctypes.byref(qc),
                                 ctypes.byref(opts), ctypes.byref(info)) == 1
        assert lib.clair_smooth_B(ctx.handle, ctypes.byref(mc), cf.data_ptr(), B.data_ptr(), s.data_ptr(), 2, 0.6, 1,
                                  None) == 1
    torch.cuda.synchronize()
    for t in (o.row_ptr, o.col_idx, o.val, q.row_ptr, q.col_idx, q.val, s):
        assert bool((t == -7).all())
    R = clair.clair_transpose(A, p.n, ctx=ctx)  # the context goes on
    assert torch.equal(clair.clair_transpose(clair.CSR(*R), p.n, ctx=ctx)[1], A.col_idx)


@pytest.mark.parametrize("chunk", [256, 768, 1280, 1792])
def test_small_batches_of_odd_chunks(chunk):
    """Tuned chunks that halve to 64, 96, 80 and 112 points: several start inside
    one 64-row block of the row lookup, some hold no C-point."""
    import scipy.sparse as sp

    from paper_2307_00229_amd import clair

    ps = []
    for n in (1, 79, 80, 81, 95, 97, 1000, 4099):
        rng = np.random.default_rng(n)
        M = sp.diags([-rng.uniform(0.2, 1, n), np.full(n, 2.5), -rng.uniform(0.2, 1, n)], [-1, 0, 1], shape=(n, n)).tocsr()
        cf = ((np.arange(n) % 3 == 1) & ((np.arange(n) // 100) % 2 == 0)) | (n == 1)
        ps.append(P.Problem(f"line_{n}", n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data,
                            cf.astype(np.int8), rng.uniform(0.5, 1.5, n), 2))
    ctx = clair.Context()
    ctx.set_tuning(chunk=chunk)
    As, cfs, Bs, ells = to_device(ps)
    for _ in range(2):
        outs, infos, st = clair.clair_build_R_batched(As, cfs, Bs, ells, ctx=ctx)
        assert st == 0
        for p, o, inf in zip(ps, outs, infos):
            assert_matches_oracle(p, _host(o), oracle.build_R_problem(p), inf)


@pytest.mark.parametrize("group", [8, 16, 32])
def test_graph_replays_with_larger_blocks(group):
    """A captured setup whose values, and with them the blocks, change between
    replays: 9 points when captured, then 16, on the same buffers."""
    from paper_2307_00229_amd import clair

    big = _groups([16, 14, 9, 3] * 9, 5, 6)
    rows = np.repeat(np.arange(big.n), np.diff(big.row_ptr))
    rank = np.arange(big.nnz) - big.row_ptr[rows]
    few = np.where((big.cf[rows] != 0) & (rows != big.col_idx) & (rank >= 10), 0.0, big.val)
    small = P.Problem("few", big.n, big.row_ptr, big.col_idx, few, big.cf, big.B, 1)
    want = {q.name: oracle.build_R_problem(q) for q in (small, big)}
    assert np.diff(want["few"]["row_ptr"]).max() <= 12 < np.diff(want[big.name]["row_ptr"]).max()
    As, cfs, Bs, ells = to_device([small])
    o = want[big.name]
    outs = [clair.ROut(o["n_c"], o["nnz"])]
    ctx = clair.Context()
    ctx.set_tuning(group=group)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = clair.Graph(ctx, As, cfs, Bs, ells, outs, stream=stream)
    for q in (small, big, big, small, big):
        As[0].val.copy_(torch.from_numpy(q.val).cuda())
        torch.cuda.synchronize()
        graph.launch(stream=stream)
        stream.synchronize()
        st, infos = graph.info()
        assert st == 0 and infos[0]["n_fp64_rows"] == 0
        assert_matches_oracle(q, _host(outs[0]), want[q.name], infos[0])
    graph.close()


@pytest.mark.parametrize("top", [9, 12, 13, 16, 17, 20, 21, 24, 25, 28, 29, 32])
@pytest.mark.parametrize("group", [4, 16, 32])
def test_tile_rows_of_a_repeated_call(group, top):
    """The same call three times with its buffers: sizes read back, then known."""
    from paper_2307_00229_amd import clair

    ctx = clair.Context()
    ctx.set_tuning(group=group)
    p = _groups([top, 0, 9, top - 1, 3, top, 10, 8, 1] * 5, 200 + top, 5)
    As, cfs, Bs, ells = to_device([p, p])
    o = oracle.build_R_problem(p)
    for _ in range(3):
        outs = [clair.ROut(o["n_c"], o["nnz"]) for _ in range(2)]
        outs, infos, st = clair.clair_build_R_batched(As, cfs, Bs, ells, ctx=ctx, outs=outs)
        assert st == 0
        for out, inf in zip(outs, infos):
            assert_matches_oracle(p, _host(out), o, inf)
