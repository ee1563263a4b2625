"""The gathers that give a lane to every kept value (records with the column of each value), at the sizes where their
rounds, runs and passes can go wrong; the first pass that writes a row of one chunk straight to where it belongs; rows cut
into longer partials on small graphs; tiles assigned without draws."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2603_27156_amd as gsr
from paper_2603_27156_amd import synth
from gpu_util import Case, assert_close, rel_norm, BF16_REL
from test_gpu_layer import run_step, ROW, PLANAR

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# lengths around the sixteen steps of a run, the 64 edges of a round and two rounds, several of them inside one 16-row tile
LENGTHS = [0, 1, 2, 15, 16, 17, 3, 63, 64, 65, 1, 0, 127, 128, 129, 5, 31, 33, 48, 49, 4, 4, 4, 4, 200, 1, 7, 8, 9, 12, 13, 0, 61, 3, 62, 2, 66]


@pytest.fixture
def options():
    changed = []

    def set_option(key, value):
        changed.append(key)
        gsr.gsr_set_option(key, value)
    yield set_option
    for key in changed:
        gsr.gsr_set_option(key, 0)


def graph_of(lengths, n, seed):
    """n rows of the given lengths (then of one entry), random distinct columns and values."""
    rng = np.random.default_rng(seed)
    lengths = list(lengths) + [1] * (n - len(lengths))
    cols = np.concatenate([np.sort(rng.choice(n, size=l, replace=False)) for l in lengths] or [np.zeros(0)]).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    vals = rng.standard_normal(len(cols)).astype(np.float32)
    return rowptr, cols, vals, gsr.gsr_graph_create(rowptr, cols, vals, flags=0)


def sums_and_bound(rowptr, cols, vals, x):
    """A x in float64 and the error a float32 sum of that many products may have: (terms + 3) roundings of 2^-24."""
    import scipy.sparse as sp
    a = sp.csr_matrix((vals.astype(np.float64), cols, rowptr), shape=(len(rowptr) - 1,) * 2)
    terms = np.diff(rowptr)[:, None] + 3
    return a @ x, terms * 2.0 ** -24 * (abs(a) @ abs(x)) + 1e-30


@pytest.mark.parametrize("dg,k,dtype,threshold,chunk", [
    (64, 16, "f32", 512, 0), (64, 1, "f32", 512, 0), (64, 15, "f32", 512, 0), (64, 17, "f32", 512, 0), (64, 64, "f32", 512, 0),
    (32, 8, "f32", 512, 0), (32, 32, "f32", 512, 0), (64, 16, "bf16", 512, 0), (64, 33, "bf16", 512, 0), (32, 5, "bf16", 512, 0),
    (64, 16, "f32", 16, 16), (64, 40, "f32", 3, 64), (32, 20, "bf16", 8, 32),
    # (laid out as rows first: k above 16 in 16-bit storage, above dg / 2 in float32)
    (64, 17, "bf16", 512, 0), (64, 64, "bf16", 6, 4), (64, 33, "f32", 512, 0), (32, 17, "f32", 16, 16), (32, 31, "bf16", 512, 0),
])
def test_value_gather_at_the_edges_of_runs_and_rounds(options, dg, k, dtype, threshold, chunk):
    options("hub_threshold", threshold)
    options("hub_chunk", chunk)
    n = 421
    rowptr, cols, vals, g = graph_of(LENGTHS, n, 3)
    rng = np.random.default_rng(5)
    idx = np.stack([rng.permutation(dg)[:k] for _ in range(n)]).astype(np.int32)       # any slot order
    v = torch.from_numpy(rng.standard_normal((n, k)).astype(np.float32)).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    h = gsr.gsr_spmm_compressed(g, v, torch.from_numpy(idx).cuda(), dg).cpu().numpy()
    dense = np.zeros((n, dg))
    np.put_along_axis(dense, idx.astype(np.int64), v.float().cpu().numpy().astype(np.float64), 1)
    ref, bound = sums_and_bound(rowptr, cols, vals, dense)
    assert (np.abs(h - ref) <= bound).all(), float((np.abs(h - ref) / bound).max())


@pytest.mark.parametrize("k,dtype", [(16, "f32"), (40, "f32"), (64, "f32"), (24, "bf16")])
@pytest.mark.parametrize("wrong", ["negative", "past", "repeated"])
def test_refused_indices_write_nothing_and_leave_the_graph_usable(wrong, k, dtype):
    n, dg = 421, 64
    rowptr, cols, vals, g = graph_of(LENGTHS, n, 4)
    idx = torch.arange(k, dtype=torch.int32).repeat(n, 1)
    good = idx.clone().cuda()
    idx[300, 3] = {"negative": -1, "past": dg, "repeated": 5}[wrong]
    idx = idx.cuda()
    v = torch.randn(n, k, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    h = torch.full((n, dg), 7.0, device="cuda")
    lib = gsr.lib()
    nbytes = lib.gsr_spmm_compressed_workspace(g.ptr, ctypes.c_int32(k), ctypes.c_int32(dg))
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")

    def call(i):
        return lib.gsr_spmm_compressed(g.ptr, ctypes.c_void_p(v.data_ptr()), ctypes.c_void_p(i.data_ptr()), ctypes.c_int32(k),
                                       ctypes.c_int32(dg), ctypes.c_int32(0 if dtype == "f32" else 1), ctypes.c_void_p(h.data_ptr()),
                                       ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(nbytes), gsr._stream())
    assert call(idx) == gsr.GSR_ERR_INVALID_ARG
    assert bool((h == 7.0).all())
    assert call(good) == gsr.GSR_OK
    dense = np.zeros((n, dg))
    dense[:, :k] = v.float().cpu().numpy()
    ref, bound = sums_and_bound(rowptr, cols, vals, dense)
    assert (np.abs(h.cpu().numpy() - ref) <= bound).all()


@pytest.mark.parametrize("n,d,c,k,threshold,chunk,layout", [
    (1003, 256, 2, 40, 8, 16, ROW),          # rows of one chunk, of several, and gathered ones in the same eight rows
    (777, 384, 2, 16, 1, 512, PLANAR),       # every row of two entries or more is one chunk
    (500, 512, 2, 70, 4, 4, ROW),            # nothing fits one chunk; five passes over the kept values
    (9, 384, 3, 3, 2, 8, PLANAR),            # a half and a bit of a 16-row tile
    (601, 256, 2, 16, 4, 2 ** 31, ROW),      # "never cut", beyond what 32 bits hold
    (601, 256, 2, 16, 4, 2 ** 32 + 3, ROW),
])
def test_wide_rows_of_one_chunk_and_of_several(options, n, d, c, k, threshold, chunk, layout):
    options("hub_threshold", threshold)
    options("hub_chunk", chunk)
    cs = Case(synth.scaled(synth.workload(2), n, l=1, d=d, c=c, k=k), 0, layout)
    W = cs.inp.weights[0]
    Wd = torch.from_numpy(W).to(cs.dev)
    X = cs.x0_on_grid()
    Y_ref = oracle.layer_forward(cs.og, cs.ocfg, W, X)
    y = cs.to_dev(X)
    gsr.gsr_layer_forward(cs.gg, cs.gcfg, Wd, y)
    assert_close("Y", cs.to_host(y), Y_ref)
    dY = (np.random.default_rng(17).standard_normal((n, d)) * 1e-3).astype(np.float32).astype(np.float64)
    Xb_ref, dX_ref, dW_ref = oracle.layer_backward(cs.og, cs.ocfg, W, Y_ref, dY)
    yb, dyb = cs.to_dev(Y_ref), cs.to_dev(dY)
    dW = torch.empty((c, d // c, d // c), dtype=torch.float32, device=cs.dev)
    gsr.gsr_layer_backward(cs.gg, cs.gcfg, Wd, yb, dyb, dW)
    assert_close("X rebuilt", cs.to_host(yb), Xb_ref)
    assert_close("dX", cs.to_host(dyb), dX_ref)
    assert_close("dW", dW.cpu().numpy(), dW_ref)


@pytest.mark.parametrize("dg", [32, 64, 128])
@pytest.mark.parametrize("threshold", [2 ** 31, 2 ** 32, 2 ** 32 + 3])
def test_rows_are_never_split_with_a_threshold_beyond_32_bits(options, dg, threshold):
    options("hub_threshold", threshold)
    n, c = 601, 2
    cs = Case(synth.scaled(synth.workload(2), n, l=1, d=c * dg, c=c, k=dg // 4), 0, ROW)
    assert gsr.gsr_graph_info(cs.gg)["n_hub_rows"] == 0
    X = cs.x0_on_grid()
    y = cs.to_dev(X)
    gsr.gsr_layer_forward(cs.gg, cs.gcfg, torch.from_numpy(cs.inp.weights[0]).to(cs.dev), y)
    assert_close("Y", cs.to_host(y), oracle.layer_forward(cs.og, cs.ocfg, cs.inp.weights[0], X))
    x = torch.randn(n, 64, device="cuda")
    assert_close("A x", gsr.gsr_spmm(cs.gg, x).cpu().numpy(), oracle.spmm(cs.og, x.cpu().numpy()))


@pytest.mark.parametrize("longest", [160, 161])
def test_short_rows_are_not_split_on_a_small_graph(longest):
    rowptr, cols, vals, g = graph_of([longest] + LENGTHS[:24], 500, 8)
    assert gsr.gsr_graph_info(g)["n_hub_rows"] == (0 if longest <= 160 else sum(l > 16 for l in [longest] + LENGTHS[:24]))
    x = torch.randn(500, 64, device="cuda")
    y = gsr.gsr_spmm(g, x).cpu().numpy()
    ref, bound = sums_and_bound(rowptr, cols, vals, x.cpu().numpy().astype(np.float64))
    assert (np.abs(y - ref) <= bound).all()


def test_short_rows_are_judged_for_the_transpose_on_its_own():
    """A directed graph: every row of A has 20 entries, a net of A^T (a column of A) has 160 or 161.  Rows of A are never cut;
    those of A^T are at 16 entries once the net is too long, which shows in the room for partial rows (two arrays)."""
    import scipy.sparse as sp
    n, size, longer = 500, {}, {}
    for sinks in (160, 161):
        rng = np.random.default_rng(9)
        rows = [np.sort(rng.choice(np.arange(1, n), size=20, replace=False)) for _ in range(n)]
        for r in range(sinks):
            rows[r] = np.concatenate([[0], rows[r][1:]])
        rowptr, cols = np.arange(n + 1, dtype=np.int32) * 20, np.concatenate(rows).astype(np.int32)
        vals = rng.standard_normal(len(cols)).astype(np.float32)
        g = gsr.gsr_graph_create(rowptr, cols, vals, flags=0)
        assert gsr.gsr_graph_info(g)["n_hub_rows"] == 0
        size[sinks] = gsr.gsr_workspace_size(g, gsr.Config(n=n, d=128, c=2, k=16))[0]
        longer[sinks] = int((np.bincount(cols, minlength=n) > 16).sum())
        x = torch.randn(n, 64, device="cuda")
        y = torch.empty_like(x)
        for transpose in (False, True):
            a = sp.csr_matrix((vals, cols, rowptr), shape=(n, n))
            a = (a.T if transpose else a).tocsr()
            ref, bound = sums_and_bound(a.indptr, a.indices, a.data, x.cpu().numpy().astype(np.float64))
            assert (np.abs(gsr.gsr_spmm(g, x, transpose=transpose).cpu().numpy() - ref) <= bound).all()
            gsr.gsr_spmm_noalloc(g, x, y, transpose=transpose)
            assert (np.abs(y.cpu().numpy() - ref) <= bound).all()
    assert longer[161] > 300 and size[161] - size[160] > 2 * (longer[161] - 8) * 64 * 4


def test_transpose_stays_uncut_where_the_fixed_scratch_would_not_hold_its_chunks():
    """A net of 200, rows of A^T above 16 entries, more than 16,384 of them: gsr_spmm_noalloc takes the graph."""
    n = 20_000
    rng = np.random.default_rng(10)
    cols = np.stack([rng.permutation(n) for _ in range(20)], 1).astype(np.int32)        # every column has 20 entries
    cols[:200, 0] = cols[0, 0]                                                          # and one of them 200 more
    rowptr, ci = np.arange(n + 1, dtype=np.int32) * 20, np.sort(cols, 1).reshape(-1)
    vals = rng.standard_normal(len(ci)).astype(np.float32)
    g = gsr.gsr_graph_create(rowptr, ci, vals, flags=0)
    x = torch.randn(n, 64, device="cuda")
    y = torch.empty_like(x)
    gsr.gsr_spmm_noalloc(g, x, y, transpose=True)
    assert torch.equal(y, gsr.gsr_spmm(g, x, transpose=True))


@pytest.mark.parametrize("sinks,width", [(1_024, 64), (1_025, 64), (5_000, 64), (5_000, 16), (2_500, 32)])
def test_nets_of_thousands_of_sinks_on_a_small_graph(sinks, width):
    n = 6_001
    lengths = [sinks] * 8 + [3] * 100            # eight nets side by side in one tile
    rowptr, cols, vals, g = graph_of(lengths, n, 6)
    x = torch.randn(n, width, device="cuda")
    y = gsr.gsr_spmm(g, x).cpu().numpy()
    ref, bound = sums_and_bound(rowptr, cols, vals, x.cpu().numpy().astype(np.float64))
    assert (np.abs(y - ref) <= bound).all(), float((np.abs(y - ref) / bound).max())


@pytest.mark.parametrize("c,dg,k,dtype,save", [(2, 64, 16, "f32", 2), (4, 32, 8, "f32", 1), (3, 64, 9, "f32", 0), (3, 64, 16, "bf16", 1),
                                               (4, 32, 8, "bf16", 1)])
def test_drawn_and_given_tiles_give_the_same_bits(options, c, dg, k, dtype, save):
    """With a grid of eight workgroups the same graph has many tiles per wave (tiles are drawn, a block's backward is cut in
    two kernels); with the default one every tile has a wave of its own."""
    options("hub_threshold", 64)       # (the defaults depend on the grid)
    options("hub_chunk", 64)
    w = synth.scaled(synth.workload(2), 3001, l=3, d=c * dg, c=c, k=k, dtype=dtype)
    one = run_step(Case(w, 0, PLANAR), raw=True, save_indices=save)
    options("max_workgroups", 8)
    two = run_step(Case(w, 0, PLANAR), raw=True, save_indices=save)
    for key in ("yhat", "XL", "X0rec", "dX0"):
        assert torch.equal(one[key], two[key]), key
    assert_close("dW", two["dW"].float().cpu().numpy(), one["dW"].double().cpu().numpy())


@pytest.mark.parametrize("dg,c,chunk", [(64, 2, 4), (64, 3, 100), (32, 4, 4), (32, 2, 100)])
def test_first_pass_where_every_column_is_kept(options, dg, c, chunk):
    """k = D/C: the first pass takes the records as the rows they are (rows cut at 6 entries, chunks shorter and longer than a
    round of 64 edges)."""
    options("hub_threshold", 6)
    options("hub_chunk", chunk)
    cs = Case(synth.scaled(synth.workload(2), 700, levels=6, d=dg * c, c=c, k=dg, l=2, hubs=2), 11, PLANAR)
    assert gsr.gsr_graph_info(cs.gg)["n_hub_rows"] > 0
    ref = oracle.step(cs.og, cs.ocfg, cs.w.l, cs.x0_on_grid(), cs.inp.weights, cs.inp.w_out, cs.inp.b_out, cs.inp.target)
    out = run_step(cs)
    assert np.isclose(out["loss"], ref["loss"], rtol=1e-4)
    for key in ("yhat", "XL", "X0rec", "dW", "dwout", "dX0"):
        assert_close(key, out[key], ref[key])


def graph_with_empty_tiles(kind, n, seed):
    """Rows of one to nine entries, none in the named places (tiles are sixteen rows)."""
    rng = np.random.default_rng(seed)
    lengths = rng.integers(1, 10, size=n)
    if kind == "front":
        lengths[:37] = 0
    elif kind == "middle and end":
        lengths[48:96] = 0
        lengths[n - 33:] = 0
    else:
        lengths[:] = 0
    cols = [np.sort(rng.choice(n, size=l, replace=False)) for l in lengths]
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    cols = np.concatenate([np.zeros(0)] + cols).astype(np.int32)
    return rowptr, cols, rng.standard_normal(len(cols)).astype(np.float32) * 0.3


@pytest.mark.parametrize("kind", ["front", "middle and end", "everywhere"])
@pytest.mark.parametrize("dg,dtype", [(32, "f32"), (64, "f32"), (128, "f32"), (32, "bf16"), (64, "bf16")])
def test_tiles_without_entries(kind, dg, dtype):
    """No neighbours, no self-loops: a gather with nothing to gather, also at the very front of the arrays."""
    n, c = 203, 3
    rowptr, cols, vals = graph_with_empty_tiles(kind, n, 7)
    cs = Case(synth.scaled(synth.workload(2), n, l=1, d=c * dg, c=c, k=dg // 4, dtype=dtype), 0, ROW)
    cs.og = oracle.graph_from_csr(rowptr, cols, vals)
    cs.gg = gsr.gsr_graph_create(rowptr, cols, vals=vals, flags=0)
    if dg <= 64:
        k = 9
        idx = np.stack([np.random.default_rng(r).permutation(dg)[:k] for r in range(n)]).astype(np.int32)
        v = torch.randn(n, k, device="cuda").to(cs.tdtype)
        h = gsr.gsr_spmm_compressed(cs.gg, v, torch.from_numpy(idx).cuda(), dg).cpu().numpy()
        dense = np.zeros((n, dg))
        np.put_along_axis(dense, idx.astype(np.int64), v.float().cpu().numpy().astype(np.float64), 1)
        ref, bound = sums_and_bound(rowptr, cols, vals, dense)
        assert (np.abs(h - ref) <= bound).all()
    X = cs.x0_on_grid()
    dY = synth.to_bf16_grid((np.random.default_rng(17).standard_normal((n, c * dg))).astype(np.float32)).astype(np.float64)
    W = cs.inp.weights[0]
    Wd = torch.from_numpy(W).to(cs.dev)
    Y_ref = oracle.layer_forward(cs.og, cs.ocfg, W, X)
    y = cs.to_dev(X)
    gsr.gsr_layer_forward(cs.gg, cs.gcfg, Wd, y)
    x = cs.to_dev(Y_ref)
    gsr.gsr_layer_inverse(cs.gg, cs.gcfg, Wd, x)
    ref = oracle.layer_backward(cs.og, cs.ocfg, W, Y_ref, dY)
    yb, dyb = cs.to_dev(Y_ref), cs.to_dev(dY)
    dW = torch.full((c, dg, dg), 7.0, dtype=torch.float32, device=cs.dev)
    gsr.gsr_layer_backward(cs.gg, cs.gcfg, Wd, yb, dyb, dW)
    got = (cs.to_host(y), cs.to_host(x), cs.to_host(yb), cs.to_host(dyb), dW.cpu().numpy())
    for name, a, b in zip(("Y", "X", "X rebuilt", "dX", "dW"), got, (Y_ref, oracle.layer_inverse(cs.og, cs.ocfg, W, Y_ref), *ref)):
        if dtype == "f32":
            assert_close(name, a, b)
        else:
            assert rel_norm(a, b) < BF16_REL, name
    if kind == "everywhere":         # f_i is zero: the planes pass through, no gradient reaches W
        assert np.array_equal(got[0], X) and np.array_equal(got[3], dY) and not got[4].any()


@pytest.mark.parametrize("dg,c,k,dtype,save,threshold,chunk", [
    (64, 2, 33, "f32", 2, 6, 4), (64, 3, 63, "f32", 1, 512, 0), (64, 4, 40, "f32", 0, 6, 100), (64, 2, 64, "f32", 2, 512, 0),
    (32, 2, 17, "f32", 0, 6, 4), (32, 4, 31, "f32", 2, 512, 0), (32, 2, 32, "f32", 1, 6, 100),
    (64, 2, 33, "bf16", 1, 6, 4), (64, 3, 64, "bf16", 1, 512, 0), (32, 4, 17, "bf16", 1, 512, 0), (32, 2, 31, "bf16", 2, 6, 100),
])
@pytest.mark.parametrize("workgroups", [0, 8])
def test_records_held_as_rows(options, dg, c, k, dtype, save, threshold, chunk, workgroups):
    """More than half of the columns kept: every form of the step, at the smallest such k, the largest and between."""
    options("hub_threshold", threshold)
    options("hub_chunk", chunk)
    options("max_workgroups", workgroups)         # (8: a block's backward is cut in two kernels, tiles are drawn)
    tol = 2.0 ** -4
    cs = Case(synth.scaled(synth.workload(2), 1501, levels=6, d=dg * c, c=c, k=k, l=2, hubs=2, dtype=dtype), 11, PLANAR)
    ref = oracle.step(cs.og, cs.ocfg, cs.w.l, cs.x0_on_grid(), cs.inp.weights, cs.inp.w_out, cs.inp.b_out, cs.inp.target,
                      variant={0: 0, 1: 2, 2: 3}[save], tie_tol=tol)
    out = run_step(cs, save_indices=save, tie_tol=tol, tie_capacity=16 * cs.w.n)
    assert np.isclose(out["loss"], ref["loss"], rtol=1e-4 if dtype == "f32" else BF16_REL)
    for key in ("yhat", "XL", "dW", "dwout", "dX0") + (("X0rec",) if dtype == "f32" else ()):
        if dtype == "f32":
            assert_close(key, out[key], ref[key])
        else:
            assert rel_norm(out[key], ref[key]) < BF16_REL, key
    x = cs.to_dev(cs.x0_on_grid())                # the layer calls, and what they rebuild
    W = torch.from_numpy(cs.inp.weights[0]).to(cs.dev)
    gsr.gsr_layer_forward(cs.gg, cs.gcfg, W, x)
    gsr.gsr_layer_inverse(cs.gg, cs.gcfg, W, x)
    if dtype == "f32":
        assert_close("inverse(forward(X)) vs X", cs.to_host(x), cs.x0_on_grid(), rtol=1e-4, atol=1e-4)
