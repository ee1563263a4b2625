"""The backward on graphs of long rows in a band, where dY_i W_i^T is taken before the gather over A^T and only the recorded columns are
gathered (windows of rows staged in LDS), against the oracle: every group width, one to four values per lane, rows that end inside a
window and rows that fill several passes of one, rows without a neighbour, a last workgroup that is not full."""
import numpy as np
import pytest

import oracle
import paper_2603_27156_amd as gsr
from paper_2603_27156_amd import synth
from gpu_util import BF16_REL, NORM, Case, assert_close, rel_norm
from test_gpu_layer import run_step

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def band_graph(n, half, keep, seed):
    """Row i may reach i - half .. i + half, each neighbour with probability `keep`; some rows reach nobody."""
    rng = np.random.default_rng(seed)
    lists = []
    for i in range(n):
        js = np.arange(max(0, i - half), i)
        js = js[rng.random(len(js)) < keep]
        lists.append(js if i % 97 != 5 else js[:0])
    rowptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)
    return rowptr, np.concatenate(lists).astype(np.int32)


@pytest.mark.parametrize("workgroups", [0, 8])          # a handful of rows per workgroup, or some two hundred (several per group of lanes)
@pytest.mark.parametrize("n,half,keep,c,dg,k,norm,dtype,layout", [
    (1201, 60, 1.0, 4, 32, 8, "rms", "f32", gsr.GSR_LAYOUT_ROW_MAJOR),       # windows of 576 rows: every row ends inside one
    (1537, 50, 1.0, 2, 32, 16, "none", "f32", gsr.GSR_LAYOUT_GROUP_PLANAR),
    (1300, 70, 0.9, 3, 64, 16, "rms", "f32", gsr.GSR_LAYOUT_ROW_MAJOR),
    (1300, 70, 0.9, 2, 64, 31, "rms", "f32", gsr.GSR_LAYOUT_GROUP_PLANAR),   # two values per lane, the last lane without its second
    (1205, 80, 1.0, 2, 128, 33, "rms", "f32", gsr.GSR_LAYOUT_ROW_MAJOR),     # four values per lane
    (1900, 300, 0.5, 2, 192, 16, "rms", "f32", gsr.GSR_LAYOUT_ROW_MAJOR),    # windows of 96 rows, some 50 entries of a row in each
    (1210, 60, 1.0, 2, 192, 64, "none", "f32", gsr.GSR_LAYOUT_GROUP_PLANAR),
    (1200, 60, 1.0, 2, 256, 17, "rms", "f32", gsr.GSR_LAYOUT_ROW_MAJOR),
    (1300, 70, 0.9, 2, 64, 16, "rms", "bf16", gsr.GSR_LAYOUT_ROW_MAJOR),
    (1205, 80, 1.0, 2, 128, 16, "rms", "bf16", gsr.GSR_LAYOUT_GROUP_PLANAR),
])
def test_band_backward(n, half, keep, c, dg, k, norm, dtype, layout, workgroups):
    rowptr, colidx = band_graph(n, half, keep, dg + k)
    og = oracle.graph_build(rowptr, colidx)
    gsr.gsr_set_option("max_workgroups", workgroups)
    try:
        gg = gsr.gsr_graph_create(rowptr, colidx)
    finally:
        gsr.gsr_set_option("max_workgroups", 0)
    assert gsr.gsr_graph_info(gg)["nnz"] >= 64 * n           # long rows
    f32 = dtype == "f32"
    d, tdt = c * dg, torch.float32 if f32 else torch.bfloat16
    ocfg = oracle.Cfg(d, c, k, NORM[norm][0], 1e-5, oracle.STORE_F32 if f32 else oracle.STORE_BF16)
    cfg = gsr.Config(n=n, d=d, c=c, k=k, l=1, dtype=gsr.GSR_F32 if f32 else gsr.GSR_BF16, norm=NORM[norm][1], eps=1e-5, layout=layout)
    rng = np.random.default_rng(3)
    W = ((rng.random((c, dg, dg)) * 2 - 1) * np.sqrt(3.0 / dg)).astype(np.float32)
    plane = lambda scale: torch.from_numpy((rng.standard_normal((n, d)) * scale).astype(np.float32)).to(tdt)
    Y, dY = plane(1.0), plane(1e-3)

    def to_dev(x):
        return (x if layout == gsr.GSR_LAYOUT_ROW_MAJOR else x.view(n, c, dg).permute(1, 0, 2).contiguous()).to("cuda")

    def to_host(x):
        x = x.cpu().double()
        return (x if layout == gsr.GSR_LAYOUT_ROW_MAJOR else x.permute(1, 0, 2).reshape(n, d)).numpy()

    X_ref, dX_ref, dW_ref = oracle.layer_backward(og, ocfg, W, Y.double().numpy(), dY.double().numpy())
    outs = []
    for _ in range(2):
        y, dy, dW = to_dev(Y), to_dev(dY), torch.empty((c, dg, dg), dtype=torch.float32, device="cuda")
        gsr.gsr_layer_backward(gg, cfg, torch.from_numpy(W).to("cuda"), y, dy, dW)
        outs.append((y, dy, dW))
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    y, dy, dW = outs[0]
    if f32:
        assert_close("X", to_host(y), X_ref)
        assert_close("dX", to_host(dy), dX_ref)
        assert_close("dW", dW.cpu().numpy(), dW_ref)
    else:
        for name, got, ref in (("X", to_host(y), X_ref), ("dX", to_host(dy), dX_ref), ("dW", dW.cpu().numpy(), dW_ref)):
            assert rel_norm(got, ref) <= BF16_REL, name


@pytest.mark.parametrize("c,dg,k,workgroups", [(2, 64, 16, 8), (2, 192, 20, 8), (3, 32, 8, 0)])
def test_band_backward_on_a_directed_weighted_graph(c, dg, k, workgroups):
    """Row i reaches i .. i + 99 (cut at the end) with values of its own: the band and its entries are those of A^T."""
    n = 1300
    lists = [np.arange(i, min(n, i + 100)) for i in range(n)]
    rp = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    ci = np.concatenate(lists).astype(np.int32)
    rng = np.random.default_rng(8)
    av = rng.uniform(0.01, 0.03, len(ci)).astype(np.float32)
    gsr.gsr_set_option("max_workgroups", workgroups)
    try:
        gg = gsr.gsr_graph_create(rp, ci, vals=av, flags=0)
    finally:
        gsr.gsr_set_option("max_workgroups", 0)
    og = oracle.graph_from_csr(rp, ci, av)
    d = c * dg
    ocfg = oracle.Cfg(d, c, k, oracle.NORM_RMS, 1e-5, oracle.STORE_F32)
    cfg = gsr.Config(n=n, d=d, c=c, k=k, l=1, norm=gsr.GSR_NORM_RMS, eps=1e-5)
    W = ((rng.random((c, dg, dg)) * 2 - 1) * np.sqrt(3.0 / dg)).astype(np.float32)
    Y = rng.standard_normal((n, d)).astype(np.float32)
    dY = (rng.standard_normal((n, d)) * 1e-3).astype(np.float32)
    X_ref, dX_ref, dW_ref = oracle.layer_backward(og, ocfg, W, Y.astype(np.float64), dY.astype(np.float64))
    y, dy, dW = torch.from_numpy(Y).cuda(), torch.from_numpy(dY).cuda(), torch.empty((c, dg, dg), dtype=torch.float32, device="cuda")
    gsr.gsr_layer_backward(gg, cfg, torch.from_numpy(W).cuda(), y, dy, dW)
    assert_close("X", y.cpu().numpy(), X_ref)
    assert_close("dX", dy.cpu().numpy(), dX_ref)
    assert_close("dW", dW.cpu().numpy(), dW_ref)


def graph_of(rowptr, colidx, workgroups=0):
    gsr.gsr_set_option("max_workgroups", workgroups)
    try:
        return gsr.gsr_graph_create(rowptr, colidx)
    finally:
        gsr.gsr_set_option("max_workgroups", 0)


def with_rows(rowptr, colidx, more):
    """The graph with further entries: {row: columns}."""
    n = len(rowptr) - 1
    key = np.repeat(np.arange(n, dtype=np.int64), np.diff(rowptr)) * n + colidx
    key = np.unique(np.concatenate([key] + [np.full(len(c), r, dtype=np.int64) * n + c for r, c in more.items()]))
    return np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int32), (key % n).astype(np.int32)


def layer_bytes(g, n):
    """Of a configuration that gathers recorded columns wherever the graph lets it: two float32 planes more where it does."""
    return gsr.gsr_workspace_size(g, gsr.Config(n=n, d=128, c=2, k=16, l=1))[0]


def takes_band(rowptr, colidx, workgroups=0):
    n = len(rowptr) - 1
    hub = with_rows(rowptr, colidx, {r: np.arange(r + 1, n) for r in (0, 64, 128)})      # nodes next to every other: whole rows are gathered
    more = layer_bytes(graph_of(rowptr, colidx, workgroups), n) - layer_bytes(graph_of(*hub, workgroups), n)
    plane = n * 64 * 4
    assert abs(more) < plane // 4 or abs(more - 2 * plane) < plane // 4          # (beside them a few rows of chunk sums)
    return more > plane


@pytest.mark.parametrize("workgroups", [0, 8])
@pytest.mark.parametrize("n,half,keep,seed", [(1201, 60, 1.0, 40), (1537, 50, 1.0, 48), (1300, 70, 0.9, 80), (1205, 80, 1.0, 161), (1900, 300, 0.5, 208),
                                              (1210, 60, 1.0, 256), (1200, 60, 1.0, 273)])
def test_the_graphs_above_are_gathered_by_recorded_columns(n, half, keep, seed, workgroups):
    assert takes_band(*band_graph(n, half, keep, seed), workgroups)


def test_graphs_with_a_workgroup_or_a_row_far_above_the_mean_are_gathered_by_whole_rows():
    """The gather ends with its largest workgroup: a net over the whole graph makes one stage every row, and a row several times as long as the
    others is added up by sixteen lanes."""
    n, half = 3000, 300
    rowptr, colidx = band_graph(n, half, 0.22, 7)
    rng = np.random.default_rng(2)
    near = lambda c, count: {c: np.setdiff1d(c - half + rng.permutation(2 * half)[:count], [c])}
    assert takes_band(rowptr, colidx)
    assert takes_band(*with_rows(rowptr, colidx, near(1500, 200)))          # (a row of some 300 entries, the mean has 130)
    assert not takes_band(*with_rows(rowptr, colidx, near(1500, 600)))      # .. of 600
    assert not takes_band(*with_rows(rowptr, colidx, {20: np.arange(100, n, 200)}))
    far = with_rows(rowptr, colidx, {20: np.arange(100, n, 200), **near(1500, 600)})
    og, g = oracle.graph_build(*far), graph_of(*far)
    c, dg, k = 2, 64, 16
    W = ((rng.random((c, dg, dg)) * 2 - 1) * np.sqrt(3.0 / dg)).astype(np.float32)
    Y, dY = rng.standard_normal((n, c * dg)).astype(np.float32), (rng.standard_normal((n, c * dg)) * 1e-3).astype(np.float32)
    refs = oracle.layer_backward(og, oracle.Cfg(c * dg, c, k, oracle.NORM_RMS, 1e-5, oracle.STORE_F32), W, Y.astype(np.float64), dY.astype(np.float64))
    y, dy, dW = torch.from_numpy(Y).cuda(), torch.from_numpy(dY).cuda(), torch.empty((c, dg, dg), dtype=torch.float32, device="cuda")
    gsr.gsr_layer_backward(g, gsr.Config(n=n, d=c * dg, c=c, k=k, l=1, norm=gsr.GSR_NORM_RMS, eps=1e-5), torch.from_numpy(W).cuda(), y, dy, dW)
    for name, got, ref in zip(("X", "dX", "dW"), (y, dy, dW), refs):
        assert_close(name, got.cpu().numpy(), ref)


def band_case(n, half, keep, c, dg, k, l=3):
    """A stack of layers on a band graph: inputs as drawn for the other stacks, the graph in their place."""
    w = synth.scaled(synth.workload(2), n, l=l, d=c * dg, c=c, k=k)
    cs = Case(w, 0, gsr.GSR_LAYOUT_ROW_MAJOR)
    rowptr, colidx = band_graph(n, half, keep, dg + k)
    assert takes_band(rowptr, colidx)
    cs.og, cs.gg = oracle.graph_build(rowptr, colidx), graph_of(rowptr, colidx)
    return cs


STACKS = [(1300, 70, 0.9, 2, 64, 16), (1300, 70, 0.9, 3, 64, 16), (1201, 60, 1.0, 2, 32, 8), (1201, 60, 1.0, 4, 32, 8), (1900, 300, 0.5, 2, 192, 16),
          (1210, 60, 1.0, 3, 128, 20)]


@pytest.mark.parametrize("n,half,keep,c,dg,k,save", [(*s, save) for s in STACKS for save in (0, 1, 2) if save < 2 or s[4] <= 64])      # (near-tie lists: to 64 columns)
def test_step_on_a_band_graph_against_oracle(n, half, keep, c, dg, k, save):
    """The records of the layer below go into the slots beside those the band gather reads; kept sets come with rebuilt values; the lowest layer
    leaves no record."""
    cs, tol = band_case(n, half, keep, c, dg, k), 2.0 ** -6
    w = cs.w
    keys = ("yhat", "XL", "X0rec", "dW", "dwout", "dX0")
    ref = oracle.step(cs.og, cs.ocfg, w.l, cs.x0_on_grid(), cs.inp.weights, cs.inp.w_out, cs.inp.b_out, cs.inp.target, variant={0: 0, 1: 2, 2: 3}[save],
                      tie_tol=tol, want=keys)
    more = dict(tie_tol=tol, tie_capacity=16 * 320) if save == 2 else {}
    out = run_step(cs, save_indices=save, **more)
    assert np.isclose(out["loss"], ref["loss"], rtol=1e-4)
    for key in keys:
        assert_close(key, out[key], ref[key])


@pytest.mark.parametrize("n,half,keep,c,dg,k", [s for s in STACKS if s[4] <= 64])
def test_step_on_a_band_graph_with_every_row_listed(n, half, keep, c, dg, k):
    """Listed rows restored with the record (up to 320 places per sub-list) and in a launch after it equal the step that keeps all indices."""
    cs = band_case(n, half, keep, c, dg, k)
    saved = run_step(cs, raw=True, save_indices=1)
    for capacity in (16 * 320, 16 * 321):
        listed = run_step(cs, raw=True, save_indices=2, tie_tol=1e30, tie_capacity=capacity)
        for key in saved:
            assert torch.equal(listed[key], saved[key]), (capacity, key)


@pytest.mark.parametrize("save,c,dg,k", [(0, 2, 192, 16), (1, 3, 64, 16), (2, 2, 64, 16)])
def test_step_on_a_band_graph_replays_from_a_graph(save, c, dg, k):
    """Every replay, with eager work and synchronisations between them, gives the eager step's bits."""
    cs = band_case(1900 if dg == 192 else 1300, 300 if dg == 192 else 70, 0.5 if dg == 192 else 0.9, c, dg, k)
    want = run_step(cs, raw=True, save_indices=save)
    w, dv = cs.w, cs.dev
    cfg = gsr.Config(**{**cs.gcfg.__dict__, "save_indices": save})
    one = dict(dtype=torch.float32, device=dv)
    x0, W = cs.to_dev(cs.inp.x0), torch.from_numpy(np.ascontiguousarray(cs.inp.weights[:w.l])).to(dv)
    w_out, target, b_out = torch.from_numpy(cs.inp.w_out).to(dv), torch.from_numpy(cs.inp.target).to(dv), torch.tensor([cs.inp.b_out], **one)
    out = dict(loss=torch.zeros(1, **one), dW=torch.empty_like(W), dwout=torch.empty(w.d, **one), dbout=torch.zeros(1, **one),
               yhat=torch.empty(w.n, **one), dX0=torch.empty_like(x0), X0rec=torch.empty_like(x0))
    ws = torch.empty(gsr.gsr_workspace_size(cs.gg, cfg)[1], dtype=torch.uint8, device=dv)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            gsr.gsr_step(cs.gg, cfg, x0, W, w_out, b_out, target, out["loss"], out["dW"], out["dwout"], out["dbout"], yhat_out=out["yhat"],
                         dx0_out=out["dX0"], x0_rebuilt_out=out["X0rec"], workspace=ws)
    for rep in range(3):
        for v in out.values():
            v.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for key, v in out.items():
            assert torch.equal(v, want[key]), (rep, key)
        again = run_step(cs, raw=True, save_indices=save)          # eager work between the replays
        for key in want:
            assert torch.equal(again[key], want[key]), (rep, key)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dg,k", [(32, 8), (64, 16)])
def test_an_infinity_in_the_gradient_stays_one(dg, k, dtype):
    """dY_2 with one infinite entry: dZ of its neighbours is infinite, with the sign of the weight, at the recorded columns, and a number
    everywhere else, as in ordinary arithmetic."""
    n, half, c = 1300, 70, 2
    rowptr, colidx = band_graph(n, half, 0.9, dg + k)
    assert takes_band(rowptr, colidx)
    og, g = oracle.graph_build(rowptr, colidx), graph_of(rowptr, colidx)
    f32 = dtype == "f32"
    tdt = torch.float32 if f32 else torch.bfloat16
    rng = np.random.default_rng(11)
    W = ((rng.random((c, dg, dg)) * 2 - 1) * np.sqrt(3.0 / dg)).astype(np.float32)
    W[:, ::2] = np.round(W[:, ::2] * 8) / 8          # (exact in one 16-bit term, the others zero ..
    W[W == 0] = 0.125                                # .. but no weight is zero)
    Y = torch.from_numpy(rng.standard_normal((n, c * dg)).astype(np.float32)).to(tdt)
    dY = torch.from_numpy((rng.standard_normal((n, c * dg)) * 1e-3).astype(np.float32)).to(tdt)
    dY[601, dg + 5] = float("inf")
    dY[602, dg + 5] = float("inf")
    ref = oracle.layer_backward(og, oracle.Cfg(c * dg, c, k, oracle.NORM_NONE, 1e-5, oracle.STORE_F32 if f32 else oracle.STORE_BF16), W,
                                Y.double().numpy(), dY.double().numpy())[1][:, :dg]
    dy, dW = dY.cuda(), torch.empty((c, dg, dg), dtype=torch.float32, device="cuda")
    cfg = gsr.Config(n=n, d=c * dg, c=c, k=k, l=1, dtype=gsr.GSR_F32 if f32 else gsr.GSR_BF16, norm=gsr.GSR_NORM_NONE)
    gsr.gsr_layer_backward(g, cfg, torch.from_numpy(W).cuda(), Y.cuda(), dy, dW)
    got = dy.cpu().double().numpy()[:, :dg]          # group 1 has been added to by block 2 alone
    assert np.isinf(ref).sum() > 1000 and not np.isnan(ref).any()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    rest = ~np.isinf(ref)
    if f32:
        assert_close("dX", got[rest], ref[rest])
    else:
        assert rel_norm(got[rest], ref[rest]) <= BF16_REL
