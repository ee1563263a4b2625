"""Launch forms at their edges: a wave with several tiles of a two-block group, column packing by four (remainders, refused
indices), row widths of the head, layout copies of rows that do not start on sixteen bytes."""
import numpy as np
import pytest

import oracle
import paper_2603_27156_amd as gsr
from paper_2603_27156_amd import synth
from gpu_util import BF16_REL, Case, assert_close, bf16_bar, rel_norm
from test_gpu_layer import run_step, ROW, PLANAR
from test_gpu_wide import wide_case
from test_gpu_band import band_graph

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,c,k,layout", [(1029, 2, 16, ROW), (2051, 3, 32, PLANAR), (100, 2, 128, ROW)])
def test_two_block_groups_with_several_tiles_per_wave(n, c, k, layout):
    """Eight workgroups of eight waves: 64 waves for 65, 129 and 7 tiles (the last one ragged)."""
    gsr.gsr_set_option("max_workgroups", 8)
    try:
        cs = wide_case(n, 128 * c, c, k, 1, "rms", layout)
        w, W = cs.w, cs.inp.weights[0]
        Wd = torch.from_numpy(W).to(cs.dev)
        Y = oracle.layer_forward(cs.og, cs.ocfg, W, cs.x0_on_grid())
        y = cs.to_dev(cs.x0_on_grid())
        gsr.gsr_layer_forward(cs.gg, cs.gcfg, Wd, y)
        assert_close("Y", cs.to_host(y), Y)
        rng = np.random.default_rng(5)
        dY = (rng.standard_normal((w.n, w.d)) * 1e-3).astype(np.float32).astype(np.float64)
        X_ref, dX_ref, dW_ref = oracle.layer_backward(cs.og, cs.ocfg, W, Y, dY)
        yb, dyb = cs.to_dev(Y), cs.to_dev(dY)
        dW = torch.empty((w.c, w.dg, w.dg), dtype=torch.float32, device=cs.dev)
        gsr.gsr_layer_backward(cs.gg, cs.gcfg, Wd, yb, dyb, dW)
        assert_close("X", cs.to_host(yb), X_ref)
        assert_close("dX", cs.to_host(dyb), dX_ref)
        assert_close("dW", dW.cpu().numpy(), dW_ref)
    finally:
        gsr.gsr_set_option("max_workgroups", 0)


@pytest.mark.parametrize("dg,k", [(64, 4), (64, 12), (64, 32), (32, 16), (64, 13)])
def test_columns_packed_by_four(dg, k):
    """k / 4 lanes per row (1, 3 of 4, 8, 4), and k that is no multiple of four; any slot order; refused indices write nothing."""
    w = synth.scaled(synth.workload(2), 3003)
    rng = np.random.Generator(np.random.PCG64(k))
    rp, ci = synth.circuit_dag(w, rng)
    og, gg = oracle.graph_build(rp, ci), gsr.gsr_graph_create(rp, ci)
    V, I, _ = oracle.gs(rng.standard_normal((w.n, dg)).astype(np.float32).astype(np.float64), k)
    perm = np.argsort(rng.random((w.n, k)), axis=1)
    v = torch.from_numpy(np.take_along_axis(V, perm, axis=1).astype(np.float32)).cuda()
    i = torch.from_numpy(np.take_along_axis(I, perm, axis=1).astype(np.int32)).cuda()
    got = gsr.gsr_spmm_compressed(gg, v, i, dg)
    assert_close("A scatter(V, I)", got.cpu().numpy(), oracle.aggregate(og, V, I, dg))
    store = torch.empty(w.n * k + 1, dtype=torch.int32, device="cuda")          # an index array that starts off sixteen bytes
    store[1:] = i.reshape(-1)
    assert torch.equal(gsr.gsr_spmm_compressed(gg, v, store[1:].view(w.n, k), dg), got)
    for row, slot, value in ((0, 0, -1), (w.n - 1, k - 1, dg), (17, k - 1, 1 << 30), (5, 0, None), (w.n - 2, k - 1, None)):
        bad = i.clone()
        bad[row, slot] = bad[row, (slot + 1) % k] if value is None else value   # (None: a column named twice)
        with pytest.raises(gsr.GsrError):
            gsr.gsr_spmm_compressed(gg, v, bad, dg)


@pytest.mark.parametrize("c,dg,layout", [(3, 32, ROW), (2, 64, PLANAR), (3, 64, ROW), (5, 64, PLANAR)])
def test_head_widths_and_rows_off_sixteen_bytes(c, dg, layout):
    """D = 96, 128, 192 and 320: two, two, three and five column pieces of the head; the planes of the call on sixteen bytes and four off."""
    w = synth.scaled(synth.workload(2), 1003, l=2, d=c * dg, c=c, k=dg // 4)
    cs = Case(w, 1, layout)
    ref = oracle.step(cs.og, cs.ocfg, w.l, cs.x0_on_grid(), cs.inp.weights, cs.inp.w_out, cs.inp.b_out, cs.inp.target, variant=2)
    out = run_step(cs, raw=True, save_indices=1)
    host = run_step(cs, save_indices=1)
    assert np.isclose(host["loss"], ref["loss"], rtol=1e-4)
    for key in ("yhat", "XL", "X0rec", "dW", "dwout", "dX0"):
        assert_close(key, host[key], ref[key])
    f32 = dict(dtype=torch.float32, device=cs.dev)
    cfg = gsr.Config(**{**cs.gcfg.__dict__, "l": w.l, "save_indices": 1})
    x0 = cs.to_dev(cs.inp.x0)

    def off(like):
        return torch.empty(like.numel() + 1, **f32)[1:].view(like.shape)

    x, dx0, x0r, xl = off(x0), off(x0), off(x0), off(x0)
    x.copy_(x0)
    W = torch.from_numpy(np.ascontiguousarray(cs.inp.weights)).to(cs.dev)
    loss, db, dW, dwout, yhat = torch.zeros(1, **f32), torch.zeros(1, **f32), torch.empty_like(W), torch.empty(w.d, **f32), torch.empty(w.n, **f32)
    gsr.gsr_step(cs.gg, cfg, x, W, torch.from_numpy(cs.inp.w_out).to(cs.dev), torch.tensor([cs.inp.b_out], **f32),
                 torch.from_numpy(cs.inp.target).to(cs.dev), loss, dW, dwout, db, yhat_out=yhat, dx0_out=dx0, x0_rebuilt_out=x0r, xl_out=xl,
                 workspace=torch.empty(gsr.gsr_workspace_size(cs.gg, cfg)[1], dtype=torch.uint8, device=cs.dev))
    for key, got in (("loss", loss), ("yhat", yhat), ("dW", dW), ("dwout", dwout), ("dX0", dx0), ("X0rec", x0r), ("XL", xl)):
        assert torch.equal(got, out[key]), key


@pytest.mark.parametrize("dg,dtype", [(64, "f32"), (32, "f32"), (64, "bf16")])
def test_backward_where_every_tile_is_dealt_out(dg, dtype):
    """Few tiles, all of them with more than 512 entries: dW's partials are summed in a launch of their own there, not beside the tiles."""
    n, c, k = 1500, 2, dg // 4
    rowptr, colidx = band_graph(n, 24, 1.0, 1)
    og, gg = oracle.graph_build(rowptr, colidx), gsr.gsr_graph_create(rowptr, colidx)
    info = gsr.gsr_graph_info(gg)
    assert 40 * n < info["nnz"] < 64 * n and info["n_hub_rows"] == 0
    f32 = dtype == "f32"
    d, tdt = c * dg, torch.float32 if f32 else torch.bfloat16
    ocfg = oracle.Cfg(d, c, k, oracle.NORM_RMS, 1e-5, oracle.STORE_F32 if f32 else oracle.STORE_BF16)
    cfg = gsr.Config(n=n, d=d, c=c, k=k, l=1, dtype=gsr.GSR_F32 if f32 else gsr.GSR_BF16, norm=gsr.GSR_NORM_RMS, eps=1e-5)
    rng = np.random.default_rng(4)
    W = ((rng.random((c, dg, dg)) * 2 - 1) * np.sqrt(3.0 / dg)).astype(np.float32)
    Y, dY = (torch.from_numpy((rng.standard_normal((n, d)) * s).astype(np.float32)).to(tdt) for s in (1.0, 1e-3))
    refs = oracle.layer_backward(og, ocfg, W, Y.double().numpy(), dY.double().numpy())
    y, dy, dW = Y.cuda(), dY.cuda(), torch.empty((c, dg, dg), dtype=torch.float32, device="cuda")
    gsr.gsr_layer_backward(gg, cfg, torch.from_numpy(W).cuda(), y, dy, dW)
    for name, got, ref in zip(("X", "dX", "dW"), (y, dy, dW), refs):
        got = got.double().cpu().numpy()
        if f32:
            assert_close(name, got, ref)
        else:
            assert rel_norm(got, ref) <= BF16_REL, name


def graph_cut_at_64(rp, ci, workgroups):
    """Rows above 64 entries in chunks of 64, whatever the number of workgroups makes of the graph by itself."""
    options = {"max_workgroups": workgroups, "hub_threshold": 64, "hub_chunk": 64}
    try:
        for key, value in options.items():
            gsr.gsr_set_option(key, value)
        return gsr.gsr_graph_create(rp, ci)
    finally:
        for key in options:
            gsr.gsr_set_option(key, 0)


def net_graph(n, nets, sinks, seed):
    """Rows of two neighbours, and `nets` nodes of the second tile wired to `sinks` others each."""
    rng = np.random.default_rng(seed)
    rows, cols = np.repeat(np.arange(n), 2), rng.integers(0, n, 2 * n)
    for h in range(nets):
        rows, cols = np.concatenate([rows, np.full(sinks, 16 + h)]), np.concatenate([cols, rng.permutation(n)[:sinks]])
    key = np.unique(rows * n + cols)
    return np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int32), (key % n).astype(np.int32)


@pytest.mark.parametrize("n", [1024, 1025, 4080, 4081])
def test_rows_of_many_chunks_one_by_one_and_in_pairs(n):
    """Rows of 600 entries (ten chunks of 64), an odd number of them in one tile, with 32 waves: gsr_spmm adds them up in pairs to 64 tiles,
    gsr_spmm_compressed below 256.  The additions are the same as with a wave per tile."""
    rp, ci = net_graph(n, 3, 600, n)
    og = oracle.graph_build(rp, ci)
    got = {}
    for workgroups in (8, 0):
        g = graph_cut_at_64(rp, ci, workgroups)
        assert gsr.gsr_graph_info(g)["n_hub_rows"] == 3
        rng = np.random.default_rng(6)
        out = []
        for width in (64, 32, 16):
            X = rng.standard_normal((n, width)).astype(np.float32)
            out.append(gsr.gsr_spmm(g, torch.from_numpy(X).cuda()))
            assert_close("A X", out[-1].cpu().numpy(), oracle.spmm(og, X))
        for dg, k in ((64, 16), (32, 8), (64, 60)):
            V, I, _ = oracle.gs(rng.standard_normal((n, dg)).astype(np.float32).astype(np.float64), k)
            out.append(gsr.gsr_spmm_compressed(g, torch.from_numpy(V.astype(np.float32)).cuda(), torch.from_numpy(I.astype(np.int32)).cuda(), dg))
            assert_close("A scatter(V, I)", out[-1].cpu().numpy(), oracle.aggregate(og, V, I, dg))
        got[workgroups] = out
    assert all(torch.equal(a, b) for a, b in zip(got[8], got[0]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049])
def test_two_block_groups_by_sweep_and_by_workgroup(n, dtype):
    """8 and 9 groups of eight tiles, 16 and 17, for 8 workgroups: a sweep with W_i in LDS, a workgroup per group of tiles, and the sweep again
    (16-bit storage: the sweep from 17 on).  With 64 workgroups or more these graphs are one round: the same bits either way."""
    cs = wide_case(n, 256, 2, 32, 1, "rms", ROW, dtype)
    w, W = cs.w, cs.inp.weights[0]
    Wd = torch.from_numpy(W).to(cs.dev)
    dY = (np.random.default_rng(5).standard_normal((w.n, w.d)) * 1e-3).astype(np.float32)
    dY = torch.from_numpy(dY).to(torch.bfloat16 if dtype == "bf16" else torch.float32).double().numpy()
    Y = oracle.layer_forward(cs.og, cs.ocfg, W, cs.x0_on_grid())
    got = []
    for workgroups in (8, 0):
        g = graph_cut_at_64(cs.inp.rowptr, cs.inp.colidx, workgroups)
        y = cs.to_dev(cs.x0_on_grid())
        gsr.gsr_layer_forward(g, cs.gcfg, Wd, y)
        x, dy, dW = y.clone(), cs.to_dev(dY), torch.empty((w.c, w.dg, w.dg), dtype=torch.float32, device=cs.dev)
        gsr.gsr_layer_backward(g, cs.gcfg, Wd, x, dy, dW)
        got.append((y, x, dy, dW))
    for a, b in zip(got[0][:3], got[1][:3]):
        assert torch.equal(a, b)
    y, x, dy, dW = got[0]
    if dtype == "bf16":          # the first group's rows follow from identical inputs (16-bit near-ties make later rows select differently)
        assert not bf16_bar(cs.to_host(y)[:, :w.dg], Y[:, :w.dg]).any()
        return
    assert_close("Y", cs.to_host(y), Y)
    refs = oracle.layer_backward(cs.og, cs.ocfg, W, cs.to_host(y), dY)
    for name, have, ref in zip(("X", "dX", "dW"), (cs.to_host(x), cs.to_host(dy), dW.cpu().numpy()), refs):
        assert_close(name, have, ref)
