"""The backward on graphs of long rows in a band, where dY_i W_i^T is taken before the gather over A^T and only the recorded columns are
gathered (windows of rows staged in LDS), against the oracle: every group width, one to four values per lane, rows that end inside a
window and rows that fill several passes of one, rows without a neighbour, a last workgroup that is not full."""
import numpy as np
import pytest

import oracle
import paper_2603_27156_amd as gsr
from gpu_util import BF16_REL, NORM, assert_close, rel_norm

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
