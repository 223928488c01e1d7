"""The expansion route with its table of cells, the passes that skip empty cells and the
point runs of the L2P: the bits of the same call in a caller's workspace, which searches
for the cells and computes every one of them, and the accuracy bar."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import rel_err, to_dev

pytestmark = pytest.mark.gpu


def _make(kind, n):
    if kind == "blobs":        # a few per cent of the cells hold points
        return synth.blobs(n // 512, 512, extent=3000.0, std=30.0, sigma=120.0, seed=900 + n)
    if kind == "line":         # one row of cells along x, most of the grid empty in y and z
        return synth.uniform_box(n, extent=(4000.0, 30.0, 20.0), sigma=100.0, seed=901)
    if kind == "corners":      # two far corners of the cube
        wl = synth.uniform_box(n, extent=(200.0, 200.0, 200.0), sigma=110.0, seed=902)
        for v in (wl.x, wl.y, wl.z):
            v[n // 2:] += np.float32(3800.0)
        return wl
    return synth.uniform_box(n, extent=(1500.0, 900.0, 400.0), sigma=150.0, seed=903)


@pytest.mark.parametrize("kind,n,p", [("blobs", 16384, 8), ("blobs", 512, 8), ("line", 3001, 8), ("corners", 5000, 8),
                                      ("box", 63, 8), ("box", 65, 6), ("box", 257, 10), ("box", 30011, 13),
                                      ("box", 1048576 + 77, 8), ("blobs", 16384, 5)])
def test_same_bits_as_without_the_table(kind, n, p):
    import torch
    import paper_2301_10570_amd as msp
    wl = _make(kind, n)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    plan = tree.plan(wl.sigma, p=p, route="fgt")
    print(f"{kind} n={wl.n} p={p} level {plan['level']} grid {plan['grid']}", flush=True)
    ws = torch.empty(tree.forward_query(wl.sigma, p=p, route="fgt"), dtype=torch.uint8, device="cuda")
    ws.fill_(0xff)             # what is not written must not be read: NaN everywhere
    ref = tree.forward_ws(d["w"], ws, d["tgt"], sigma=wl.sigma, p=p, route="fgt").cpu().numpy()
    for rep in range(2):       # the table made, then kept
        u = tree.forward(d["w"], d["tgt"], sigma=wl.sigma, p=p, route="fgt").cpu().numpy()
        np.testing.assert_array_equal(u, ref)
    # another sigma at the same level (other bands), then the first again
    s2 = wl.sigma * 0.97
    if tree.plan(s2, p=p, route="fgt")["level"] == plan["level"]:
        u2 = tree.forward(d["w"], d["tgt"], sigma=s2, p=p, route="fgt").cpu().numpy()
        r2 = tree.forward_ws(d["w"], ws, d["tgt"], sigma=s2, p=p, route="fgt").cpu().numpy()
        np.testing.assert_array_equal(u2, r2)
    u = tree.forward(d["w"], d["tgt"], sigma=wl.sigma, p=p, route="fgt").cpu().numpy()
    np.testing.assert_array_equal(u, ref)
    # NaN weights leave NaN in every grid entry that is written: none of it is read again
    tree.forward(torch.full_like(d["w"], float("nan")), d["tgt"], sigma=wl.sigma, p=p, route="fgt")
    u = tree.forward(d["w"], d["tgt"], sigma=wl.sigma, p=p, route="fgt").cpu().numpy()
    np.testing.assert_array_equal(u, ref)
    tgt = np.nonzero(wl.a > 0)[0]
    sel = tgt[synth.sample_indices(tgt.size, 64, seed=904)]
    r = oracle.attraction(wl, sel)
    some = r > 1e-2 * r.max()
    assert rel_err(u[sel][some], r[some]).max() <= 1e-4
    # other points in the same handle: the table is made again
    tree.build(d["y"], d["x"], d["z"])
    u3 = tree.forward(d["w"], d["tgt"], sigma=wl.sigma, p=p, route="fgt").cpu().numpy()
    assert rel_err(u3[sel][some], r[some]).max() <= 1e-4
    tree.close()


@pytest.mark.parametrize("p", [1, 2, 3, 5, 6, 7])
@pytest.mark.parametrize("m2l", ["mfma", "bf16x3"])
def test_padded_translation_tiles(p, m2l):
    """Orders below eight run on the tiles of eight terms per cell, padded with zeros:
    against the vector passes, 1e-5 (float32) and 5e-5 (about 2^-16 per product) as for
    the unpadded tiles, on a grid ragged in every axis."""
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(9001, extent=(1300.0, 700.0, 500.0), sigma=400.0, seed=905)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    print(f"padded tiles p={p} {m2l} grid {tree.plan(wl.sigma, p=p, level=4, route='fgt')['grid']}", flush=True)
    kw = dict(sigma=wl.sigma, p=p, level=4, route="fgt")
    u = tree.forward(d["w"], d["tgt"], m2l=m2l, **kw).cpu().numpy()
    C = tree.debug_buffer(1).cpu().numpy()
    v = tree.forward(d["w"], d["tgt"], m2l="valu", **kw).cpu().numpy()
    Cv = tree.debug_buffer(1).cpu().numpy()
    tgt = wl.a > 0
    assert np.abs(C - Cv).max() <= (1e-5 if m2l == "mfma" else 2e-4) * np.abs(Cv).max()
    assert rel_err(u[tgt], v[tgt]).max() <= (1e-5 if m2l == "mfma" else 5e-5)
    tree.close()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 48, 63, 64, 65, 257, 5001, 1048575, 1048577])
def test_l2p_runs(n):
    """The L2P at p = 8 on runs that end inside a group of 16 or of 64 points, cells of one
    point and of thousands, keys per lane and cells from the table: small cells (half a cell
    is 0.05 sigma), so that the series' tails are far below the rounding of 64 float32 terms,
    2e-6."""
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(n, extent=(300.0, 300.0, 300.0), sigma=200.0, seed=906 + n)
    wl.w[:] = np.maximum(wl.w, 1)
    if n > 4:   # a cell that holds many
        for v in (wl.x, wl.y, wl.z):
            v[n // 2:n // 2 + n // 4] = np.float32(150.5) + np.float32(0.01) * v[n // 2:n // 2 + n // 4]
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    print(f"l2p runs n={n}", flush=True)
    u = tree.forward(d["w"], None, sigma=wl.sigma, p=8, level=4, route="fgt").cpu().numpy()
    pick = np.arange(n) if n < 300 else np.random.default_rng(n).permutation(n)[:100]
    ref = oracle.attraction(wl, pick)
    assert rel_err(u[pick], ref).max() <= 2e-6
    tree.close()


def test_batch_layouts_alternate():
    """Calls of one batch with other sigmas, orders and tiles in turn, replayed: each finds the
    tables and cleared cells of its own plan.  The expansions are summed in one order, so a
    call's bits are those of a batch of its own."""
    import torch
    import paper_2301_10570_amd as msp
    rng = np.random.default_rng(77)
    sizes = [9000, 40, 7000, 12000]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    pts = (rng.random((n, 3)) * np.repeat([1.0, 0.3, 0.5, 1.0], sizes)[:, None] * 900.0).astype(np.float32)
    pts[:3000] = pts[:3000] * 0.2   # cells without points, and full ones
    x = [torch.from_numpy(np.ascontiguousarray(pts[:, k])).cuda() for k in range(3)]
    w = torch.from_numpy(rng.integers(0, 4, n).astype(np.float32)).cuda()
    g = torch.from_numpy(rng.random(n).astype(np.float32)).cuda()
    sig = [np.full(4, s, dtype=np.float32) for s in (150.0, 260.0)]
    calls = [(0, 8, "mfma"), (1, 8, "mfma"), (1, 6, "mfma"), (0, 8, "bf16x3")]

    def run(b, call, back):
        s, p, m2l = calls[call]
        if back:
            r = b.backward(w, g, sig[s], p=p, route="fgt", m2l=m2l, out=outs.setdefault((id(b), call), None),
                           use_graph=True)
            outs[(id(b), call)] = r
            return [r["w"].clone(), r["pos"][1].clone(), r["sigma"].clone()]
        u = us.setdefault((id(b), call), torch.empty(n, device="cuda"))
        return [b.forward(w, sig[s], p=p, route="fgt", m2l=m2l, out=u, use_graph=True).clone()]

    outs, us, own = {}, {}, {}
    for call in range(len(calls)):
        for back in (False, True):
            b = msp.Batch().build(*x, off)
            own[call, back] = run(b, call, back)
            torch.cuda.synchronize()
            b.close()
    b = msp.Batch().build(*x, off)
    for call, back in [(0, False), (1, True), (0, False), (1, True), (1, True), (2, False), (1, True), (2, False),
                       (3, True), (2, False), (3, True), (0, False), (0, True), (0, False), (3, True), (0, False)]:
        print(f"call {calls[call]} backward={back}", flush=True)
        for got, want in zip(run(b, call, back), own[call, back]):
            torch.testing.assert_close(got, want, rtol=0, atol=0)
    b.close()


@pytest.mark.parametrize("extent", [(240.0, 640.0, 80.0), (640.0, 240.0, 80.0), (240.0, 80.0, 640.0)])
def test_masks_where_a_tile_may_not_fit(extent):
    """Cells far smaller than sigma along 64 cells: nearly every pair of cells translates, so
    the tile of that axis takes more LDS than those of the others.  Whatever passes run, none
    reads what a pass that skips cells has not written: every grid entry is NaN beforehand."""
    import torch
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(2000, extent=(1.0, 1.0, 1.0), sigma=125.0, seed=907)
    half = wl.n // 2
    for v, e in zip((wl.x, wl.y, wl.z), extent):     # clusters at opposite ends of the grid
        v[:] = v * np.float32(0.1 * e)
        v[half:] += np.float32(0.9 * e)
        v[0], v[-1] = 0.0, e
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=8, level=6, route="fgt")
    print(f"masks extent {extent} grid {tree.plan(**kw)['grid']}", flush=True)
    ws = torch.empty(tree.forward_query(**kw), dtype=torch.uint8, device="cuda")
    ref = tree.forward_ws(d["w"], ws, d["tgt"], **kw).cpu().numpy()
    tree.forward(torch.full_like(d["w"], float("nan")), d["tgt"], m2l="valu", **kw)   # (writes all of the grids)
    for rep in range(2):
        u = tree.forward(d["w"], d["tgt"], **kw).cpu().numpy()
        np.testing.assert_array_equal(u, ref)
    tgt = np.nonzero(wl.a > 0)[0]
    sel = tgt[synth.sample_indices(tgt.size, 64, seed=908)]
    assert rel_err(u[sel], oracle.attraction(wl, sel)).max() <= 1e-4
    tree.close()


@pytest.mark.parametrize("kind,n,p", [("blobs", 16384, 8), ("box", 1048576 + 77, 8), ("box", 1048576 + 77, 6),
                                      ("box", 30011, 10)])
def test_recorded_call_and_the_table(kind, n, p):
    """A forward recorded into a caller's graph finds its cells at each replay: the eager call
    after the recording makes its own table, and a replay after another build (other points in
    the same box and buffers) gives the sums of those points."""
    import torch
    import paper_2301_10570_amd as msp
    wl = _make(kind, n)
    d = to_dev(wl)
    g = torch.Generator().manual_seed(n)
    other = d["x"][torch.randperm(wl.n, generator=g).cuda()].contiguous()   # the same extent
    kw = dict(sigma=wl.sigma, p=p, route="fgt")
    print(f"recorded {kind} n={wl.n} p={p}", flush=True)
    tree = msp.Tree().build(other, d["y"], d["z"])
    ref_other = tree.forward(d["w"], d["tgt"], **kw).cpu().numpy()
    tree.build(d["x"], d["y"], d["z"])
    ref = tree.forward(d["w"], d["tgt"], **kw).cpu().numpy()
    tree.build(other, d["y"], d["z"])
    tree.build(d["x"], d["y"], d["z"])
    out = torch.zeros_like(d["w"])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tree.forward(d["w"], d["tgt"], out=out, **kw)
    np.testing.assert_array_equal(tree.forward(d["w"], d["tgt"], **kw).cpu().numpy(), ref)
    for rep in range(2):
        out.zero_()
        graph.replay()
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
    tree.build(other, d["y"], d["z"])
    for rep in range(2):
        out.zero_()
        graph.replay()
        np.testing.assert_array_equal(out.cpu().numpy(), ref_other)
        np.testing.assert_array_equal(tree.forward(d["w"], d["tgt"], **kw).cpu().numpy(), ref_other)
    tree.close()


@pytest.mark.parametrize("kind,n", [("blobs", 16384), ("corners", 5000)])
def test_debug_buffers_hold_whole_grids(kind, n):
    """The Taylor grid that the debug buffer gives after a call that skipped empty cells: every
    cell, as the vector passes have it (1e-5 of the largest), and the moments untouched by it."""
    import torch
    import paper_2301_10570_amd as msp
    wl = _make(kind, n)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=8, route="fgt")
    print(f"debug buffers {kind} n={wl.n} grid {tree.plan(**kw)['grid']}", flush=True)
    tree.forward(d["w"], d["tgt"], m2l="valu", **kw)
    Av, Cv = (tree.debug_buffer(k).cpu().numpy() for k in (0, 1))
    tree.forward(torch.full_like(d["w"], float("nan")), d["tgt"], m2l="valu", **kw)   # (writes all of the grids)
    for rep in range(2):
        tree.forward(d["w"], d["tgt"], **kw)
        A, C = (tree.debug_buffer(k).cpu().numpy() for k in (0, 1))
        np.testing.assert_array_equal(A, Av)
        assert np.abs(C - Cv).max() <= 1e-5 * np.abs(Cv).max()
        np.testing.assert_array_equal(tree.debug_buffer(1).cpu().numpy(), C)
    tree.close()


@pytest.mark.parametrize("p,extent", [(1, (1275.0, 1275.0, 75.0)), (3, (1275.0, 1275.0, 75.0)),
                                      (4, (1275.0, 1275.0, 75.0)), (5, (1175.0, 1275.0, 75.0)),
                                      (4, (300.0, 1275.0, 75.0)), (7, (1175.0, 1275.0, 75.0))])
def test_whole_rows_where_the_padded_tile_does_not_serve(p, extent):
    """Grids up to 128 cells wide: the tile of p terms per cell where the padded one is too large
    or (p below five) does more work, in forward sums as in gradients: the same Taylor grid from
    the same weights; and the vector passes to 1e-5."""
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(20000, extent=extent, sigma=96.0, seed=909)
    for k, v in enumerate((wl.x, wl.y, wl.z)):
        v[0], v[-1] = 0.0, extent[k] + (4.9 if k == 1 else 0.0)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=p, level=7, route="fgt")
    print(f"wide grid p={p} {tree.plan(**kw)['grid']}", flush=True)
    u = tree.forward(d["w"], None, **kw).cpu().numpy()
    C = tree.debug_buffer(1).cpu().numpy()
    v = tree.forward(d["w"], None, m2l="valu", **kw).cpu().numpy()
    Cv = tree.debug_buffer(1).cpu().numpy()
    assert np.abs(C - Cv).max() <= 1e-5 * np.abs(Cv).max()
    assert rel_err(u, v).max() <= 1e-5
    if p != 7:
        tree.backward(d["w"], d["w"], None, want=("w",), **kw)    # the field of the same weights
        np.testing.assert_array_equal(tree.debug_buffer(1).cpu().numpy(), C)
    tree.close()


@pytest.mark.parametrize("extent", [(560.0, 635.0, 35.0), (570.0, 635.0, 35.0), (620.0, 635.0, 35.0), (35.0, 635.0, 630.0)])
def test_wide_rows_that_reach_each_other(extent):
    """p = 8 on 56 to 64 cells an axis that all translate into each other: operator blocks apart
    in LDS, or packed where only that fits; against the vector passes, 1e-5."""
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(60000, extent=extent, sigma=200.0, seed=910)
    for k, v in enumerate((wl.x, wl.y, wl.z)):
        v[0], v[-1] = 0.0, extent[k] - 0.1 + (5.0 if k == 1 else 0.0)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=8, level=6, route="fgt")
    print(f"wide rows {tree.plan(**kw)['grid']}", flush=True)
    tree.forward(d["w"], None, **kw)
    tree.set_timing(True)
    u = tree.forward(d["w"], None, **kw).cpu().numpy()
    print({k: round(1e3 * v[0], 1) for k, v in tree.timing().items() if "m2l" in k}, flush=True)
    C = tree.debug_buffer(1).cpu().numpy()
    v = tree.forward(d["w"], None, m2l="valu", **kw).cpu().numpy()
    Cv = tree.debug_buffer(1).cpu().numpy()
    assert np.abs(C - Cv).max() <= 1e-5 * np.abs(Cv).max()
    assert rel_err(u, v).max() <= 1e-5
    tree.close()


@pytest.mark.parametrize("n,p", [(1, 9), (65, 9), (700, 9), (30011, 11), (4000, 12), (700, 13), (20000, 16)])
def test_l2p_by_cells(n, p):
    """Orders above eight, a block per cell: cells of one point, of more than a block's 1,024, and
    none; the bits of the same call in a workspace, and the float32 sums' rounding, 2e-6."""
    import torch
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(n, extent=(400.0, 300.0, 200.0), sigma=200.0, seed=920 + n)
    wl.w[:] = np.maximum(wl.w, 1)
    if n > 4000:   # a cell that holds many
        for v in (wl.x, wl.y, wl.z):
            v[n // 2:n // 2 + 1500] = np.float32(150.5) + np.float32(0.01) * v[n // 2:n // 2 + 1500]
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=p, level=4, route="fgt")
    print(f"l2p by cells n={n} p={p}", flush=True)
    u = tree.forward(d["w"], d["tgt"], **kw).cpu().numpy()
    ws = torch.empty(tree.forward_query(**kw), dtype=torch.uint8, device="cuda")
    np.testing.assert_array_equal(tree.forward_ws(d["w"], ws, d["tgt"], **kw).cpu().numpy(), u)
    tgt = np.nonzero(wl.a > 0)[0]
    pick = tgt[:100]
    assert np.all(u[wl.a <= 0] == 0) and (pick.size == 0 or rel_err(u[pick], oracle.attraction(wl, pick)).max() <= 2e-6)
    tree.close()


@pytest.mark.parametrize("n", [6143, 6144, 12287, 49152, 98303, 98304])
@pytest.mark.parametrize("p", [5, 8])
def test_l2p_run_lengths(n, p):
    """Either side of the point counts where a wavefront's run halves, cells across runs: the bits
    of the workspace call, which searches the cells, and the series' bar at that cell size (half
    a cell is some 0.16 sigma), 1e-4."""
    import torch
    import paper_2301_10570_amd as msp
    wl = synth.blobs(n // 256 + 1, 256, extent=3000.0, std=60.0, sigma=340.0, seed=930 + n)
    for k in ("x", "y", "z", "w", "a"):
        setattr(wl, k, getattr(wl, k)[:n].copy())
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=p, level=5, route="fgt")
    print(f"l2p run lengths n={n} p={p}", flush=True)
    u = tree.forward(d["w"], None, **kw).cpu().numpy()
    ws = torch.empty(tree.forward_query(**kw), dtype=torch.uint8, device="cuda")
    np.testing.assert_array_equal(tree.forward_ws(d["w"], ws, None, **kw).cpu().numpy(), u)
    pick = np.random.default_rng(n).permutation(n)[:60]
    ref = oracle.attraction(wl, pick)
    assert rel_err(u[pick], ref).max() <= 1e-4
    tree.close()


@pytest.mark.parametrize("n,sigma", [(30011, 150.0), (1048576 + 77, 110.0)])
def test_l2p_rounds_no_more_than_horner(n, sigma):
    """The series at p = 8 from the Taylor grid itself, against float64 at the same float32 local
    coordinates: the root mean square rounding of the sums is at most that of a Horner evaluation
    in float32 multiply-adds (a float64 step rounded to float32)."""
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(n, extent=(1500.0, 900.0, 400.0), sigma=sigma, seed=940)
    wl.w[:] = np.maximum(wl.w, 1)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    kw = dict(sigma=wl.sigma, p=8, route="fgt")
    plan, info = tree.plan(**kw), tree.info()
    G, cell = plan["grid"], info["side"] / 2.0 ** plan["level"]
    u = tree.forward(d["w"], None, **kw).cpu().numpy()
    C = tree.debug_buffer(1).cpu().numpy().reshape(G[2], 8, G[1], 8, G[0], 8)
    pick = np.random.default_rng(n).permutation(n)[:20000]
    pos = np.stack([wl.x, wl.y, wl.z], 1)[pick]
    k = np.minimum(((pos.astype(np.float64) - info["lo"]) / cell).astype(int), np.array(G) - 1)
    c32 = (np.array(info["lo"]) + (k + 0.5) * cell).astype(np.float32)
    t = (pos - c32) * np.float32(1.0 / wl.sigma)
    keep = np.abs(t).max(1) < 0.4999 * cell / wl.sigma       # (the key decides on a cell's faces)
    t, k, got = t[keep].astype(np.float64), k[keep], u[pick][keep]
    co = C[k[:, 2], :, k[:, 1], :, k[:, 0], :].astype(np.float64)      # [point][az][ay][ax]
    powers = [t[:, a, None] ** np.arange(8) for a in range(3)]
    exact = np.matmul(np.matmul(np.matmul(co, powers[0][:, None, :, None])[..., 0], powers[1][:, :, None])[..., 0][:, None, :],
                      powers[2][:, :, None])[:, 0, 0]
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    h = co
    for a in range(3):                                       # x, then y, then z
        x = t[:, a].reshape((-1,) + (1,) * (h.ndim - 2))
        acc = h[..., 7]
        for q in range(6, -1, -1):
            acc = f32(acc * x + h[..., q])
        h = acc
    rms = [float(np.sqrt(np.mean(((v - exact) / exact) ** 2))) for v in (got.astype(np.float64), h)]
    print(f"l2p rounding n={n} rho {plan['rho']:.2f}: kernel {rms[0]:.2e}, Horner {rms[1]:.2e}", flush=True)
    assert rms[0] <= rms[1]
    tree.close()
