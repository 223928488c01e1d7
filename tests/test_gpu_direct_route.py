"""The direct route and the all-pairs sum at the sizes where their launch shapes change:
wavefronts per leaf (16, 8, 4, 1), interaction lists as rows or compact, leaves of more
than 64 points, and targets per block of the all-pairs sum (2, 8, 32, 64).

Tolerances.  A float32 term exp2(-d2) has the relative error of d2, whose coordinates
are rounded at up to six scaled units: below 4e-6 for the farthest terms, far less for
the ones that carry a sum; a chunk adds at most 64 of them in float32.  1e-5 of a sum,
and 2e-5 of the largest gradient (float32 running sums over some thousand terms), hold."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import rel_err, to_dev

pytestmark = pytest.mark.gpu


def _T(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n,leaf_max,exclude", [(1, 64, False), (70, 64, True), (5003, 64, False), (4096, 128, True),
                                                (1700, 2, False), (2400, 1, True), (5003, 1, False)])
def test_leaf_sums_and_gradients(n, leaf_max, exclude):
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(n, extent=(900.0, 900.0, 700.0), sigma=100.0, seed=4000 + n)
    wl.w[0] = 2.0
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"], leaf_max=leaf_max)
    print(f"direct route n={n} leaf_max={leaf_max} nodes={tree.info()['n_nodes']}", flush=True)
    u = tree.forward(d["w"], None, sigma=wl.sigma, route="direct", exclude_self=exclude).cpu().numpy()
    ref = oracle.attraction(wl, np.arange(n), exclude_self=exclude)
    assert np.abs(u - ref).max() <= 1e-5 * np.abs(ref).max() + 1e-30
    some = ref > 1e-3 * np.abs(ref).max()
    if some.any():
        assert rel_err(u[some], ref[some]).max() <= 1e-5
    rng = np.random.default_rng(n)
    g = (rng.random(n) + 0.5).astype(np.float32)
    got = tree.backward(d["w"], _T(g), d["tgt"], sigma=wl.sigma, route="direct", exclude_self=exclude)
    gt = np.where(wl.a > 0, g, 0).astype(np.float64)
    pos = wl.pos64()
    r = oracle.gauss_grad(pos, gt, pos, wl.w, wl.sigma)
    gw = r["w"] - (gt if exclude else 0.0)
    assert np.abs(got["w"].cpu().numpy() - gw).max() <= 2e-5 * max(np.abs(gw).max(), 1.0)
    for k in range(3):
        gp = r["t"][:, k] + r["s"][:, k]
        assert np.abs(got["pos"][k].cpu().numpy() - gp).max() <= 2e-5 * max(np.abs(r["t"]).max(), 1e-3) + 1e-6
    # the same gradients one field at a time
    only_w = tree.backward(d["w"], _T(g), d["tgt"], sigma=wl.sigma, route="direct", exclude_self=exclude, want=("w",))
    np.testing.assert_array_equal(only_w["w"].cpu().numpy(), got["w"].cpu().numpy())
    only_s = tree.backward(d["w"], _T(g), d["tgt"], sigma=wl.sigma, route="direct", exclude_self=exclude,
                           want=("sigma",))
    assert only_s["sigma"].item() == got["sigma"].item()
    # another cutoff, a workspace call in between, and back: the lists follow
    u0 = tree.forward(d["w"], None, sigma=wl.sigma, route="direct", cutoff_sigmas=0.0, exclude_self=exclude)
    assert np.abs(u0.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max() + 1e-30
    import torch
    ws = torch.empty(tree.forward_query(wl.sigma, route="direct"), dtype=torch.uint8, device="cuda")
    uw = tree.forward_ws(d["w"], ws, None, sigma=wl.sigma, route="direct", exclude_self=exclude).cpu().numpy()
    np.testing.assert_array_equal(uw, u)
    again = tree.forward(d["w"], None, sigma=wl.sigma, route="direct", exclude_self=exclude).cpu().numpy()
    np.testing.assert_array_equal(again, u)
    tree.close()


@pytest.mark.parametrize("m", [1, 2, 9, 10, 16, 17, 18, 19, 32, 33, 48, 49, 63, 64, 130])
@pytest.mark.parametrize("sigma", [24.0, 60.0, 500.0])
@pytest.mark.parametrize("exclude", [False, True])
def test_leaf_forms(m, sigma, exclude):
    """Leaves of m targets (every count of tiles and of targets per lane) of half side 25,
    scaled reach 2.2, 0.87 and 0.1: differences, and matrix products near and far from the
    bound; a list of some hundred leaves, consecutive or not; a far cluster whose terms
    all underflow.  A sum's relative error: three roundings of 2 t.s, at most 2 x 1.5 x 7
    scaled units squared in the terms of 2^-30 and 2 x 1.5 x 2.5 in those that carry a
    sum, 9e-7, with the factors' and the float32 additions' 5e-7: 2e-6."""
    import paper_2301_10570_amd as msp
    rng = np.random.default_rng(m)
    cells = np.array([(i, j, k) for i in range(8) for j in range(8) for k in range(8)])
    keep = cells[np.sort(rng.permutation(512)[: 512 if m < 20 else 100])]
    pts = (keep[:, None, :] * 50.0 + 1.0 + rng.random((len(keep), m, 3)) * 48.0).reshape(-1, 3)
    pts = np.concatenate([pts, [[0.0, 0.0, 0.0], [399.99, 399.99, 399.99]]]).astype(np.float32)
    n = len(pts)
    w = rng.integers(0, 4, n).astype(np.float32)
    w[0] = 3.0
    tree = msp.build_tree(*(_T(pts[:, k]) for k in range(3)), leaf_max=max(m, 2), max_depth=3)
    print(f"leaf forms m={m} sigma={sigma} exclude={exclude} nodes={tree.info()['n_nodes']}", flush=True)
    u = tree.forward(_T(w), None, sigma=sigma, route="direct", cutoff_sigmas=6.5, exclude_self=exclude).cpu().numpy()
    pick = rng.permutation(n)[:300]
    ref = oracle.gauss_sum(pts[pick], pts, w, sigma) - (w[pick].astype(np.float64) if exclude else 0.0)
    far = w.astype(np.float64).sum() * np.exp(-6.5 ** 2)   # what the cutoff may drop
    assert np.all(np.abs(u[pick] - ref) <= 2e-6 * np.abs(ref) + far)
    tree.close()


@pytest.mark.parametrize("m", [1, 2, 3, 15, 16, 17, 21, 22, 32, 33, 64, 100])
@pytest.mark.parametrize("cells", [100, 4000])
def test_gradient_units(m, cells):
    """Leaves of m targets: units of the running sums of every length (64 / m groups), eight
    wavefronts a leaf (100 leaves), one (4,000), four (the batch), the same bits from each
    of them where the sums run in order; the oracle on some points, 2e-5 of the largest."""
    import paper_2301_10570_amd as msp
    if cells * m > 150000:
        pytest.skip("the same units as with 33 targets")
    rng = np.random.default_rng(m + cells)
    grid = np.stack(np.meshgrid(*[np.arange(16)] * 3, indexing="ij"), -1).reshape(-1, 3)
    keep = grid[np.sort(rng.permutation(4096)[:cells])]
    pts = (keep[:, None, :] * 20.0 + 0.5 + rng.random((cells, m, 3)) * 19.0).reshape(-1, 3)
    pts = np.concatenate([pts, [[0.0, 0.0, 0.0], [319.99, 319.99, 319.99]]]).astype(np.float32)
    n, sigma = len(pts), 8.0 if cells > 100 else 80.0   # lists of some thousand points
    w = rng.integers(0, 4, n).astype(np.float32)
    g = (rng.random(n) + 0.5).astype(np.float32)
    x = [_T(pts[:, k]) for k in range(3)]
    tree = msp.build_tree(*x, leaf_max=max(m, 2), max_depth=4)
    print(f"gradient units m={m} cells={cells} nodes={tree.info()['n_nodes']}", flush=True)
    got = tree.backward(_T(w), _T(g), None, sigma=sigma, route="direct")
    pick = rng.permutation(n)[:60]
    pos = pts.astype(np.float64)
    u = oracle.gauss_sum(pts[pick], pts, g, sigma)
    assert np.abs(got["w"].cpu().numpy()[pick] - u).max() <= 2e-5 * np.abs(u).max()
    d = pos[pick][:, None, :] - pos[None]
    e = np.exp(-(d ** 2).sum(-1) / sigma ** 2)
    both = e * (g[pick][:, None].astype(np.float64) * w + w[pick][:, None].astype(np.float64) * g)
    gp = -2.0 / sigma ** 2 * (both[..., None] * d).sum(1)
    for k in range(3):
        assert np.abs(got["pos"][k].cpu().numpy()[pick] - gp[:, k]).max() <= 2e-5 * np.abs(gp).max()
    b = msp.Batch().build(*x, np.array([0, n], dtype=np.int64), leaf_max=np.array([max(m, 2)], dtype=np.int32),
                          max_depth=4)
    gb = b.backward(_T(w), _T(g), np.array([sigma], dtype=np.float32), route="direct")
    np.testing.assert_array_equal(gb["w"].cpu().numpy(), got["w"].cpu().numpy())
    assert abs(gb["sigma"].cpu().numpy()[0] - got["sigma"].item()) <= 1e-12 * abs(got["sigma"].item())
    b.close()
    tree.close()


@pytest.mark.parametrize("nt,ns", [(1, 1), (3, 127), (50, 4097), (4095, 129), (4096, 2048), (16383, 130), (16385, 2049),
                                   (65535, 300), (65537, 127), (7, 0)])
def test_all_pairs(nt, ns):
    import paper_2301_10570_amd as msp
    print(f"all-pairs sum {nt} x {ns}", flush=True)
    rng = np.random.default_rng(nt + ns)
    t = rng.random((nt, 3)).astype(np.float32) * 300
    s = rng.random((ns, 3)).astype(np.float32) * 300
    w = rng.random(ns).astype(np.float32) + 0.1
    u = msp.direct_sum(*(_T(t[:, k]) for k in range(3)), *(_T(s[:, k]) for k in range(3)), _T(w), 80.0).cpu().numpy()
    if ns == 0:
        assert np.all(u == 0)
        return
    pick = np.unique(np.concatenate([np.arange(min(nt, 70)), np.arange(max(0, nt - 70), nt)]))
    assert rel_err(u[pick], oracle.gauss_sum(t[pick], s, w, 80.0)).max() <= 1e-5
    assert np.all(np.isfinite(u)) and np.all(u > 0)


@pytest.mark.parametrize("n", [300, 5003, 40000])
def test_lists_are_not_made_in_a_recorded_call(n):
    """A direct-route call whose lists are not there yet is refused while it is recorded, and
    leaves the handle as it was; with their lengths counted (the query) or the lists there it
    is recorded, and neither it nor the eager calls between its replays take the other's."""
    import torch
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(n, extent=(900.0, 900.0, 700.0), sigma=60.0, seed=4100 + n)
    d = to_dev(wl)
    kw = dict(sigma=wl.sigma, route="direct")
    tree = msp.build_tree(d["x"], d["y"], d["z"])
    print(f"recorded direct call n={n} nodes={tree.info()['n_nodes']}", flush=True)
    ref = tree.forward(d["w"], d["tgt"], **kw).cpu().numpy()
    out = torch.zeros_like(d["w"])
    tree.build(d["x"], d["y"], d["z"])       # the buffers are there, the lists are not
    torch.cuda.synchronize()
    empty = torch.cuda.CUDAGraph()
    with torch.cuda.graph(empty):
        out.fill_(1.0)
        with pytest.raises(msp.MspError):
            tree.forward(d["w"], d["tgt"], out=out, **kw)
    for counted in (True, False):
        if counted:
            tree.forward_query(**kw)
        else:
            np.testing.assert_array_equal(tree.forward(d["w"], d["tgt"], **kw).cpu().numpy(), ref)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            tree.forward(d["w"], d["tgt"], out=out, **kw)
        for rep in range(3):
            if rep or not counted:
                np.testing.assert_array_equal(tree.forward(d["w"], d["tgt"], **kw).cpu().numpy(), ref)
            out.zero_()
            graph.replay()
            np.testing.assert_array_equal(out.cpu().numpy(), ref)
        tree.build(d["x"], d["y"], d["z"])
    tree.close()


def test_leaf_sums_take_weights_of_any_size():
    """Leaves small against sigma (scaled reach 0.95): weights of 2^-50 at 8.6 scaled units, whose
    terms of 2^-124 are normal numbers while the weight times exp2(-s^2) is not, and one of 3e38
    beside its targets, whose sum is finite while w exp2(2 t.s - s^2) is not.  Tolerances: the
    rounding of coordinates of 9.5 units, twice in d^2 = 74, and of s^2, 5e-5 of a far sum; 2e-6
    of a near one."""
    import paper_2301_10570_amd as msp
    rng = np.random.default_rng(50)
    near = 195.0 + 4.0 * rng.random((12, 3))          # towards the far corner of cell 3 of 32
    far = 420.0 + 10.0 * rng.random((9, 3))           # the middle of cell 8
    pts = np.concatenate([[[0.0] * 3], near, far, [[1599.99] * 3]]).astype(np.float32)
    tree = msp.build_tree(*(_T(pts[:, k]) for k in range(3)), leaf_max=8, max_depth=5)
    sigma, kw = 54.75, dict(sigma=54.75, route="direct", cutoff_sigmas=0.0)
    pick = np.arange(1, 13)
    w = np.zeros(len(pts), dtype=np.float32)
    w[13:22] = rng.integers(1, 4, 9) * np.float32(2.0 ** -50)
    u = tree.forward(_T(w), None, **kw).cpu().numpy()[pick]
    ref = oracle.gauss_sum(pts[pick], pts, w, sigma)
    print("far", rel_err(u, ref).max(), flush=True)
    assert ref.min() > 2.0 ** -126 and rel_err(u, ref).max() <= 5e-5
    w[:] = 0.0
    w[5] = 3e38
    u = tree.forward(_T(w), None, **kw).cpu().numpy()[pick]
    ref = oracle.gauss_sum(pts[pick], pts, w, sigma)
    assert np.all(np.isfinite(u)) and rel_err(u, ref).max() <= 2e-6
    tree.close()


@pytest.mark.parametrize("reach,bar", [(0.999, 8.2e-8), (1.2, 9.0e-8), (1.499, 1.14e-7)])
def test_leaf_sums_on_either_side_of_the_matrix_form(reach, bar):
    """Root mean square relative error of a leaf's sums, 512 leaves of 10 points, against float64:
    no larger than that of compensated float32 sums of exp2(-d^2) on the same sort of input
    (the bars, as measured)."""
    import paper_2301_10570_amd as msp
    e2 = []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        cells = np.stack(np.meshgrid(*[np.arange(8)] * 3, indexing="ij"), -1).reshape(-1, 3).repeat(10, 0)
        pts = ((cells + rng.random((5120, 3)) * 0.999 + 0.0005) * 50.0).astype(np.float32)
        pts[0], pts[-1] = 0.0, 399.9999
        w = (rng.random(5120) * 5).astype(np.float32)
        sigma = float(np.float32(np.sqrt(3.0 * np.log2(np.e)) * 25.0 / reach))
        tree = msp.build_tree(*(_T(pts[:, k]) for k in range(3)), leaf_max=10, max_depth=3)
        u = tree.forward(_T(w), None, sigma=sigma, route="direct", cutoff_sigmas=0.0).cpu().numpy()
        e2.append(rel_err(u, oracle.gauss_sum(pts, pts, w, sigma)) ** 2)
        tree.close()
    rms = np.sqrt(np.mean(e2))
    print(f"reach {reach} rms {rms:.3e}", flush=True)
    assert rms <= bar


@pytest.mark.parametrize("sigma,exclude", [(12.0, False), (40.0, True), (160.0, False), (1000.0, False)])
def test_one_wavefront_per_leaf(sigma, exclude):
    """A tree of more than 4,096 nodes: a wavefront per leaf over windows of 64 list entries, lists
    shorter and longer than one window; the batch's four wavefronts per leaf cut them alike."""
    import paper_2301_10570_amd as msp
    wl = synth.uniform_box(6000, extent=(800.0, 800.0, 800.0), sigma=sigma, seed=4200)
    d = to_dev(wl)
    tree = msp.build_tree(d["x"], d["y"], d["z"], leaf_max=1)
    assert tree.info()["n_nodes"] > 4096
    print(f"one wavefront per leaf sigma={sigma} nodes={tree.info()['n_nodes']}", flush=True)
    u = tree.forward(d["w"], None, sigma=sigma, route="direct", exclude_self=exclude).cpu().numpy()
    pick = np.random.default_rng(5).permutation(wl.n)[:500]
    ref = oracle.attraction(wl, pick, exclude_self=exclude)
    far = wl.w.astype(np.float64).sum() * np.exp(-4.5 ** 2)
    assert np.all(np.abs(u[pick] - ref) <= 1e-5 * np.abs(ref) + far)
    b = msp.Batch().build(d["x"], d["y"], d["z"], np.array([0, wl.n], dtype=np.int64),
                          leaf_max=np.array([1], dtype=np.int32))
    ub = b.forward(d["w"], np.array([sigma], dtype=np.float32), route="direct", exclude_self=exclude).cpu().numpy()
    np.testing.assert_array_equal(ub, u)
    b.close()
    tree.close()


@pytest.mark.parametrize("nt,ns", [(1279, 300), (1280, 300), (1281, 4097)])
def test_all_pairs_where_eight_targets_share_a_block(nt, ns):
    import paper_2301_10570_amd as msp
    print(f"all-pairs sum {nt} x {ns}", flush=True)
    rng = np.random.default_rng(nt + ns)
    t = rng.random((nt, 3)).astype(np.float32) * 300
    s = rng.random((ns, 3)).astype(np.float32) * 300
    w = rng.random(ns).astype(np.float32) + 0.1
    u = msp.direct_sum(*(_T(t[:, k]) for k in range(3)), *(_T(s[:, k]) for k in range(3)), _T(w), 80.0).cpu().numpy()
    assert rel_err(u, oracle.gauss_sum(t, s, w, 80.0)).max() <= 1e-5
