"""The work that a program using this framework has it do, as cases to be timed.

Each case goes through the public entry points (Tree, Batch, attraction, direct_sum)
the way a simulation or training loop calls them.  The placements are the synthetic
ones of the tests and the bench (uniform cubes and slabs of the same neuron density,
Gaussian blobs, batches of uneven populations), drawn on the GPU from the seed.

Kinds
  sums         octree build and attraction sums: neurons whose positions have changed
  cached       attraction sums on a tree that is kept: positions stay, counts change
  step         one connectivity update: weighted build, sums, partner probabilities,
               the last two on two streams
  train        attraction() forward and its backward to positions, weights and sigma
  batch        sums of many uneven populations on trees that are kept
  batch_train  the same, with the gradients
  descent      the whole partner descent with the acceptance, on a tree that is kept
  direct       the all-pairs sum, for targets and sources given apart
"""
import math

import numpy as np
import torch

import paper_2301_10570_amd as msp

SLAB = (10000.0, 10000.0, 2000.0, 4194304)   # micrometres, neurons: 21 neurons per (100 um)^3
CUBE = (1000.0, 4096)
QUERIES_PER_NEURON = 65536 / 4194304


def listed():
    return [
        # a small network that is still moving (growth phase): launches and host work
        dict(name="sums_cube_1k", kind="sums", shape="cube", n=1021, sigma=100.0, p=8),
        # the smallest of the benchmark's networks, positions fixed: one call per update
        dict(name="cached_cube_4k", kind="cached", shape="cube", n=4096, sigma=100.0, p=8),
        # clustered neurons (cortical columns), positions fixed
        dict(name="cached_blobs_262k", kind="cached", shape="blobs", n=262144, sigma=200.0, p=8),
        # an odd size at another order, translation in split bfloat16, no self connections
        dict(name="cached_slab_1m_p6_split", kind="cached", shape="slab", n=1000003, sigma=750.0, p=6, m2l="bf16x3",
             exclude_self=True),
        # the benchmark's network, positions fixed: what most updates of a simulation do
        dict(name="cached_slab_4m", kind="cached", shape="slab", n=4194304, sigma=750.0, p=8),
        # the benchmark's step: everything of one connectivity update
        dict(name="step_slab_4m", kind="step", shape="slab", n=4194304, sigma=750.0, p=8),
        # fitting a small network's placement: forward and backward, latency bound
        dict(name="train_cube_5k", kind="train", shape="cube", n=5003, sigma=100.0, p=8),
        # the gradient benchmark: 1,048,576 sources and as many separate targets
        dict(name="train_pair_2m", kind="train", shape="pair", n=2097152, sigma=200.0, p=8),
        # the batch benchmark: 256 uneven populations on one GPU
        dict(name="batch_256", kind="batch", npop=256, lo=1024, hi=65536, p=8),
        # a smaller batch, with gradients
        dict(name="batch_train_48", kind="batch_train", npop=48, lo=1024, hi=32768, p=8),
        # who connects to whom: Algorithm 1 over the clustered neurons
        dict(name="descent_blobs_262k", kind="descent", shape="blobs", n=262144, sigma=200.0, p=8),
        # the reference sum at sampled targets against every source of a larger network
        dict(name="direct_16k_262k", kind="direct", shape="slab", n=262144, targets=16384, sigma=750.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sums", "cached", "cached", "step", "train", "batch", "batch_train", "descent", "direct"])
    if kind in ("batch", "batch_train"):
        most = 256 if kind == "batch" else 48
        p = rng.choice([6, 8, 8, 8])
        return dict(kind=kind, npop=_log(rng, 4, most), lo=_log(rng, 200, 2000), hi=_log(rng, 4000, 32768), p=p,
                    m2l=rng.choice(["mfma", "mfma", "bf16x3"]) if p == 8 else "mfma")
    if kind == "direct":
        return dict(kind=kind, shape=rng.choice(["cube", "slab"]), n=_log(rng, 300, 262144), targets=_log(rng, 50, 16384),
                    sigma=float(rng.randint(80, 750)))
    lo, hi = dict(sums=(300, 2000000), cached=(300, 4000000), step=(20000, 3000000), train=(500, 1500000),
                  descent=(500, 200000))[kind]
    shape = rng.choice(dict(step=["slab", "slab", "blobs"], train=["cube", "slab", "pair"], descent=["blobs", "cube"])
                       .get(kind, ["cube", "slab", "blobs"]))
    n = _log(rng, lo, hi)
    # the kernel's width follows the placement, as in the benchmark's workloads
    sigma = dict(cube=rng.randint(80, 200), slab=rng.randint(500, 800), blobs=rng.randint(150, 300),
                 pair=rng.randint(150, 250))[shape]
    case = dict(kind=kind, shape=shape, n=min(n, 262144) if shape == "blobs" else n, sigma=float(sigma),
                p=rng.choice([6, 8, 8, 8, 10]))
    if kind in ("sums", "cached", "train"):
        case["exclude_self"] = rng.random() < 0.25
        case["m2l"] = rng.choice(["mfma", "mfma", "mfma", "bf16x3"])
    return case


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _counts(n, g):
    """Vacant elements of each neuron, 0..5."""
    return torch.randint(0, 6, (n,), device="cuda", generator=g).to(torch.float32)


def _place(shape, n, g):
    """x, y, z (float32) of n neurons."""
    if shape == "blobs":      # 64 Gaussian clusters in a 4 mm cube, std 50 um
        c = torch.rand((64, 3), device="cuda", dtype=torch.float64, generator=g) * 4000.0
        of = torch.arange(n, device="cuda") * 64 // n
        pos = c[of] + 50.0 * torch.randn((n, 3), device="cuda", dtype=torch.float64, generator=g)
    else:
        if shape == "slab":   # the slab's thickness and density, as wide as n needs
            wide = SLAB[0] * math.sqrt(n / SLAB[3])
            ext = (wide, wide, SLAB[2])
        elif shape == "pair":  # 1,048,576 sources and as many targets in a 2 mm cube
            ext = (2000.0 * (n / 2097152) ** (1 / 3),) * 3
        else:                 # 4,096 neurons in a 1 mm cube
            ext = (CUBE[0] * (n / CUBE[1]) ** (1 / 3),) * 3
        pos = torch.rand((n, 3), device="cuda", dtype=torch.float64, generator=g) * torch.tensor(ext, device="cuda", dtype=torch.float64)
    return [pos[:, k].to(torch.float32).contiguous() for k in range(3)]


def _inputs(case, seed):
    """Positions, vacant dendrites w, vacant axons a (a target is a neuron with a > 0)
    and upstream gradients of one point set."""
    g = _gen(seed)
    n = case["n"]
    xyz = _place(case["shape"], n, g)
    a, w = _counts(n, g), _counts(n, g)
    if case["shape"] == "pair":
        second = torch.arange(n, device="cuda") >= n // 2
        a, w = second.to(torch.float32), torch.where(second, 0.0, w)
    up = torch.rand(n, device="cuda", generator=g) + 0.5
    return dict(xyz=xyz, a=a, w=w, tg=(a > 0).to(torch.uint8), up=up, gen=g)


def _populations(case, seed):
    """Sizes, sigmas, and the concatenated arrays of a batch."""
    r = np.random.default_rng(int(seed))
    # spread evenly over the logarithm, so that every seed asks the same amount of work
    q = (np.arange(case["npop"]) + 0.5) / case["npop"]
    sizes = np.rint(np.exp(np.log(case["lo"]) + q * np.log(case["hi"] / case["lo"]))).astype(np.int64)
    sigmas = np.exp(np.log(50.0) + np.random.default_rng(5).permutation(q) * np.log(6.0)).astype(np.float32)
    order = r.permutation(case["npop"])
    off = np.concatenate([[0], np.cumsum(sizes[order])]).astype(np.int64)
    g = _gen(seed)
    n = int(off[-1])
    xyz = [torch.rand(n, device="cuda", generator=g) * 1000.0 for _ in range(3)]
    a, w = _counts(n, g), _counts(n, g)
    return dict(off=off, sigmas=sigmas[order], xyz=xyz, w=w, tg=(a > 0).to(torch.uint8),
                up=torch.rand(n, device="cuda", generator=g) + 0.5)


def _keys(xyz):
    """63-bit Morton keys in the cube from the smallest corner with the largest extent."""
    lo = [float(v.min()) for v in xyz]
    side = max(float(v.max()) - l for v, l in zip(xyz, lo)) or 1.0
    key = torch.zeros_like(xyz[0], dtype=torch.int64)
    for k, (v, l) in enumerate(zip(xyz, lo)):
        q = ((v.double() - l) * (2.0 ** 21 / side)).floor().clamp(max=2 ** 21 - 1).to(torch.int64)
        for b in range(21):
            key |= ((q >> b) & 1) << (3 * b + 2 - k)
    return key


def _queries(xyz, k, g, leaf_max=64):
    """k partner queries in the descent's proportions: the node uniform among the inner
    nodes, the target uniform among its points.  Node ids count the nodes breadth first,
    by level and then by key; a cell is a node if its parent holds more than leaf_max."""
    key, perm = torch.sort(_keys(xyz), stable=True)
    ids, firsts, counts, levels, at = [], [], [], [], 0
    split = torch.ones(1, dtype=torch.bool, device="cuda")
    owner = torch.zeros_like(key)
    for level in range(21):
        cell, of, cnt = torch.unique_consecutive(key >> (3 * (21 - level)), return_inverse=True, return_counts=True)
        first = torch.cumsum(cnt, 0) - cnt
        node = split[owner[first]]                  # the parent cell is an inner node
        number = at + torch.cumsum(node, 0) - 1
        inner = node & (cnt > leaf_max)
        ids.append(number[inner]), firsts.append(first[inner]), counts.append(cnt[inner])
        levels.append(torch.full_like(first[inner], level))
        at += int(node.sum())
        if not bool(inner.any()):
            break
        split, owner = inner, of
    ids, firsts, counts, levels = (torch.cat(v) for v in (ids, firsts, counts, levels))
    pick = torch.randint(0, ids.numel(), (k,), device="cuda", generator=g)
    pos = firsts[pick] + (torch.rand(k, device="cuda", dtype=torch.float64, generator=g) * counts[pick]).to(torch.int64)
    uni = torch.rand(k, device="cuda", generator=g)
    return dict(target=perm[pos].to(torch.int32), node=ids[pick].to(torch.int32), uni=uni,
                key=key, perm=perm, first=firsts[pick], count=counts[pick], level=levels[pick])


def _options(case):
    return dict(p=case["p"], exclude_self=case.get("exclude_self", False), m2l=case.get("m2l", "mfma"))


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "batch_train"):
        s = _populations(case, seed)
        s["batch"] = msp.Batch().build(*s["xyz"], s["off"])
        s["u"] = torch.empty_like(s["w"])
        s["grads"] = None
        return dict(s, case=case)
    s = _inputs(case, seed)
    if kind == "direct":
        pick = torch.randperm(case["n"], device="cuda", generator=s["gen"])[:min(case["targets"], case["n"])]
        s["t"] = [v[pick].contiguous() for v in s["xyz"]]
        s["u"] = torch.empty_like(s["t"][0])
        return dict(s, case=case)
    s["tree"] = msp.Tree()
    s["u"] = torch.empty_like(s["w"])
    if kind in ("cached", "descent"):
        s["tree"].build(*s["xyz"])
    if kind == "step":
        k = max(64, int(case["n"] * QUERIES_PER_NEURON))
        q = _queries(s["xyz"], k, s["gen"])
        s.update(target=q["target"], node=q["node"], uni=q["uni"], side=torch.cuda.Stream(),
                 probs=torch.empty(8 * k, device="cuda"), choice=torch.empty(k, dtype=torch.int32, device="cuda"))
    if kind == "train":
        s["leaf"] = [v.requires_grad_() for v in s["xyz"]] + [s["w"].requires_grad_()]
        s["sigma"] = torch.tensor(case["sigma"], dtype=torch.float64, device="cuda", requires_grad=True)
    return dict(s, case=case)


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "direct":
        return msp.direct_sum(*s["t"], *s["xyz"], s["w"], case["sigma"], out=s["u"])
    if kind == "cached":
        return s["tree"].forward(s["w"], s["tg"], sigma=case["sigma"], out=s["u"], **_options(case))
    if kind == "sums":
        s["tree"].build(*s["xyz"])
        return s["tree"].forward(s["w"], s["tg"], sigma=case["sigma"], out=s["u"], **_options(case))
    if kind == "step":
        tree, side, main = s["tree"], s["side"], torch.cuda.current_stream()
        tree.build(*s["xyz"], w=s["w"])
        side.wait_stream(main)
        tree.forward(s["w"], s["tg"], sigma=case["sigma"], p=case["p"], out=s["u"], weights_staged=True)
        with torch.cuda.stream(side):
            tree.partner_probabilities(s["w"], s["target"], s["node"], case["sigma"], p=case["p"], uniforms=s["uni"],
                                       weights_staged=True, out=(s["probs"], s["choice"]))
        main.wait_stream(side)
        return dict(u=s["u"], probs=s["probs"], choice=s["choice"])
    if kind == "train":
        u = msp.attraction(*s["leaf"], s["sigma"], is_target=s["tg"], tree=s["tree"], **_options(case))
        return [u] + list(torch.autograd.grad(u, s["leaf"] + [s["sigma"]], grad_outputs=s["up"]))
    if kind == "descent":
        r = s["tree"].partner_descent(s["w"], s["a"], case["sigma"], 11, p=case["p"], cutoff_sigmas=4.5)
        # the synapses of this update, by neuron: whom it asked, and whether that was granted
        at = r["axon"].long()
        asked = torch.full((case["n"],), -1, dtype=torch.int32, device="cuda").index_put_((at,), r["dendrite"])
        granted = torch.zeros(case["n"], dtype=torch.uint8, device="cuda").index_put_((at,), r["accepted"])
        return dict(asked=asked, granted=granted, steps=r["steps"])
    opt = dict(p=case["p"], m2l=case.get("m2l", "mfma"))
    u = s["batch"].forward(s["w"], s["sigmas"], is_target=s["tg"], out=s["u"], **opt)
    if kind == "batch":
        return u
    s["grads"] = s["batch"].backward(s["w"], s["up"], s["sigmas"], is_target=s["tg"], out=s["grads"], use_graph=True, **opt)
    return dict(u=u, w=s["grads"]["w"], pos=s["grads"]["pos"], sigma=s["grads"]["sigma"])


def work(case):
    """Inputs read once and outputs written once; 2 p^3 flops for every neuron as a source
    and again as a target (6.5 p^3 where the gradient is taken too), 11 per direct pair."""
    kind = case["kind"]
    if kind == "direct":
        nt = min(case["targets"], case["n"])
        return dict(bytes=16.0 * case["n"] + 16.0 * nt, flops=11.0 * case["n"] * nt)
    if "npop" in case:
        q = (np.arange(case["npop"]) + 0.5) / case["npop"]
        n = float(np.sum(np.exp(np.log(case["lo"]) + q * np.log(case["hi"] / case["lo"]))))
    else:
        n = float(case["n"])
    p3 = float(case["p"] ** 3)
    per = dict(sums=21, cached=21, step=21, train=41, batch=21, batch_train=41, descent=29)[kind]
    flops = (4 + (2 * 8.5 if "train" in kind else 0)) * p3 * n
    if kind == "step":
        k = max(64, int(n * QUERIES_PER_NEURON))
        return dict(bytes=per * n + 48.0 * k, flops=flops + 2 * p3 * n)
    return dict(bytes=per * n, flops=flops)


# ---------------------------------------------------------------------------------------
# the same sums in 64 bits
# ---------------------------------------------------------------------------------------
class _Gauss64:
    """Sums over a point set in float64.  On the points' box the kernel exp(-(x-y)^2/sigma^2)
    of each axis is taken as a Chebyshev series in x and in y of so many terms that what is
    left out is at the rounding of float64, so a sum is three small products per point."""

    def __init__(self, xyz, sigma):
        self.sigma = float(sigma)
        self.mid, self.half, self.deg = [], [], []
        for v in xyz:
            lo, hi = float(v.min()), float(v.max())
            self.mid.append(0.5 * (lo + hi)), self.half.append(max(0.5 * (hi - lo), 1e-3 * self.sigma) * (1 + 1e-12))
            self.deg.append(int(13.0 * self.half[-1] / self.sigma) + 34)

    def basis(self, axis, v):
        t = ((v.double() - self.mid[axis]) / self.half[axis]).clamp(-1, 1)
        return torch.cos(torch.acos(t)[:, None] * torch.arange(self.deg[axis], device="cuda", dtype=torch.float64))

    def operator(self, axis, f):
        """Series coefficients in x and y of f(x - y, kernel)."""
        m = self.deg[axis]
        th = (torch.arange(m, device="cuda", dtype=torch.float64) + 0.5) * math.pi / m
        at = torch.cos(th) * self.half[axis]
        d = at[:, None] - at[None, :]
        c = torch.cos(th[None, :] * torch.arange(m, device="cuda", dtype=torch.float64)[:, None]) * (2.0 / m)
        c[0] *= 0.5
        return c @ f(d, torch.exp(-(d / self.sigma) ** 2)) @ c.T

    def _chunks(self, n):
        step = max(1024, (1 << 27) // (self.deg[0] * self.deg[1]))
        return [slice(i, min(n, i + step)) for i in range(0, n, step)]

    def moments(self, xyz, w):
        out = torch.zeros((self.deg[0] * self.deg[1], self.deg[2]), device="cuda", dtype=torch.float64)
        for c in self._chunks(w.numel()):
            bx, by, bz = (self.basis(k, xyz[k][c]) for k in range(3))
            out += (bx[:, :, None] * by[:, None, :]).flatten(1).T @ (bz * w[c].double()[:, None])
        return out

    def fields(self, mom, xyz, which):
        """which: any of "u", "x", "y", "z" (derivative at the target), "s" (by sigma)."""
        s = self.sigma
        plain = lambda d, k: k                                    # noqa: E731
        slope = lambda d, k: -2.0 * d / s ** 2 * k                # noqa: E731
        width = lambda d, k: 2.0 * d * d / s ** 3 * k             # noqa: E731
        terms = dict(u=[(plain,) * 3], x=[(slope, plain, plain)], y=[(plain, slope, plain)], z=[(plain, plain, slope)],
                     s=[(width, plain, plain), (plain, width, plain), (plain, plain, width)])
        m, coef = mom.view(*self.deg), []
        for name in which:
            acc = 0
            for f in terms[name]:
                a, b, c = (self.operator(k, f[k]) for k in range(3))
                r = torch.matmul(a, m.flatten(1)).view(self.deg)
                r = torch.matmul(r.transpose(1, 2).contiguous(), b.T.contiguous()).transpose(1, 2)
                acc = acc + torch.matmul(r.contiguous().view(-1, self.deg[2]), c.T.contiguous())
            coef.append(acc.view(-1, self.deg[2]))
        out = [[] for _ in which]
        for c in self._chunks(xyz[0].numel()):
            bx, by, bz = (self.basis(k, xyz[k][c]) for k in range(3))
            b = (bx[:, :, None] * by[:, None, :]).flatten(1)
            for o, co in zip(out, coef):
                o.append(((b @ co) * bz).sum(1))
        return [torch.cat(o) for o in out]


def _sums64(xyz, w, tg, sigma, exclude_self):
    g = _Gauss64(xyz, sigma)
    u = g.fields(g.moments(xyz, w), xyz, "u")[0]
    return torch.where(tg > 0, u - (w.double() if exclude_self else 0.0), 0.0)


def _grads64(xyz, w, tg, up, sigma, exclude_self):
    """u, then the derivatives of sum up_i u_i by x, y, z, w and sigma."""
    g = _Gauss64(xyz, sigma)
    gt = torch.where(tg > 0, up.double(), 0.0)
    w = w.double()
    u, fx, fy, fz, fs = g.fields(g.moments(xyz, w), xyz, "uxyzs")
    v, hx, hy, hz = g.fields(g.moments(xyz, gt), xyz, "uxyz")
    if exclude_self:
        u, v = u - w, v - gt
    return torch.where(tg > 0, u, 0.0), [gt * f + w * h for f, h in ((fx, hx), (fy, hy), (fz, hz))], v, (gt * fs).sum()


def _probs64(xyz, w, q, sigma):
    """Shares of a node's eight cells in the attraction on the query's target."""
    pos = [v.double()[q["perm"]] for v in xyz]
    ws = w.double()[q["perm"]]
    nq = q["target"].numel()
    t = [v.double()[q["target"].long()] for v in xyz]
    shift = 3 * (20 - q["level"])
    total = torch.zeros(nq * 8, device="cuda", dtype=torch.float64)
    ends = torch.cumsum(q["count"], 0).cpu()
    lo = 0
    while lo < nq:
        base = int(ends[lo - 1]) if lo else 0
        hi = max(lo + 1, int(torch.searchsorted(ends, torch.tensor(base + (1 << 25)), right=True)))
        of = torch.repeat_interleave(torch.arange(lo, hi, device="cuda"), q["count"][lo:hi])
        skip = torch.cumsum(q["count"][lo:hi], 0) - q["count"][lo:hi]
        at = torch.arange(of.numel(), device="cuda") - skip[of - lo] + q["first"][of]
        d2 = sum((p[at] - v[of]) ** 2 for p, v in zip(pos, t))
        total.index_add_(0, of * 8 + ((q["key"][at] >> shift[of]) & 7), ws[at] * torch.exp(-d2 / sigma ** 2))
        lo = hi
    total = total.view(nq, 8)
    return (total / total.sum(1, keepdim=True).clamp(min=1e-300)).flatten()


def exact(case, seed):
    kind = case["kind"]
    if kind == "descent":
        return None      # indices of neurons
    if kind in ("batch", "batch_train"):
        s = _populations(case, seed)
        u, gw, gp, gs = [], [], [[], [], []], []
        for k in range(case["npop"]):
            c = slice(int(s["off"][k]), int(s["off"][k + 1]))
            args = ([v[c] for v in s["xyz"]], s["w"][c], s["tg"][c])
            if kind == "batch":
                u.append(_sums64(*args, s["sigmas"][k], False))
                continue
            r = _grads64(*args, s["up"][c], s["sigmas"][k], False)
            u.append(r[0]), gw.append(r[2]), gs.append(r[3])
            for a, b in zip(gp, r[1]):
                a.append(b)
        if kind == "batch":
            return torch.cat(u)
        return dict(u=torch.cat(u), w=torch.cat(gw), pos=[torch.cat(v) for v in gp], sigma=torch.stack(gs))
    s = _inputs(case, seed)
    if kind == "direct":
        pick = torch.randperm(case["n"], device="cuda", generator=s["gen"])[:min(case["targets"], case["n"])]
        g = _Gauss64(s["xyz"], case["sigma"])
        return g.fields(g.moments(s["xyz"], s["w"]), [v[pick] for v in s["xyz"]], "u")[0]
    if kind == "train":
        u, pos, gw, gs = _grads64(s["xyz"], s["w"], s["tg"], s["up"], case["sigma"], case.get("exclude_self", False))
        return [u] + pos + [gw, gs]
    u = _sums64(s["xyz"], s["w"], s["tg"], case["sigma"], case.get("exclude_self", False))
    if kind != "step":
        return u
    q = _queries(s["xyz"], max(64, int(case["n"] * QUERIES_PER_NEURON)), s["gen"])
    return dict(u=u, probs=_probs64(s["xyz"], s["w"], q, case["sigma"]), choice=None)
