"""The work that performance is measured on: whole calls of the public entry
points over the sizes, dimensions and options that programs use them with.

A case is a dict of plain values:

  call    build     emst.build of one cloud
          noalloc   Context.build_noalloc (static workspace, preallocated outputs)
          batched   Context.build_batched of a list of clouds
          solver    Solver: admit every request, step until all are done, take_many
          mreach    Context.build_mreach (MST under mutual reachability, k_pts = k)
          core      Context.core_distances (k_pts = k)
  cloud   uniform | clustered | mixture | cosmology | skewed: the point
          distributions of the package's workloads, drawn on the GPU
  n, dim  points and dimension of one cloud
  k       neighbours of the mutual reachability calls
  count, lo, hi, median, sizes    batches and request streams: number of
          clouds and the spread of their sizes (log-uniform in [lo, hi], or
          lognormal around `median` clipped to [lo, hi]), drawn from `sizes`

Points are independent draws, so input indices carry no spatial order.
"""
import math
import random

import torch

import paper_2207_00514_amd as emst

DEV = "cuda:0"


# ----------------------------------------------------------------------------
# clouds

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)


def _uniform(g, n, dim):
    return _rand(g, n, dim).float()


def _clustered(g, n, dim):
    """90 % of the points in 200 Gaussians of widths 0.002 .. 0.02, the rest uniform."""
    centres = _rand(g, 200, dim)
    sigma = torch.exp(math.log(0.002) + (math.log(0.02) - math.log(0.002)) * _rand(g, 200))
    owner = torch.randint(200, (n,), generator=g, device=DEV)
    pts = centres[owner] + sigma[owner, None] * _randn(g, n, dim)
    back = _rand(g, n) < 0.10
    return torch.where(back[:, None], _rand(g, n, dim), pts).float()


def _mixture(g, n, dim):
    """20 Gaussians of width 0.01 (half of the serving requests and batch clouds)."""
    centres = _rand(g, 20, dim)
    owner = torch.randint(20, (n,), generator=g, device=DEV)
    return (centres[owner] + 0.01 * _randn(g, n, dim)).float()


def _cosmology(g, n, dim):
    """60 % of the points in Plummer halos with power-law member counts, the
    rest uniform, in a periodic box of side 64; made in pieces."""
    box, halos = 64.0, max(1, min(50_000, int(0.6 * n) // 20))
    members = 20.0 * _rand(g, halos).clamp_min(1e-9) ** (-1.0 / 0.9)
    members = members.clamp_max(0.1 * 0.6 * n)
    members = members * (0.6 * n / members.sum())
    centres = _rand(g, halos, dim) * box
    scale = 0.0005 * members.clamp_min(20.0) ** (1.0 / 3.0)
    # integer cumulative weights: the same owners whatever the order of the sum
    ends = torch.cumsum((members * 1024.0).to(torch.int64).clamp_min(1), 0)
    out = torch.empty(n, dim, device=DEV)
    for at in range(0, n, 1 << 22):
        m = min(1 << 22, n - at)
        owner = torch.searchsorted(ends, (_rand(g, m) * ends[-1].double()).to(torch.int64), right=True)
        owner = owner.clamp_max(halos - 1)
        u = _rand(g, m).clamp(1e-12, 1.0 - 1e-12)
        r = scale[owner] / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
        v = _randn(g, m, dim)
        v = v / torch.linalg.vector_norm(v, dim=1, keepdim=True)
        p = torch.remainder(centres[owner] + r[:, None] * v, box)
        field = _rand(g, m) < 0.4
        p = torch.where(field[:, None], _rand(g, m, dim) * box, p).float()
        out[at:at + m] = torch.where(p >= box, torch.zeros_like(p), p)
    return out


def _skewed(g, n, dim):
    """Random walks (1000 of them, step 1e-6) that start in a cube of side
    1e-3, and one point in a thousand uniform in a cube of side 1000."""
    walks = min(1000, max(1, n // 8))
    per = -(-n // walks)
    steps = torch.round(1e-6 * _randn(g, walks, per, dim) * 2.0 ** 50).to(torch.int64)
    walk = torch.cumsum(steps, 1).double() * 2.0 ** -50  # integer sums: exact in any order
    pts = (0.5 + 1e-3 * _rand(g, walks, 1, dim) + walk).reshape(-1, dim)
    pts = pts[torch.argsort(_rand(g, walks * per), stable=True)][:n]
    far = _rand(g, n) < 0.001
    return torch.where(far[:, None], 1000.0 * _rand(g, n, dim), pts).float()


CLOUDS = {"uniform": _uniform, "clustered": _clustered, "mixture": _mixture, "cosmology": _cosmology,
          "skewed": _skewed}


def _sizes(case):
    r = random.Random(int(case["sizes"]))
    lo, hi, out = case["lo"], case["hi"], []
    for _ in range(case["count"]):
        if "median" in case:
            x = case["median"] * math.exp(1.2 * r.gauss(0.0, 1.0))
        else:
            x = math.exp(r.uniform(math.log(lo), math.log(hi)))
        out.append(int(min(max(x, lo), hi)))
    return out


def _clouds(case, seed):
    """The clouds of a call.  Batches alternate 2D uniform clouds and 3D
    mixtures; requests are 3D, uniform or mixtures."""
    g = _gen(seed)
    if "count" not in case:
        return [CLOUDS[case["cloud"]](g, case["n"], case["dim"]).contiguous()]
    out = []
    for c, n in enumerate(_sizes(case)):
        if c % 2:
            out.append(_mixture(g, n, 3))
        else:
            out.append(_uniform(g, n, 2 if case["call"] == "batched" else 3))
    return out


# ----------------------------------------------------------------------------
# cases

def listed():
    return [
        # the smallest clouds of the size sweep: a call made of launches and latencies
        dict(name="uniform2d_1k", call="build", cloud="uniform", n=1_000, dim=2),
        # the small 2D workload
        dict(name="uniform2d_10k", call="build", cloud="uniform", n=10_000, dim=2),
        # one serving request of median size, solved without an allocation, an odd size
        dict(name="request3d_50k", call="noalloc", cloud="mixture", n=50_021, dim=3),
        # below the size from which query lists are made
        dict(name="clustered3d_300k", call="build", cloud="clustered", n=299_993, dim=3),
        # the clustered 3D workload
        dict(name="clustered3d_2m", call="build", cloud="clustered", n=2_000_000, dim=3),
        # extreme density contrast: the rank-space rebuild of the tree
        dict(name="skewed3d_2m", call="build", cloud="skewed", n=2_000_000, dim=3),
        # a large 2D cloud, an odd size
        dict(name="uniform2d_5m", call="build", cloud="uniform", n=4_999_999, dim=2),
        # the headline workload: the largest cloud measured as a whole
        dict(name="cosmology3d_37m", call="build", cloud="cosmology", n=37_000_000, dim=3),
        # many small clouds of both dimensions in one pass
        dict(name="batched512", call="batched", count=512, lo=1_000, hi=200_000, sizes=4),
        # a burst of serving requests through the round-granular solver
        dict(name="solver_burst24", call="solver", count=24, lo=5_000, hi=400_000, median=50_000, sizes=5),
        # mutual reachability at a clustering's usual neighbourhood
        dict(name="mreach3d_2m_k8", call="mreach", cloud="clustered", n=2_000_000, dim=3, k=8),
        # core distances alone, a larger neighbourhood
        dict(name="core3d_100k_k16", call="core", cloud="clustered", n=100_003, dim=3, k=16),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["build", "noalloc", "batched", "solver", "mreach", "core"], [10, 2, 2, 2, 2, 1])[0]
    dim = rng.choice([2, 3])
    if kind == "build":
        cloud = rng.choice(["uniform", "clustered", "clustered", "mixture", "cosmology", "skewed"])
        hi = {"cosmology": 30_000_000, "skewed": 4_000_000}.get(cloud, 20_000_000)
        return dict(call="build", cloud=cloud, n=_logint(rng, 1_000, hi), dim=3 if cloud == "cosmology" else dim)
    if kind == "noalloc":
        return dict(call="noalloc", cloud=rng.choice(["uniform", "clustered", "mixture"]),
                    n=_logint(rng, 1_000, 270_000), dim=dim)
    if kind == "batched":
        return dict(call="batched", count=_logint(rng, 8, 400), lo=1_000, hi=_logint(rng, 10_000, 200_000),
                    sizes=rng.randrange(1 << 30))
    if kind == "solver":
        return dict(call="solver", count=_logint(rng, 4, 48), lo=5_000, hi=_logint(rng, 100_000, 1_000_000),
                    median=50_000, sizes=rng.randrange(1 << 30))
    if kind == "mreach":
        return dict(call="mreach", cloud=rng.choice(["uniform", "clustered", "mixture"]),
                    n=_logint(rng, 2_000, 4_000_000), dim=dim, k=rng.choice([2, 4, 5, 8, 10, 16]))
    return dict(call="core", cloud=rng.choice(["uniform", "clustered", "mixture"]),
                n=_logint(rng, 2_000, 2_000_000), dim=dim, k=rng.choice([2, 4, 5, 8, 10, 16, 30]))


# ----------------------------------------------------------------------------
# what a program holds, and one pass

def prepare(case, seed):
    clouds = _clouds(case, seed)
    state = dict(call=case["call"], clouds=clouds, ctx=emst.context(0), k=case.get("k", 0))
    if case["call"] == "noalloc":
        m = clouds[0].shape[0] - 1
        state["out"] = (torch.empty((m, 2), dtype=torch.int32, device=DEV), torch.empty(m, device=DEV),
                        torch.empty(m, device=DEV))
    if case["call"] == "solver":
        budget = sum(emst.Solver.slot_bytes(c.shape[0], c.shape[1]) for c in clouds) * 5 // 4
        state["solver"] = emst.Solver(state["ctx"], budget, max_slots=max(64, len(clouds)))
    return state


def run(state):
    call, clouds, ctx = state["call"], state["clouds"], state["ctx"]
    if call == "build":
        edges, weights, d2 = emst.build(clouds[0])
        return {"edges": edges, "weights": weights, "d2": d2}
    if call == "noalloc":
        edges, weights, d2 = ctx.build_noalloc(clouds[0], out=state["out"])
        return {"edges": edges, "weights": weights, "d2": d2}
    if call == "batched":
        # (the results of one batch are views of shared outputs, back to back)
        res = ctx.build_batched(clouds)
        m = sum(max(c.shape[0] - 1, 0) for c in clouds)
        e, w, d = (x._base if x._base is not None else x for x in res[0])
        return {"edges": e[:m], "weights": w[:m], "d2": d[:m]}
    if call == "solver":
        sv = state["solver"]
        slots = [sv.admit(c) for c in clouds]
        waiting = len(slots)
        while waiting > 0:
            waiting -= sv.step()
        edges, weights, d2, offsets = sv.take_many(slots)
        return {"edges": edges, "weights": weights, "d2": d2}
    if call == "mreach":
        edges, weights, m2, core2 = ctx.build_mreach(clouds[0], state["k"])
        return {"edges": edges, "weights": weights, "d2": m2, "core2": core2}
    return {"core2": ctx.core_distances(clouds[0], state["k"])}


def work(case):
    """Points in once, results out once; one squared distance an edge."""
    if "count" in case:
        sizes = _sizes(case)
        dims = [3 if c % 2 or case["call"] == "solver" else 2 for c in range(len(sizes))]
    else:
        sizes, dims = [case["n"]], [case["dim"]]
    read = sum(4 * n * d for n, d in zip(sizes, dims))
    edges = sum(n - 1 for n in sizes)
    if case["call"] == "core":
        return {"bytes": read + 4 * sizes[0], "flops": (3 * dims[0] - 1) * case["k"] * sizes[0]}
    extra = 4 * sizes[0] if case["call"] == "mreach" else 0
    flops = sum((3 * d - 1) * (n - 1) for n, d in zip(sizes, dims))
    if case["call"] == "mreach":
        flops += (3 * dims[0] - 1) * case["k"] * sizes[0]
    return {"bytes": read + 16 * edges + extra, "flops": flops}


# ----------------------------------------------------------------------------
# the same values in 64 bits, by brute force over all pairs

_DENSE = 101_000  # points up to which all pairs are searched


def _pairs(x, a, b):
    d = (x[a:b, 0, None] - x[None, :, 0]) ** 2
    for k in range(1, x.shape[1]):
        d += (x[a:b, k, None] - x[None, :, k]) ** 2
    return d


def _core64(x, k):
    n, out = x.shape[0], []
    step = max(1, (1 << 27) // n)
    for a in range(0, n, step):
        out.append(torch.topk(_pairs(x, a, min(a + step, n)), k, dim=1, largest=False).values[:, k - 1])
    return torch.cat(out)


def _mst64(x, core=None):
    """Squared lengths of a minimum spanning tree, ascending (Boruvka over
    all pairs; the rounds' edges join through a union-find, so equal lengths
    make no cycle)."""
    n = x.shape[0]
    comp = torch.arange(n, device=x.device)
    parent, lengths = list(range(n)), []

    def find(a):
        while parent[a] != a:
            parent[a] = parent[parent[a]]
            a = parent[a]
        return a

    step = max(1, (1 << 27) // n)
    while len(lengths) < n - 1:
        best, arg = [], []
        for a in range(0, n, step):
            b = min(a + step, n)
            d = _pairs(x, a, b)
            if core is not None:
                d = torch.maximum(d, torch.maximum(core[a:b, None], core[None, :]))
            d.masked_fill_(comp[a:b, None] == comp[None, :], math.inf)
            v, j = d.min(dim=1)
            best.append(v)
            arg.append(j)
        best, arg = torch.cat(best), torch.cat(arg)
        low = torch.full((n,), math.inf, dtype=torch.float64, device=x.device)
        low.scatter_reduce_(0, comp, best, "amin")
        hit = torch.nonzero((best == low[comp]) & torch.isfinite(best)).flatten()
        w, u, v = best[hit].cpu(), hit.cpu(), arg[hit].cpu()
        order = torch.argsort(w, stable=True)
        for d, a, b in zip(w[order].tolist(), u[order].tolist(), v[order].tolist()):
            ra, rb = find(a), find(b)
            if ra != rb:
                parent[max(ra, rb)] = min(ra, rb)
                lengths.append(d)
        comp = torch.tensor([find(a) for a in range(n)], device=x.device)
    return torch.sort(torch.tensor(lengths, dtype=torch.float64))[0]


def exact(case, seed):
    sizes = _sizes(case) if "count" in case else [case["n"]]
    if sum(n * n for n in sizes) > _DENSE * _DENSE:
        return None
    clouds = [c.double() for c in _clouds(case, seed)]
    if case["call"] == "core":
        return {"core2": _core64(clouds[0], case["k"])}
    core = _core64(clouds[0], case["k"]) if case["call"] == "mreach" else None
    d2 = torch.cat([_mst64(c, core) for c in clouds])
    out = {"edges": None, "weights": torch.sqrt(d2), "d2": d2}
    if core is not None:
        out["core2"] = core
    return out
