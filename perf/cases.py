"""The work that users of this library time: neighbor-list rebuilds from positions on the GPU.

Every case is what a molecular-dynamics program does at one list update: it
holds positions, a handle from earlier updates and its list buffers, and asks
for the tree and the list again.  The listed sizes, densities, cutoffs and
options are those of the workloads in ``workloads/`` and ``bench.py``; the
inputs are made on the GPU from the seed.

A case has
  path     how the list is asked for: "list" (qbvh_build + nlist_build with a
           kept handle), "noalloc" (nlist_build_noalloc), "batch"
           (nlist_build_many), "paper" (nlist_build_ex in paper mode)
  fluid    "lj", "wca", "spinodal" or "colloid" (two types)
  n        particles (of a batch: of its largest system)
  f64      double-precision positions (path "list")
  systems  systems of a batch
  rho      density of the "lj" and "wca" fluids
"""
import math

import numpy as np
import torch

import paper_1901_08088_amd as Q

DEV = "cuda:0"
SKIN = 0.4
WCA_RC = float(2.0 ** (1.0 / 6.0))


def listed():
    def case(name, path, fluid, n, f64=False, systems=1, rho=0.85):
        return dict(name=name, path=path, fluid=fluid, n=n, f64=f64, systems=systems, rho=rho)

    return [
        # the smallest calls: a small box rebuilt without allocation, where launches and latency count
        case("noalloc_lj_1k", "noalloc", "lj", 1000),
        # the 4000-particle fluid of the plain benchmark leg and of smoke()
        case("list_lj_4k", "list", "lj", 4000),
        # a mid-sized box of a ragged size
        case("list_lj_30k", "list", "lj", 30011),
        # double-precision particle data
        case("list_f64_lj_200k", "list", "lj", 200003, f64=True),
        # ordinary production sizes: the standard fluid, its short-cutoff relative, strongly varying density
        case("list_lj_1m", "list", "lj", 1_000_000),
        case("list_wca_1m", "list", "wca", 1_000_000),
        case("list_spinodal_1m", "list", "spinodal", 1_000_000),
        # two types of very different size and number
        case("list_colloid_1m", "list", "colloid", 1_000_000),
        # the headline size
        case("list_lj_8m", "list", "lj", 8_000_000),
        # an ensemble of independent replicas in one launch sequence
        case("batch_64", "batch", "lj", 50_000, systems=64, rho=0.6),
        # the largest box that fits the fixed workspace comfortably, as inside a captured step
        case("noalloc_lj_500k", "noalloc", "lj", 500_001),
        # the paper's own list semantics on its 10-bit grid
        case("paper_lj_100k", "paper", "lj", 100_000),
    ]


def draw(rng):
    def n_in(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n | 1 if rng.random() < 0.5 else n

    path = rng.choice(["list"] * 6 + ["noalloc"] * 2 + ["batch", "batch", "paper"])
    fluid, f64, systems, rho = "lj", False, 1, 0.85
    if path == "list":
        fluid = rng.choice(["lj", "lj", "wca", "spinodal", "colloid"])
        f64 = fluid in ("lj", "wca") and rng.random() < 0.35
        rho = round(rng.uniform(0.3, 0.9), 3) if fluid in ("lj", "wca") else 0.85
        n = n_in(2000, 3_000_000)
    elif path == "noalloc":
        fluid = rng.choice(["lj", "wca"])
        n = n_in(800, 1_000_000)
    elif path == "batch":
        systems, rho = rng.randint(2, 64), round(rng.uniform(0.3, 0.9), 3)
        n = n_in(2000, 100_000)
    else:
        n = n_in(2000, 300_000)
    return dict(path=path, fluid=fluid, n=n, f64=f64, systems=systems, rho=rho)


# ------------------------------------------------------------------ inputs


def _wrap32(x, L):
    x = torch.remainder(x, L).to(torch.float32)
    return torch.where(x >= float(np.float32(L)), torch.zeros_like(x), x).contiguous()


def _edge(volume):
    return float(np.float32(volume ** (1.0 / 3.0)))  # the box is an fp32 value


def _sites(side, which, spacing):
    x = torch.stack((which % side, (which // side) % side, which // (side * side)), 1)
    return (x.to(torch.float64) + 0.5) * spacing


def _lattice(g, n, L, jitter=0.3):
    """n sites of a simple-cubic lattice in random order, each coordinate jittered: an unsorted liquid snapshot."""
    side = int(math.ceil(n ** (1.0 / 3.0) - 1e-9))
    which = torch.randperm(side ** 3, generator=g, device=DEV)[:n]
    u = torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64)
    return _sites(side, which, L / side) + (2.0 * u - 1.0) * jitter


def _spinodal(g, n):
    """Two interpenetrating halves, a liquid at density 0.75 and a vapor at 0.05, split by a smooth random field."""
    L = _edge(n / 0.4)
    kmax = max(1, round(L / 30.0))
    k = torch.randint(-kmax, kmax + 1, (24, 3), generator=g, device=DEV).to(torch.float64)
    k[:, 0] += (k.abs().sum(1) == 0).to(torch.float64)
    phase = torch.rand(24, generator=g, device=DEV, dtype=torch.float64) * (2 * math.pi)

    def field(x):
        f = torch.zeros(x.shape[0], device=DEV, dtype=torch.float64)
        for m in range(24):
            f += torch.cos((x @ k[m]) * (2 * math.pi / L) + phase[m])
        return f

    level = field(torch.rand((200_000, 3), generator=g, device=DEV, dtype=torch.float64) * L).median()
    side = max(1, round(L * 0.75 ** (1.0 / 3.0)))
    x = _sites(side, torch.arange(side ** 3, device=DEV), L / side)
    x = x[field(x) > level]
    m = int(round(n / 16.0))  # vapor: half the volume at 0.05
    x = x[torch.randperm(x.shape[0], generator=g, device=DEV)[: n - m]]
    x = x + (2.0 * torch.rand(x.shape, generator=g, device=DEV, dtype=torch.float64) - 1.0) * 0.3
    m = n - x.shape[0]
    v = torch.rand((4 * m + 1000, 3), generator=g, device=DEV, dtype=torch.float64) * L
    v = v[field(v) <= level][:m]
    x = torch.cat((x, v))
    return _wrap32(x[torch.randperm(n, generator=g, device=DEV)], L), L


def _colloid(g, n):
    """2% colloids of diameter 5 (type 1) among solvent of diameter 1 at density 0.5 in the volume it can reach."""
    nc = max(1, int(round(0.02 * n)))
    L = _edge((n - nc) / 0.5 + nc * (4.0 / 3.0) * math.pi * 27.0)
    side = int(math.ceil(nc ** (1.0 / 3.0) - 1e-9))
    a = L / side
    taken = torch.randperm(side ** 3, generator=g, device=DEV)[:nc]
    centre = torch.full((side ** 3, 3), 1e9, device=DEV, dtype=torch.float64)
    jit = max(0.0, min(1.0, (a - 5.0) / 2.0))
    centre[taken] = _sites(side, taken, a) + (2.0 * torch.rand((nc, 3), generator=g, device=DEV, dtype=torch.float64) - 1.0) * jit
    fine = int(L)
    x = _sites(fine, torch.arange(fine ** 3, device=DEV), L / fine)
    c = torch.clamp((x / a).long(), max=side - 1)
    free = torch.ones(x.shape[0], device=DEV, dtype=torch.bool)
    for k in range(27):
        d = torch.remainder(c + torch.tensor([k % 3 - 1, k // 3 % 3 - 1, k // 9 - 1], device=DEV), side)
        d = x - centre[(d[:, 2] * side + d[:, 1]) * side + d[:, 0]]
        d -= L * torch.round(d / L) * (d.abs() < 1e6)
        free &= d.square().sum(1) >= 9.0
    x = x[free]
    x = x[torch.randperm(x.shape[0], generator=g, device=DEV)[: n - nc]]
    x = x + (2.0 * torch.rand(x.shape, generator=g, device=DEV, dtype=torch.float64) - 1.0) * 0.2
    v = torch.rand((n - nc - x.shape[0], 3), generator=g, device=DEV, dtype=torch.float64) * L
    types = torch.zeros(n, dtype=torch.int32, device=DEV)
    types[n - nc:] = 1
    order = torch.randperm(n, generator=g, device=DEV)
    return _wrap32(torch.cat((x, v, centre[taken]))[order], L), types[order].contiguous(), L


def _particles(g, case, n):
    """Positions, types and box edge of one system."""
    fluid = case["fluid"]
    if fluid == "colloid":
        return _colloid(g, n)
    if fluid == "spinodal":
        pos, L = _spinodal(g, n)
        return pos, None, L
    L = _edge(n / case["rho"])
    x = _lattice(g, n, L)
    if case["f64"]:
        x = torch.remainder(x, L)
        return torch.where(x >= L, torch.zeros_like(x), x).contiguous(), None, L
    return _wrap32(x, L), None, L


def _sizes(case):
    """Sizes of the systems: log-spaced up to n in a batch."""
    k, hi = case["systems"], case["n"]
    if case["path"] != "batch":
        return [hi]
    lo = min(hi, 2000)
    return [int(round(lo * (hi / lo) ** ((i + 1) / k))) for i in range(k)]


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    sizes = _sizes(case)
    total, width = sum(sizes), 64 if case["fluid"] == "wca" else 256
    # one buffer each for the lists, counts and flags of all systems
    out = dict(nbr=torch.full((total, width), -1, dtype=torch.int32, device=DEV),
               count=torch.zeros(total, dtype=torch.int32, device=DEV),
               overflow=torch.zeros(len(sizes), dtype=torch.int32, device=DEV))
    colloid = case["fluid"] == "colloid"
    rcut = [[1.0, 3.0], [3.0, 5.0]] if colloid else [[WCA_RC]] if case["fluid"] == "wca" else [[3.0]]
    systems, at = [], 0
    for i, n in enumerate(sizes):
        pos, types, L = _particles(g, case, n)
        systems.append(dict(pos=pos, types=types, ntypes=2 if colloid else 1, box=[L, L, L], rcut=rcut, skin=SKIN,
                            max_nbr=width, nbr=out["nbr"][at:at + n], count=out["count"][at:at + n],
                            overflow=out["overflow"][i:i + 1]))
        at += n
    return dict(path=case["path"], systems=systems, out=out, tree=Q.Tree())


# Options that a program fixes once it has tuned them (the defaults of the plain path).
BATCH_OPTS = dict(leaf_size=16, qbits=16, block_size=64)


def run(state):
    path, systems = state["path"], state["systems"]
    s = systems[0]
    if path == "batch":
        Q.nlist_build_many(systems, opts=BATCH_OPTS)
    elif path == "noalloc":
        Q.nlist_build_noalloc(s["pos"], s["types"], s["box"], s["ntypes"], s["rcut"], s["skin"], s["max_nbr"],
                              s["nbr"], s["count"], s["overflow"])
    elif path == "paper":
        tree = Q.qbvh_build(s["pos"], s["types"], s["box"], s["ntypes"], opts=dict(qbits=10), tree=state["tree"])
        Q.nlist_build_ex(tree, s["rcut"], s["skin"], s["max_nbr"], Q.LIST_PAPER, s["nbr"], s["count"], s["overflow"])
    else:
        tree = Q.qbvh_build(s["pos"], s["types"], s["box"], s["ntypes"], tree=state["tree"])
        Q.nlist_build(tree, s["rcut"], s["skin"], s["max_nbr"], s["nbr"], s["count"], s["overflow"])
    return state["out"]


# ------------------------------------------------------------------ what a pass cannot do without


def _per_particle(case):
    """Expected list entries per particle."""
    if case["fluid"] == "colloid":
        return 4.2
    if case["fluid"] == "spinodal":
        return 108.0
    r = (WCA_RC if case["fluid"] == "wca" else 3.0) + SKIN
    return case["rho"] * (4.0 / 3.0) * math.pi * r ** 3


def work(case):
    n = sum(_sizes(case))
    m = _per_particle(case)
    read = 24 if case["f64"] else 16 if case["fluid"] == "colloid" else 12
    # positions (and types) read once, counts and stored entries written once; one distance per listed pair
    return {"bytes": n * (read + 4.0 + 4.0 * m), "flops": 8.0 * n * m}


def _counts(pos, types, box, rcut):
    """True counts by brute force in fp64 with the minimum image."""
    x = pos.to(torch.float64)
    L = torch.tensor(box, dtype=torch.float64, device=x.device)
    r = torch.tensor(np.asarray(rcut, dtype=np.float32).astype(np.float64) + float(np.float32(SKIN)), device=x.device)
    t = types.long() if types is not None else torch.zeros(x.shape[0], dtype=torch.long, device=x.device)
    out = []
    for lo in range(0, x.shape[0], 256):
        d2 = 0.0
        for k in range(3):
            d = x[None, :, k] - x[lo:lo + 256, None, k]
            d = d - L[k] * torch.round(d / L[k])
            d2 = d2 + d * d
        out.append((d2 <= r[t[lo:lo + 256]][:, t].square()).sum(1) - 1)
    return torch.cat(out).to(torch.int32)


def exact(case, seed):
    """Counts and overflow flag of the single-system paths; the order of a row's entries is not defined by value."""
    if case["path"] not in ("list", "noalloc") or case["n"] > 40_000:
        return None
    s = prepare(case, seed)["systems"][0]
    c = _counts(s["pos"], s["types"], s["box"], s["rcut"])
    return dict(nbr=None, count=c, overflow=(c > s["max_nbr"]).any().to(torch.int32).reshape(1))
