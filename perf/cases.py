"""The work a user of this library has it do, as cases that can be timed.

Every case goes through the public entry points of
``paper_2209_13121_amd.binding``.  Three kinds of position sets: points
uniform in a cube (uniform octree), three-site clusters with a lumpy density
(adaptive octree), and batches of independent systems (adaptive octree, one
system per box of a level).  Kinds of call:

  * ``step``     : a time step of a simulation: ``fmm_replan`` for the current
                   positions, then ``fmm_evaluate`` (potentials, forces, energy).
  * ``evaluate`` : new charges on fixed positions (one plan kept): an iteration
                   of a charge solver.
  * ``static``   : ``fmm_evaluate_static``, plan and evaluation in one call
                   without allocations, positions new on every call (serving).
  * ``grad``     : the energy and its gradients in positions and charges through
                   ``torch.autograd`` (``fmm_energy`` forward and backward).

Precision: FP64 is the library's default; a program that asks for the mixed
mode keeps its own state in FP32, so it passes FP32 tensors to ``fmm_energy``
and rounds what the other calls write (always FP64 buffers) to FP32.

The sizes 4096 / 2^19 / 2^20 / 3e6 sites / 256 systems and their depths,
orders and leaf capacities are those of ``paper_2209_13121_amd/workloads.py``;
the others are generic.
"""
import math
import random

import torch

from paper_2209_13121_amd import binding as B

DEV = "cuda"
CHARGES = (-0.834, 0.417, 0.417)  # a three-site cluster
BOND, ANGLE = 0.0957, math.radians(104.5)


def listed():
    return [
        # the smallest call in ordinary use: a few thousand charges, where launches and latency count
        _case("step-4096-d3-p4-fp64", "uniform", "step", 4096, 3, 4, "fp64"),
        # a serving call on a small odd-sized set: tree, operators and evaluation each time
        _case("static-10007-d3-p6-mixed", "uniform", "static", 10007, 3, 6, "mixed"),
        # an ordinary simulation step of odd size, the cube derived from the positions
        _case("step-100003-d4-p6-mixed", "uniform", "step", 100003, 4, 6, "mixed", derived=True),
        # an iterative solver at high order: new charges, the same positions
        _case("evaluate-200001-d5-p12-fp64", "uniform", "evaluate", 200001, 5, 12, "fp64"),
        # an FP64 step with ordinary leaves (64 charges each)
        _case("step-262144-d4-p8-fp64", "uniform", "step", 1 << 18, 4, 8, "fp64"),
        # the step of the benchmark, in both precisions: many small leaves, the far field dominates
        _case("step-1048576-d6-p8-mixed", "uniform", "step", 1 << 20, 6, 8, "mixed"),
        _case("step-1048576-d6-p8-fp64", "uniform", "step", 1 << 20, 6, 8, "fp64"),
        # large leaves (256 charges each): the near field dominates
        _case("step-1048576-d4-p8-mixed", "uniform", "step", 1 << 20, 4, 8, "mixed"),
        # training: energy and gradients of FP32 tensors, the largest set the differentiation is tested on
        _case("grad-524288-d6-p8-mixed", "uniform", "grad", 1 << 19, 6, 8, "mixed"),
        # molecular clusters on the adaptive tree at order 10: the largest system, and a tenth of it in FP64
        _case("clusters-3000000-p10-mixed", "clusters", "step", 3000000, 7, 10, "mixed", leaf_max=64),
        _case("clusters-300000-p10-fp64", "clusters", "step", 300000, 6, 10, "fp64", leaf_max=64),
        # 256 independent systems of 1e3 .. 2^16 charges in one plan
        _case("batch-256-p6-mixed", "batch", "step", 256, 7, 6, "mixed", leaf_max=64, batch_level=3),
    ]


def _case(name, points, call, n, depth, p, precision, leaf_max=0, batch_level=0, derived=False):
    c = {"points": points, "call": call, "n": n, "depth": depth, "p": p, "precision": precision,
         "leaf_max": leaf_max, "batch_level": batch_level, "derived": derived}
    if name:
        c["name"] = name
    return c


def draw(rng):
    """One more case: sizes over their logarithm, every call, both precisions."""
    points = rng.choice(["uniform"] * 7 + ["clusters"] * 2 + ["batch"])
    precision = rng.choice(["fp64", "mixed"])
    fp64 = precision == "fp64"
    if points == "clusters":
        sites = 3 * round(math.exp(rng.uniform(math.log(2e3), math.log(1e5 if fp64 else 1e6))))
        p = rng.choice([4, 6, 8, 10])
        leaf = rng.choice([24, 32, 48, 64, 100, 128])
        depth = min(7, max(4, math.ceil(math.log(12.0 * sites / leaf) / math.log(8.0)) + 1))
        return _case("", points, "step", sites, depth, p, precision, leaf_max=leaf)
    if points == "batch":
        systems = round(math.exp(rng.uniform(math.log(4), math.log(64 if fp64 else 256))))
        return _case("", points, "step", systems, 7, rng.choice([4, 6, 8]), precision,
                     leaf_max=rng.choice([32, 64, 96, 128]), batch_level=3)
    call = rng.choice(["step", "step", "step", "evaluate", "grad", "static"])
    p = rng.choice([3, 4, 5, 6, 7, 8] if call == "static" else [3, 4, 5, 6, 7, 8, 8, 10, 12])  # static: 128 MiB
    top = {"static": 1 << 17, "grad": 1 << 19}.get(call, 1 << 20)
    n = round(math.exp(rng.uniform(math.log(1000), math.log(top))))
    # 4 .. 256 charges a leaf on average, and no more work than the largest listed cases
    fill = math.exp(rng.uniform(math.log(4.0), math.log(256.0)))
    depth = max(2, round(math.log(n / fill) / math.log(8.0)))
    depth = min(depth, 4 if call == "static" else 6)
    while 8 ** depth * (p + 1) ** 4 > 8 ** 6 * 9 ** 4:
        depth -= 1
    while n * (n / 8 ** depth) > (1 << 20) * 257 * (0.5 if fp64 else 1.0) and depth < 4:
        depth += 1
    return _case("", points, call, n, depth, p, precision,
                 derived=call == "step" and rng.random() < 0.3)


# ---- inputs --------------------------------------------------------------

def _uniform(n, gen):
    pos = torch.rand((n, 3), generator=gen, device=DEV, dtype=torch.float64)
    q = torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
    return pos, q - q.mean()


def _clusters(sites, gen):
    """Three-site clusters, first sites by rejection from 1 + 3 exp(-d^2 / 2
    sigma^2) over 16 blob centres (sigma a sixteenth of the side), about 100
    sites per unit volume, random orientations; shape and charges of
    ``workloads.molecular_clusters``."""
    k = sites // 3
    rand = lambda *s: torch.rand(s, generator=gen, device=DEV, dtype=torch.float64)  # noqa: E731
    centres = rand(16, 3)
    dens = lambda x: 1 + 3 * torch.exp(-128.0 * (  # noqa: E731
        (x[:, None, :] - centres).square().sum(dim=2).min(dim=1).values))
    side = (3.0 * k / (100.0 * float(dens(rand(200000, 3)).mean()))) ** (1.0 / 3.0)
    first = torch.empty((0, 3), device=DEV, dtype=torch.float64)
    while first.shape[0] < k:
        cand = rand(max(1024, 2 * (k - first.shape[0])), 3)
        first = torch.cat([first, cand[4.0 * rand(cand.shape[0]) < dens(cand)]])
    first = first[:k] * side
    u = torch.randn((k, 3), generator=gen, device=DEV, dtype=torch.float64)
    v = torch.randn((k, 3), generator=gen, device=DEV, dtype=torch.float64)
    u = u / u.norm(dim=1, keepdim=True)
    v = v - (u * v).sum(dim=1, keepdim=True) * u
    v = v / v.norm(dim=1, keepdim=True)
    a, b = BOND * math.sin(ANGLE / 2), BOND * math.cos(ANGLE / 2)
    pos = torch.stack([first, first + a * u + b * v, first - a * u + b * v], dim=1)
    q = torch.tensor(CHARGES, device=DEV, dtype=torch.float64).repeat(k)
    return pos.reshape(-1, 3).contiguous(), q


def _counts(systems):
    """Even system sizes, log-uniform over 1e3 .. 2^16; the same for every seed."""
    rng = random.Random(1005 * systems)
    c = [round(math.exp(rng.uniform(math.log(1000), math.log(65536)))) for _ in range(systems)]
    return [m + m % 2 for m in c]


def _batch(systems, gen):
    """Systems of 1e3 .. 2^16 charges +-1 (net zero), each uniform in its own
    cell of an 8^3 grid."""
    counts = _counts(systems)
    pos, q = [], []
    for k, m in enumerate(counts):
        cell = torch.tensor([k % 8, (k // 8) % 8, k // 64], device=DEV, dtype=torch.float64)
        pos.append(cell + torch.rand((m, 3), generator=gen, device=DEV, dtype=torch.float64))
        s = torch.ones(m, device=DEV, dtype=torch.float64)
        s[torch.randperm(m, generator=gen, device=DEV)[: m // 2]] = -1.0
        q.append(s)
    return torch.cat(pos), torch.cat(q), counts


def _inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 17)
    if case["points"] == "clusters":
        return (*_clusters(case["n"], gen), None)
    if case["points"] == "batch":
        return _batch(case["n"], gen)
    return (*_uniform(case["n"], gen), None)


def _cube(case):
    """(lo, side) handed to the library; side 0 asks for the derived cube."""
    if case["points"] == "batch":
        return (0.0, 0.0, 0.0), 8.0
    return (0.0, 0.0, 0.0), 0.0 if case["derived"] or case["points"] == "clusters" else 1.0


def prepare(case, seed):
    pos, q, _ = _inputs(case, seed)
    mixed = case["precision"] == "mixed"
    prec = B.FMM_PREC_MIXED if mixed else B.FMM_PREC_FP64
    lo, side = _cube(case)
    n = pos.shape[0]
    s = {"call": case["call"], "mixed": mixed, "n": n}
    if case["call"] == "grad":
        dt = torch.float32 if mixed else torch.float64
        s.update(pos=pos.to(dt).requires_grad_(), q=q.to(dt).requires_grad_(), p=case["p"],
                 depth=case["depth"], precision=prec)
        return s
    s.update(pos=pos, q=q, phi=torch.empty_like(q), force=torch.empty_like(pos),
             energy=torch.empty(1, device=DEV, dtype=torch.float64))
    if case["call"] == "static":
        s["cfg"] = B.make_config(p=case["p"], depth=case["depth"], precision=prec, lo=lo, side=side)
    else:
        s["fmm"] = B.FMM(pos, p=case["p"], depth=case["depth"], precision=prec, lo=lo, side=side,
                         leaf_max=case["leaf_max"], batch_level=case["batch_level"])
    return s


def run(s):
    if s["call"] == "grad":
        e = B.fmm_energy(s["pos"], s["q"], p=s["p"], depth=s["depth"], precision=s["precision"])
        dx, dq = torch.autograd.grad(e, (s["pos"], s["q"]))
        return {"energy": e.detach(), "dx": dx, "dq": dq}
    if s["call"] == "static":
        B.fmm_evaluate_static(s["cfg"], s["n"], s["pos"], s["q"], s["phi"], s["force"], s["energy"])
    else:
        if s["call"] == "step":
            B.fmm_replan(s["fmm"].plan, s["pos"])
        B.fmm_evaluate(s["fmm"].plan, s["q"], s["phi"], s["force"], s["energy"])
    out = {"phi": s["phi"], "force": s["force"], "energy": s["energy"]}
    return {k: v.float() for k, v in out.items()} if s["mixed"] else out


# ---- what a pass cannot do without ----------------------------------------

def _tree_work(n, depth, p):
    """(M2L flop, P2P flop) of n uniform charges on a uniform tree: an M2L pair
    by rotation, axial shift and rotation back (two rotations of
    sum (2 n + 1)^2 products, a shift of sum (p + 1 - m)^2 per +-m), a P2P
    pair of particles 19 flop."""
    near = lambda l: (3 * 2 ** l - 2) ** 3  # noqa: E731  ordered pairs of adjacent boxes
    pairs = sum(64 * near(l - 1) - near(l) for l in range(2, depth + 1))
    rot = (p + 1) * (2 * p + 1) * (2 * p + 3) // 3
    shift = 2 * sum((p + 1 - m) ** 2 for m in range(1, p + 1)) + (p + 1) ** 2
    return pairs * 2 * (2 * rot + shift), near(depth) * (n / 8 ** depth) ** 2 * 19


def work(case):
    n, depth, p = case["n"], case["depth"], case["p"]
    systems = 1
    if case["points"] == "batch":
        systems, n = n, sum(_counts(n)) / n
    if case["leaf_max"]:
        depth = max(2, round(math.log(n / (0.4 * case["leaf_max"])) / math.log(8.0)))
    m2l, p2p = _tree_work(n, depth, p)
    flops = systems * (m2l + p2p)
    word = 4 if case["call"] == "grad" and case["precision"] == "mixed" else 8
    # positions and charges read, potentials and forces (or gradients) written
    return {"bytes": float(systems * n * 8 * word), "flops": float(flops * (2 if case["call"] == "grad" else 1))}


# ---- the exact sums ---------------------------------------------------------

def _direct(pos, q):
    """phi_i = sum_j q_j / r_ij and F_i = q_i sum_j q_j (x_i - x_j) / r_ij^3 in FP64."""
    n = pos.shape[0]
    phi, force = torch.empty_like(q), torch.empty_like(pos)
    xq = torch.cat([pos, torch.ones((n, 1), device=pos.device, dtype=pos.dtype)], dim=1)
    step = max(1, (1 << 28) // n)
    for a in range(0, n, step):
        t = pos[a:a + step]
        m = t.shape[0]
        r = (t[:, 0:1] - pos[:, 0]).square_()
        for k in (1, 2):
            d = t[:, k:k + 1] - pos[:, k]
            r.addcmul_(d, d)
        r[torch.arange(m), torch.arange(a, a + m)] = math.inf
        r.rsqrt_()
        phi[a:a + m] = r @ q
        r.pow_(3).mul_(q)
        w = r @ xq  # sum_j w_ij (x_j, 1)
        force[a:a + m] = q[a:a + m, None] * (t * w[:, 3:] - w[:, :3])
    return phi, force


def exact(case, seed):
    """The exact sums (about 3e-11 s a pair); None where they take too long."""
    pos, q, counts = _inputs(case, seed)
    if case["call"] == "grad" and case["precision"] == "mixed":
        pos, q = pos.float().double(), q.float().double()
    counts = counts or [pos.shape[0]]
    if sum(float(c) ** 2 for c in counts) > 3e11:
        return None
    parts = [_direct(x, c) for x, c in zip(pos.split(counts), q.split(counts))]
    phi, force = (torch.cat(t) for t in zip(*parts))
    energy = 0.5 * (q * phi).sum()
    if case["call"] == "grad":
        return {"energy": energy, "dx": -force, "dq": phi}
    return {"phi": phi, "force": force, "energy": energy.reshape(1)}
