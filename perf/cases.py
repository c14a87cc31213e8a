"""Performance cases of the p-bit sweep: the anneals a user of this library runs.

Every case is one call through the public entry points on synthetic +-1
instances: a whole anneal (random start, every half-sweep of the schedule, final
energies and spins) on device buffers or through the host interface, a batch of
anneals, or one window of budgets of Algorithm 1.  ``listed()`` holds the fixed
cases, ``draw()`` more of the same ranges.  Spins and energies are whole numbers
and a pure function of the inputs, so two versions of the library have to agree
on every one of them.
"""
import math

import numpy as np
import torch

import synth
from paper_2510_23419_amd import alg1, pbit

DEVICE = "cuda:0"


def listed():
    return [
        # the smallest benchmark configuration: a 6^3 cube with 64 replicas, where a sweep is a
        # handful of workgroups and latency is everything
        dict(name="cube6", kind="cube", dims="6x6x6", field="zero", zeros=0.0, replicas=64, sweeps=1000,
             schedule="linear", beta0=0.1, beta1=3.0, entry="dev", trace=0),
        # the two cubes of the headline benchmark at their 4096 replicas (a fifth of its 10^4 sweeps)
        dict(name="cube16", kind="cube", dims="16x16x16", field="zero", zeros=0.0, replicas=4096, sweeps=2000,
             schedule="geometric", beta0=0.1, beta1=5.0, entry="dev", trace=0),
        dict(name="cube32", kind="cube", dims="32x32x32", field="zero", zeros=0.0, replicas=4096, sweeps=2000,
             schedule="geometric", beta0=0.1, beta1=5.0, entry="dev", trace=0),
        # an odd-shaped box with external fields and a ragged replica count, through the host
        # interface with an energy trace: how a solution-quality study looks at one instance
        dict(name="box_fields", kind="cube", dims="24x10x14", field="uniform3", zeros=0.0, replicas=300, sweeps=1000,
             schedule="geometric", beta0=0.1, beta1=5.0, entry="host", trace=100),
        # the dimerized cube that stands in for hardware-embedded lattices: a general graph of
        # 5488 spins in five update groups
        dict(name="dimer14", kind="dimer", side=14, field="zero", replicas=4096, sweeps=500,
             schedule="geometric", beta0=0.1, beta1=5.0, entry="dev", trace=0),
        # Algorithm 1 near its answer for 98 % quality on 10^3 cubes: 16 neighbouring budgets of
        # 20 trials each, evaluated in one batched launch
        dict(name="alg1_window", kind="alg1", side=10, trials=20, budget=1600, window=16),
        # a biclique of the paper's size range with unequal, ragged sides and few replicas
        dict(name="bq_small", kind="biclique", na=200, nb=137, field="uniform3", zeros=0.0, replicas=100, sweeps=1000,
             schedule="linear", beta0=0.05, beta1=2.0, entry="host", trace=0),
        # the biclique benchmark sizes at 1024 replicas (parts of its 2000 sweeps)
        dict(name="bq512", kind="biclique", na=512, nb=512, field="uniform3", zeros=0.0, replicas=1024, sweeps=1000,
             schedule="linear", beta0=0.05, beta1=2.0, entry="dev", trace=0),
        dict(name="bq1024", kind="biclique", na=1024, nb=1024, field="uniform3", zeros=0.0, replicas=1024, sweeps=1000,
             schedule="linear", beta0=0.05, beta1=2.0, entry="dev", trace=0),
        dict(name="bq2048", kind="biclique", na=2048, nb=2048, field="uniform3", zeros=0.0, replicas=1024, sweeps=500,
             schedule="linear", beta0=0.05, beta1=2.0, entry="dev", trace=0),
        dict(name="bq4096", kind="biclique", na=4096, nb=4096, field="uniform3", zeros=0.0, replicas=1024, sweeps=250,
             schedule="linear", beta0=0.05, beta1=2.0, entry="dev", trace=0),
        # an eighth of the mixed bag of 256 jobs (cubes of side 8 to 24, bicliques of 64 to 1024 per
        # side, 32 to 512 replicas), all in one batched call: what the server does in a busy second
        dict(name="bag32", kind="bag", jobs=32, bag_seed=0, max_side=24, max_n=1024, min_sweeps=1000, max_sweeps=5000),
    ]


# ---------------------------------------------------------------- drawn cases

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    """A rough running time in seconds, only used to keep drawn cases below the largest listed one."""
    if case["kind"] == "alg1":
        return case["budget"] * 8e-6 + case["window"] * case["trials"] * case["budget"] * case["side"] ** 3 / 5e11
    if case["kind"] == "bag":
        return case["jobs"] * case["max_sweeps"] / 5000 * 4e-3 + case["max_sweeps"] * 2e-5
    n, bond_ends, groups = _sizes(case)
    per_sweep = case["replicas"] * (n / 1.2e12 + (bond_ends / 8e14 if case["kind"] == "biclique" else 0))
    snapshots = case["sweeps"] // case["trace"] if case["trace"] else 0
    return case["sweeps"] * max(per_sweep, groups * 4e-6) + (snapshots + 1) * 1e-4


def draw(rng):
    """One more case of the listed ranges: shapes, replicas and sweeps spread over their
    logarithms, ragged ones among them, fields, diluted couplings and both interfaces."""
    cap = 0.8 * _cost(listed()[2])
    kind = rng.choice(["cube", "cube", "cube", "dimer", "random", "biclique", "biclique", "biclique", "alg1", "bag"])
    if kind == "alg1":
        case = dict(kind=kind, side=rng.randint(3, 10), trials=20, budget=_log_int(rng, 20, 2000),
                    window=rng.choice([8, 16]))
    elif kind == "bag":
        lo = _log_int(rng, 100, 1000)
        case = dict(kind=kind, jobs=_log_int(rng, 4, 30), bag_seed=rng.randint(1, 10**6),
                    max_side=rng.choice([12, 16, 24, 32]), max_n=_log_int(rng, 128, 1024), min_sweeps=lo,
                    max_sweeps=min(5000, 5 * lo))
    else:
        if kind == "cube":
            if rng.random() < 0.5:
                sides = [2 * _log_int(rng, 2, 16)] * 3
            else:
                sides = [2 * _log_int(rng, 1, 16) for _ in range(3)]
            case = dict(kind=kind, dims="x".join(map(str, sides)), zeros=rng.choice([0.0, 0.0, 0.0, 0.2]))
        elif kind == "dimer":
            case = dict(kind=kind, side=rng.randint(3, 14))
        elif kind == "random":
            case = dict(kind=kind, spins=_log_int(rng, 30, 8000), degree=rng.choice([3, 4, 6, 10]))
        else:
            na = _log_int(rng, 10, 4096)
            nb = na if rng.random() < 0.6 else min(4096, max(1, int(na * rng.uniform(0.4, 2.5))))
            case = dict(kind=kind, na=na, nb=nb, zeros=rng.choice([0.0, 0.0, 0.0, 0.2]))
        linear = rng.random() < 0.5
        case.update(field=rng.choice(["zero", "uniform3"]), replicas=_log_int(rng, 16, 4096 if kind != "biclique" else 1536),
                    sweeps=_log_int(rng, 30, 3000), schedule="linear" if linear else "geometric",
                    beta0=0.05 if kind == "biclique" else 0.1, beta1=rng.choice([2.0, 3.0, 5.0]),
                    entry=rng.choice(["dev", "dev", "host"]), trace=0)
        if case["entry"] == "host" and rng.random() < 0.5:
            case["trace"] = max(1, case["sweeps"] // rng.randint(3, 20))
    while _cost(case) > cap:
        key = {"alg1": "budget", "bag": "jobs"}.get(kind, "sweeps")
        if case[key] <= 4:
            case["replicas"] = max(16, case["replicas"] // 2)
        else:
            case[key] = max(4, int(case[key] * 0.7))
    if case.get("trace"):
        case["trace"] = min(case["trace"], case["sweeps"])
    return case


# ---------------------------------------------------------------- inputs

def _instance(case, seed):
    kind, field = case["kind"], case.get("field", "zero")
    if kind == "cube":
        inst = synth.ea_instance(tuple(int(v) for v in case["dims"].split("x")), seed=seed, field=field)
    elif kind == "dimer":
        return synth.dimerized_cube(case["side"], seed=seed, field=field)
    elif kind == "random":
        return synth.random_sparse_graph(case["spins"], case["degree"], seed=seed, field=field)
    else:
        inst = synth.biclique_instance(case["na"], seed=seed, nb=case["nb"], field=field)
    if case["zeros"]:
        keep = np.random.default_rng(seed + 1).random(inst["J"].shape) >= case["zeros"]
        inst["J"] = (inst["J"] * keep).astype(np.int8)
    return inst


def _alg1_instance(case, seed):
    """A +-1 cube of Algorithm 1's ladder; odd sides go through the general-graph form."""
    inst = synth.ea_instance(case["side"], seed=seed)
    return inst if case["side"] % 2 == 0 else synth.ea_bond_list(inst)


def _schedule(case):
    make = synth.beta_linear if case["schedule"] == "linear" else synth.beta_geometric
    return make(case["beta0"], case["beta1"], case["sweeps"])


def _bag(case):
    """The jobs' shapes, replicas and schedules (the couplings come from the input seed)."""
    return synth.mixed_bag(seed=case["bag_seed"], n_instances=case["jobs"],
                           ea_sides=tuple(range(8, case["max_side"] + 1, 2)), n_range=(64, case["max_n"]),
                           sweep_range=(case["min_sweeps"], case["max_sweeps"]))


def _bag_instance(job, seed):
    dims = job["instance"]["dims"]
    if job["instance"]["kind"] == "ea3d":
        return synth.ea_instance(dims, seed=seed)
    return synth.biclique_instance(dims[0], seed=seed, nb=dims[1])


def _budgets(case):
    return [case["budget"] + k for k in range(case["window"])]


def prepare(case, seed):
    """A context, its loaded problems and the schedule; device buffers where the case uses them."""
    context = pbit.Context(0)
    state = dict(case=case, context=context, seed=seed + 1)
    if case["kind"] == "bag":
        state["jobs"] = [dict(problem=pbit.load_instance(context.ctx, _bag_instance(j, 1000 * seed + k)),
                              beta=j["beta"], n_replicas=j["replicas"], seed=j["seed"] + seed)
                         for k, j in enumerate(_bag(case))]
    elif case["kind"] == "alg1":
        problem = pbit.load_instance(context.ctx, _alg1_instance(case, seed))
        state["runner"] = alg1.gpu_runner(context.ctx, problem, 0.35, 3.5, case["trials"], seed + 1)
        state["budgets"] = _budgets(case)
    else:
        state["problem"] = pbit.load_instance(context.ctx, _instance(case, seed))
        state["beta"] = _schedule(case)
        if case["entry"] == "dev":
            n = pbit.pbit_problem_spins(context.ctx, state["problem"])
            state["spins"] = torch.empty((case["replicas"], n), dtype=torch.int8, device=DEVICE)
            state["energies"] = torch.empty(case["replicas"], dtype=torch.int64, device=DEVICE)
    return state


def run(state):
    """One pass: the anneal (or the batch, or the window of budgets); spins and energies."""
    case, ctx = state["case"], state["context"].ctx
    if case["kind"] == "bag":
        return [(o.spins, o.energies) for o in pbit.pbit_anneal_batch(ctx, state["jobs"])]
    if case["kind"] == "alg1":
        return list(state["runner"](state["budgets"]))
    if case["entry"] == "dev":
        pbit.pbit_anneal_dev(ctx, state["problem"], state["beta"], case["replicas"], state["seed"], state["spins"],
                             d_energies=state["energies"])
        return state["spins"], state["energies"]
    out = pbit.pbit_anneal(ctx, state["problem"], state["beta"], case["replicas"], state["seed"],
                           trace_every=case["trace"])
    return (out.spins, out.energies) + ((out.energy_trace,) if case["trace"] else ())


# ---------------------------------------------------------------- work

def _sizes(case):
    """(spins, bond ends, update groups) of a single-anneal case."""
    if case["kind"] == "cube":
        n = math.prod(int(v) for v in case["dims"].split("x"))
        return n, 6 * n, 2
    if case["kind"] == "dimer":
        n = 2 * case["side"] ** 3
        return n, 4 * n, 5  # a pair bond and three cube bonds per spin, on average
    if case["kind"] == "random":
        return case["spins"], case["spins"] * max(2, case["degree"] // 2 * 2), 5
    return case["na"] + case["nb"], 2 * case["na"] * case["nb"], 2


def _anneal_work(n, bond_ends, replicas, sweeps):
    # a p-bit update: one multiply-add per bond end, a quarter of a ten-round Philox block
    # (two products and two XORs a round), a comparison; couplings in, spins and energies out
    return dict(bytes=bond_ends / 2 + replicas * (n + 8.0), flops=1.0 * replicas * sweeps * (2 * bond_ends + 11 * n))


def work(case):
    total = dict(bytes=0.0, flops=0.0)
    if case["kind"] == "bag":
        parts = []
        for j in _bag(case):
            d = j["instance"]["dims"]
            n, ends = (math.prod(d), 6 * math.prod(d)) if j["instance"]["kind"] == "ea3d" else (sum(d), 2 * d[0] * d[1])
            parts.append(_anneal_work(n, ends, j["replicas"], len(j["beta"])))
    elif case["kind"] == "alg1":
        n = case["side"] ** 3
        parts = [_anneal_work(n, 6 * n, case["trials"], b) for b in _budgets(case)]
    else:
        n, ends, _ = _sizes(case)
        parts = [_anneal_work(n, ends, case["replicas"], case["sweeps"])]
    for p in parts:
        total["bytes"] += p["bytes"]
        total["flops"] += p["flops"]
    return total


# ---------------------------------------------------------------- the sweep in plain torch

def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors of 32-bit words; returns the four words."""
    low = 0xFFFFFFFF
    for _ in range(10):
        p, q = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # modulo 2^64: the bits of the unsigned product
        c0, c1, c2, c3 = ((q >> 32) & low) ^ c1 ^ k0, q & low, ((p >> 32) & low) ^ c3 ^ k1, p & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return c0, c1, c2, c3


def _words(sites, sweep, replicas, domain, seed):
    """One word per (site, replica): word (replica mod 4) of the block of (site, sweep, replica / 4, domain)."""
    groups = torch.arange((replicas + 3) // 4, dtype=torch.int64, device=sites.device)
    shape = (sites.numel(), groups.numel())
    full = [sites[:, None].expand(shape), torch.full(shape, sweep, dtype=torch.int64, device=sites.device),
            groups[None, :].expand(shape), torch.full(shape, domain, dtype=torch.int64, device=sites.device)]
    w = _philox(*full, seed & 0xFFFFFFFF, seed >> 32)
    return torch.stack(w, dim=2).reshape(sites.numel(), -1)[:, :replicas]


def _greedy_colours(n, bi, bj):
    near = [[] for _ in range(n)]
    for a, b in zip(bi.tolist(), bj.tolist()):
        near[a].append(b)
        near[b].append(a)
    colour = [-1] * n
    for v in range(n):
        used = {colour[u] for u in near[v]}
        colour[v] = next(c for c in range(n) if c not in used)
    return np.array(colour)


def _bonds(inst):
    """(spins, bond ends i, j, couplings, fields, colours) of any instance."""
    if inst["kind"] == "graph":
        colours = _greedy_colours(inst["n"], inst["bond_i"], inst["bond_j"])
        return inst["n"], inst["bond_i"], inst["bond_j"], inst["bond_J"], inst["h"], colours
    if inst["kind"] == "ea3d":
        lx, ly, lz = inst["dims"]
        i = np.arange(lx * ly * lz)
        x, y, z = i % lx, i // lx % ly, i // (lx * ly)
        far = [(x + 1) % lx + lx * (y + ly * z), x + lx * ((y + 1) % ly + ly * z), x + lx * (y + ly * ((z + 1) % lz))]
        return i.size, np.tile(i, 3), np.concatenate(far), inst["J"].reshape(-1), inst["h"], (x + y + z) % 2
    na, nb = inst["dims"]
    a, b = np.meshgrid(np.arange(na), na + np.arange(nb), indexing="ij")
    return na + nb, a.ravel(), b.ravel(), inst["J"].reshape(-1), inst["h"], (np.arange(na + nb) >= na).astype(int)


def exact(case, seed):
    """Spins and energies of one anneal by the definition of the sweep, in 64-bit integers
    (the fields, below 2^53, as float64 products); None where that would take too long."""
    if case["kind"] in ("bag", "alg1"):
        return None
    n, ends, groups = _sizes(case)
    elements = case["replicas"] * n
    if case["sweeps"] * (groups * 1.5e-3 + elements * 6e-10) > 12 or n * n * 8 > 2 << 30:
        return None
    n, bi, bj, bJ, h, colours = _bonds(_instance(case, seed))
    R, beta, anneal_seed = case["replicas"], _schedule(case), seed + 1
    J = torch.zeros((n, n), dtype=torch.float64, device=DEVICE)
    bi, bj = torch.as_tensor(bi, dtype=torch.int64, device=DEVICE), torch.as_tensor(bj, dtype=torch.int64, device=DEVICE)
    bJ = torch.as_tensor(bJ, device=DEVICE).double()
    J.index_put_((bi, bj), bJ, accumulate=True)
    J.index_put_((bj, bi), bJ, accumulate=True)
    h = torch.zeros(n, dtype=torch.float64, device=DEVICE) if h is None else torch.as_tensor(h, device=DEVICE).double()
    amax = int((J.abs().sum(1) + h.abs()).max().item())
    sites = [torch.as_tensor(np.flatnonzero(colours == c), device=DEVICE) for c in range(int(colours.max()) + 1)]
    rows = [J[s].contiguous() for s in sites]
    start = _words(torch.arange(n, dtype=torch.int64, device=DEVICE), 0, R, 1, anneal_seed)
    m = torch.where(start < 2**31, 1.0, -1.0).double()  # [n][R]

    def energy():
        return (-(m * (J @ m)).sum(0) / 2 - h @ m).round().long()

    def threshold(b, a):  # ceil(2^32 / (1 + exp(2 b a)) - 1/2)
        x = 2.0 * b * a
        return int(math.ceil(math.ldexp(1.0 / (1.0 + math.exp(x)) if x < 709.0 else 0.0, 32) - 0.5))

    trace = []
    for t, b in enumerate(beta.tolist()):
        row = torch.tensor([threshold(b, a) for a in range(amax + 1)], dtype=torch.int64, device=DEVICE)
        for s, Js in zip(sites, rows):
            field = (Js @ m + h[s, None]).round().long()
            w = _words(s, t, R, 0, anneal_seed)
            up = field >= 0
            minority = torch.where(up, 0xFFFFFFFF - w, w) < row[field.abs()]
            m[s] = torch.where(up != minority, 1.0, -1.0).double()
        if case["trace"] and (t + 1) % case["trace"] == 0:
            trace.append(energy())
    spins, energies = m.t().to(torch.int8).contiguous(), energy()
    if case["entry"] == "dev":
        return spins, energies
    out = (spins.cpu().numpy(), energies.cpu().numpy())
    return out + ((torch.stack(trace).cpu().numpy(),) if case["trace"] else ())
