"""The bit-held sweep on the GPU against the oracle, bit-exact, at the edges of its
dispatch: every record form, tile width (4, 8 and 16 replicas) and unit of work
(pairs, positions, four replicas of a position), groups that do not fill a wave,
sites of 8 to 15 terms, runs across the threshold-row boundaries, saturated
thresholds, and cubes of more than 8192 sites."""
import os

import numpy as np
import pytest

import synth
from oracle import oracle
from paper_2510_23419_amd import pbit

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["4", "8", "16"])
def width_ctx(request):
    old = os.environ.get("PBIT_GRAPH_SLAB")
    os.environ["PBIT_GRAPH_SLAB"] = request.param
    try:
        c = pbit.Context(0)
    finally:
        if old is None:
            del os.environ["PBIT_GRAPH_SLAB"]
        else:
            os.environ["PBIT_GRAPH_SLAB"] = old
    yield c.ctx
    c.close()


@pytest.fixture(scope="module")
def ctx():
    c = pbit.Context(0)
    yield c.ctx
    c.close()


def _graph(inst):
    if inst["kind"] == "ea3d":
        return oracle.ea_graph(inst["dims"], inst["J"], inst["h"])
    return oracle.graph_from_bonds(inst["n"], inst["bond_i"], inst["bond_j"], inst["bond_J"], inst.get("h"))


def _sampled(ctx, inst, beta, R, seed, **kw):
    """Spins and energies of the first, a middle and the last replica group."""
    prob = pbit.load_instance(ctx, inst)
    print("bits", inst["kind"], inst.get("dims", inst.get("n")), "R", R, "S", len(beta), flush=True)
    got = pbit.pbit_anneal(ctx, prob, beta, R, seed, **kw)
    pbit.pbit_unload_problem(ctx, prob)
    g = _graph(inst)
    for q in sorted({0, (R // 4) // 2, (R - 1) // 4}):
        cnt = min(4, R - 4 * q)
        ref = oracle.anneal(g, beta, cnt, seed, replica_offset=4 * q)
        assert np.array_equal(got.spins[4 * q:4 * q + cnt], ref.spins), q
        assert np.array_equal(got.energies[4 * q:4 * q + cnt], ref.energies), q


# tiles of 16, 8 and 4 replicas by the rule's choice at 4096, 2048 and 1024; pairs at 16^3, positions
# at 10^3 and 6^3; the aligned and the unaligned form, and the general one
@pytest.mark.parametrize("dims,R", [((16, 16, 16), 4096), ((16, 16, 16), 2048), ((16, 16, 16), 1024), ((10, 10, 10), 4096),
                                    ((10, 10, 10), 2052), ((6, 6, 6), 4096), ((6, 4, 2), 8200), ((4, 4, 2), 20)])
@pytest.mark.parametrize("field", ["zero", "uniform3"])
def test_cubes(ctx, dims, R, field):
    inst = synth.ea_instance(dims, seed=R, field=field)
    _sampled(ctx, inst, synth.beta_geometric(0.1, 5.0, 70), R, 5)


@pytest.mark.parametrize("S", [1, 2, 15, 16, 17, 31, 32, 33, 49])
def test_threshold_row_runs(ctx, S):
    inst = synth.ea_instance((8, 6, 4), seed=S, field="uniform3")
    _sampled(ctx, inst, synth.beta_linear(0.2, 4.0, S), 10, 8, sweep_offset=0)


# betas at which |I| >= 6, 4, 2 (and, with fields, odd ones) have zero thresholds
@pytest.mark.parametrize("betas", [[1.9, 1.95, 2.9, 3.9], [5.8, 11.5, 2.3, 1.91, 0.0]])
@pytest.mark.parametrize("field", ["zero", "uniform3"])
def test_saturated_thresholds(ctx, betas, field):
    inst = synth.ea_instance((8, 8, 8), seed=7, field=field)
    _sampled(ctx, inst, np.array(betas * 6), 24, 3)


def _hub_graph(n, degrees, seed):
    rng = np.random.default_rng(seed)
    pairs = set()
    for a, t in enumerate(degrees):
        for b in rng.choice(np.arange(len(degrees), n), size=t, replace=False):
            pairs.add((a, int(b)))
    for _ in range(n):
        a, b = rng.integers(len(degrees), n, 2)
        if a != b:
            pairs.add((int(min(a, b)), int(max(a, b))))
    pairs = sorted(pairs)
    J = np.where(rng.random(len(pairs)) < 0.5, 1, -1).astype(np.int8)
    return {"kind": "graph", "n": n, "bond_i": np.array([p[0] for p in pairs], np.int32),
            "bond_j": np.array([p[1] for p in pairs], np.int32), "bond_J": J,
            "h": rng.integers(-1, 2, size=n).astype(np.int8)}


@pytest.mark.parametrize("n,degrees", [(3, [2]), (70, [14, 8, 7]), (400, [8] * 33), (3000, [14, 9] * 20), (600, [20])])
@pytest.mark.parametrize("R", [1, 37])
def test_graphs_at_each_width(width_ctx, n, degrees, R):
    """Wide pairs (none, some, an odd number), one site per group, groups beyond one
    workgroup's threads, and a degree past the records' 15 (byte tiles)."""
    _sampled(width_ctx, _hub_graph(n, degrees, seed=n), synth.beta_geometric(0.1, 4.0, 40), R, 9)
    assert pbit.pbit_profile_graph_path(width_ctx) == 2


@pytest.mark.parametrize("dims,R", [((22, 22, 22), 16), ((24, 24, 24), 1024), ((32, 32, 32), 1024), ((32, 32, 32), 2048),
                                    ((32, 32, 30), 4096)])
def test_large_cubes(ctx, dims, R):
    field = "uniform3" if dims[2] == 30 else "zero"
    _sampled(ctx, synth.ea_instance(dims, seed=R, field=field), synth.beta_geometric(0.1, 5.0, 20), R, 2)
    assert pbit.pbit_profile_ea_path(ctx) == 1


@pytest.mark.parametrize("forced", [False, True])
def test_one_update_group(ctx, width_ctx, forced):
    """Sites without bonds form one group: its cursor stays on it over sweeps that one launch
    runs, per instance and batched (1200 spins take the bit-held form by themselves)."""
    n, R = (1200, 40) if not forced else (90, 21)
    inst = {"kind": "graph", "n": n, "bond_i": np.zeros(0, np.int32), "bond_j": np.zeros(0, np.int32),
            "bond_J": np.zeros(0, np.int8), "h": np.random.default_rng(n).integers(-1, 2, size=n).astype(np.int8)}
    c = width_ctx if forced else ctx
    beta = synth.beta_linear(0.1, 1.0, 40)
    _sampled(c, inst, beta, R, 6)
    prob = pbit.load_instance(c, inst)
    assert pbit.pbit_problem_colouring(c, prob)[1] == 1
    out = pbit.pbit_anneal_batch(c, [dict(problem=prob, beta=beta, n_replicas=R, seed=6)])[0]
    ref = oracle.anneal(_graph(inst), beta, 4, 6)
    assert np.array_equal(out.spins[:4], ref.spins) and np.array_equal(out.energies[:4], ref.energies)
    pbit.pbit_unload_problem(c, prob)


@pytest.mark.parametrize("kind", ["cube", "graph"])
def test_problems_load_without_room_for_records(kind):
    """Under every budget that a problem's other arrays and an anneal get by with, it loads and
    anneals; a cube in a batch needs the records (E_NOMEM without)."""
    inst = synth.ea_instance(16, seed=4) if kind == "cube" else _hub_graph(3000, [9] * 20, seed=4)
    n = 4096 if kind == "cube" else 3000
    beta = synth.beta_linear(0.1, 2.0, 6)
    ref = oracle.anneal(_graph(inst), beta, 4, 1)
    loaded, batched = [], []
    # a cube's other arrays take 7 bytes a site and a graph's at least 16, before spins (16 + rows)
    for budget in range(20_000, 400_000, 10_000):
        with pbit.Context(0, hbm_budget_bytes=budget) as c:
            try:
                p = pbit.load_instance(c.ctx, inst)
            except pbit.PbitError as err:
                assert err.code == pbit.PBIT_E_NOMEM and not loaded
                continue
            held = pbit.pbit_bytes_in_use(c.ctx)
            loaded.append(held)
            if held + 34 * n < budget:
                got = pbit.pbit_anneal(c.ctx, p, beta, 4, 1)
                assert np.array_equal(got.spins, ref.spins) and np.array_equal(got.energies, ref.energies)
            try:
                out = pbit.pbit_anneal_batch(c.ctx, [dict(problem=p, beta=beta, n_replicas=4, seed=1)])[0]
                assert np.array_equal(out.spins, ref.spins)
                batched.append(budget)
            except pbit.PbitError as err:
                assert err.code == pbit.PBIT_E_NOMEM
    print(kind, "held without and with records", min(loaded), max(loaded), flush=True)
    assert min(loaded) + 20 * n < max(loaded) and batched
    if kind == "cube":
        assert min(loaded) <= 7 * n + 1024


@pytest.mark.parametrize("n,records", [(39_936, True), (39_937, False), (60_000, False)])
def test_graphs_too_large_for_the_tiles_hold_no_records(ctx, n, records):
    inst = synth.random_sparse_graph(n, 3, seed=1)
    nb = len(inst["bond_J"])
    before = pbit.pbit_bytes_in_use(ctx)
    prob = pbit.load_instance(ctx, inst)
    held = pbit.pbit_bytes_in_use(ctx) - before
    # per vertex a class record of 16 bytes, per bond 8 + 9; the site records come to 34 a vertex
    assert (held > 16 * n + 17 * nb + 30 * n) == records, (held, n, nb)
    pbit.pbit_unload_problem(ctx, prob)


@pytest.mark.parametrize("dims,R,S", [((22, 22, 18), 24, 600), ((26, 26, 26), 130, 300), ((24, 24, 24), 64, 40),
                                      ((32, 32, 30), 20, 400), ((32, 32, 32), 512, 20)])
def test_cubes_whose_path_is_timed(ctx, dims, R, S):
    """Between the tiles and the launches by a timing; again from the cache, in part and at another
    replica count."""
    inst = synth.ea_instance(dims, seed=R)
    beta = synth.beta_geometric(0.1, 5.0, S)
    _sampled(ctx, inst, beta, R, 2)
    path = pbit.pbit_profile_ea_path(ctx)
    _sampled(ctx, inst, beta[:5], R, 3)
    assert pbit.pbit_profile_ea_path(ctx) == path
    _sampled(ctx, inst, beta[:20], R + 130, 4)


def test_large_cubes_run_in_tiles(ctx):
    """Runs of sweeps in LDS are one timed launch counted as its half-sweeps; of launches per half-sweep
    a window of eight is timed."""
    S = 40
    for dims, R, tiles in [((24, 24, 24), 4096, True), ((32, 32, 32), 4096, True), ((36, 36, 48), 16, False)]:
        prob = pbit.load_instance(ctx, synth.ea_instance(dims, seed=1))
        pbit.pbit_anneal(ctx, prob, synth.beta_linear(0.1, 1.0, S), R, 1, want_spins=False)
        pbit.pbit_profile_read(ctx, pbit.PBIT_EA3D, reset=True)
        pbit.pbit_profile_enable(ctx, 1000)
        pbit.pbit_anneal(ctx, prob, synth.beta_linear(0.1, 1.0, S), R, 1, want_spins=False)
        pbit.pbit_profile_enable(ctx, 0)
        launches = pbit.pbit_profile_read(ctx, pbit.PBIT_EA3D, reset=True)[1]
        assert launches == (2 * S if tiles else 8), (dims, R, launches)
        pbit.pbit_unload_problem(ctx, prob)
