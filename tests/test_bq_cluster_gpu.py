"""The biclique kernel whose couplings stay in registers across an XCD, forced through
PBIT_BQ_VARIANT=5 and by the timed choice, against the oracle, bit-exact: blocks that
only one side has, ragged sides, row tiles that are not full, more row tiles than the
device takes at once, runs past its threshold-row buffer, saturated rows, and what it
leaves to the other kernels."""
import os

import numpy as np
import pytest

import synth
from oracle import oracle
from paper_2510_23419_amd import pbit
from tests.test_bq_variants_gpu import _biclique_with_zeros
from tests.test_parity_gpu import EXTREME_BETAS, HIGH_REPLICA, HIGH_SWEEP, _every_sweep, graph_of

pytestmark = pytest.mark.gpu

CLUSTER = 5


def _forced_context(variant, budget=0):
    old = os.environ.get("PBIT_BQ_VARIANT")
    os.environ["PBIT_BQ_VARIANT"] = variant
    try:
        return pbit.Context(0, hbm_budget_bytes=budget)
    finally:
        if old is None:
            del os.environ["PBIT_BQ_VARIANT"]
        else:
            os.environ["PBIT_BQ_VARIANT"] = old


@pytest.fixture(scope="module")
def forced():
    c = _forced_context("5")
    yield c.ctx
    c.close()


@pytest.fixture(scope="module")
def ctx():
    c = pbit.Context(0)
    yield c.ctx
    c.close()


def _sampled(ctx, inst, beta, R, seed, **kw):
    """Spins and energies of the first, a middle and the last replica group."""
    print("cluster", inst["J"].shape, "R", R, "S", len(beta), flush=True)
    prob = pbit.load_instance(ctx, inst)
    got = pbit.pbit_anneal(ctx, prob, beta, R, seed, **kw)
    variant = pbit.pbit_profile_variant(ctx)
    pbit.pbit_unload_problem(ctx, prob)
    g = graph_of(inst)
    for q in sorted({0, (R // 4) // 2, (R - 1) // 4}):
        cnt = min(4, R - 4 * q)
        ref = oracle.anneal(g, beta, cnt, seed, replica_offset=4 * q)
        assert np.array_equal(got.spins[4 * q:4 * q + cnt], ref.spins), q
        assert np.array_equal(got.energies[4 * q:4 * q + cnt], ref.energies), q
    return variant


# block counts at the edges of the four operand sizes (8, 16, 32 and 64 blocks), blocks of one side
# only, an odd count of blocks in pairs
@pytest.mark.parametrize("na,nb,R,S", [
    (1, 1, 1, 3), (33, 1, 5, 20), (1, 65, 33, 20), (32, 32, 32, 33), (256, 256, 64, 17), (257, 31, 40, 17),
    (129, 512, 31, 18), (513, 480, 70, 16), (100, 1024, 36, 9), (1024, 993, 128, 40), (64, 96, 1100, 12),
    (1025, 1100, 70, 9), (2048, 2017, 33, 6), (40, 1800, 300, 17), (1056, 30, 600, 5),
])
def test_cluster_sides_and_replicas(forced, na, nb, R, S):
    inst = synth.biclique_instance(na, seed=na + 5 * nb, nb=nb)
    assert _sampled(forced, inst, synth.beta_linear(0.05, 2.0, S), R, seed=na + R) == CLUSTER


@pytest.mark.parametrize("sched", sorted(EXTREME_BETAS))
def test_cluster_extreme_betas(forced, sched):
    """Rows as wide as the largest field are left to the other kernels beyond 256 entries."""
    inst = _biclique_with_zeros(97, 60, seed=7)
    variant = _sampled(forced, inst, np.array(EXTREME_BETAS[sched]), 40, seed=43)
    assert variant == CLUSTER


def test_cluster_wide_rows_fall_back(forced):
    inst = synth.biclique_instance(300, seed=3, nb=290)
    assert _sampled(forced, inst, np.zeros(4), 8, seed=1) != CLUSTER


def test_cluster_given_spins_traces_and_resume(forced):
    inst = _biclique_with_zeros(130, 70, seed=81)
    beta = synth.beta_linear(0.05, 2.0, 8)
    _every_sweep(forced, inst, beta, 40, seed=71, init=synth.random_spins(40, 200, seed=6))
    assert pbit.pbit_profile_variant(forced) == CLUSTER
    prob = pbit.load_instance(forced, inst)
    first = pbit.pbit_anneal(forced, prob, beta[:3], 40, seed=71)
    second = pbit.pbit_anneal(forced, prob, beta[3:], 40, seed=71, sweep_offset=3, init_spins=first.spins)
    pbit.pbit_unload_problem(forced, prob)
    whole = oracle.anneal(graph_of(inst), beta, 40, seed=71)
    assert np.array_equal(second.spins, whole.spins) and np.array_equal(second.energies, whole.energies)


def test_cluster_counters_past_31_bits(forced):
    inst = _biclique_with_zeros(70, 100, seed=79)
    _every_sweep(forced, inst, synth.beta_linear(0.05, 2.0, 6), 40, seed=59, sweep_offset=HIGH_SWEEP,
                 replica_offset=HIGH_REPLICA)
    assert pbit.pbit_profile_variant(forced) == CLUSTER


def test_timed_choice_takes_it(ctx):
    """Sides of 600 to 1000 in runs of sweeps, where the others need two to four times as long;
    not in shorter runs."""
    inst = synth.biclique_instance(1000, seed=9, nb=600)
    assert _sampled(ctx, inst, synth.beta_linear(0.05, 2.0, 64), 100, seed=5) == CLUSTER
    assert _sampled(ctx, inst, synth.beta_linear(0.05, 2.0, 8), 100, seed=5) != CLUSTER


def test_exchange_memory_costs_no_budget():
    """Two problems annealed one after the other under every budget that the 64 x 64 kernel
    gets by with."""
    insts = [synth.biclique_instance(n, seed=n) for n in (600, 520)]
    beta = synth.beta_linear(0.05, 2.0, 16)
    refs = [oracle.anneal(graph_of(i), beta, 4, 1) for i in insts]

    def sequence(variant, budget):
        c = _forced_context(variant, budget)
        try:
            for inst, ref in zip(insts, refs):
                got = pbit.pbit_anneal(c.ctx, pbit.load_instance(c.ctx, inst), beta, 64, 1)
                assert np.array_equal(got.spins[:4], ref.spins)
            return True
        except pbit.PbitError as err:
            assert "budget" in str(err)
            return False
        finally:
            c.close()

    seen = set()
    for budget in range(3_000_000, 8_000_000, 100_000):
        ok = sequence("1", budget)
        seen.add(ok)
        assert not ok or sequence("5", budget), budget
    assert seen == {True, False}


def _impatient_context():
    old = os.environ.get("PBIT_BQ_MEET_US")
    os.environ["PBIT_BQ_MEET_US"] = "0"
    try:
        c = _forced_context("5")
    finally:
        if old is None:
            del os.environ["PBIT_BQ_MEET_US"]
        else:
            os.environ["PBIT_BQ_MEET_US"] = old
    return c


def test_workgroups_that_do_not_meet():
    """A wait limit of zero: the workgroups leave before touching the spins, another kernel runs
    the sweeps, and the next anneals do not try again."""
    c = _impatient_context()
    try:
        for na, nb, R, S in [(300, 200, 40, 20), (520, 600, 70, 18), (64, 32, 8, 5), (1100, 700, 33, 16)]:
            inst = synth.biclique_instance(na, seed=na, nb=nb)
            for _ in range(2):
                assert _sampled(c.ctx, inst, synth.beta_linear(0.05, 2.0, S), R, seed=R) != CLUSTER
    finally:
        c.close()


def test_static_scratch_takes_the_kernel_already_timed():
    """pbit_anneal_dev_noalloc after an anneal that timed the shape, and chose the cluster kernel,
    runs the fastest of the others, as an anneal too short for that kernel does."""
    import torch
    inst = synth.biclique_instance(1000, seed=11, nb=600)
    c = pbit.Context(0)
    try:
        prob = pbit.load_instance(c.ctx, inst)
        beta = synth.beta_linear(0.05, 2.0, 64)
        pbit.pbit_anneal(c.ctx, prob, beta, 100, 3)
        assert pbit.pbit_profile_variant(c.ctx) == CLUSTER
        pbit.pbit_anneal(c.ctx, prob, beta[:8], 100, 3)
        timed = pbit.pbit_profile_variant(c.ctx)
        spins = torch.empty((100, 1600), dtype=torch.int8, device="cuda:0")
        pbit.pbit_anneal_dev(c.ctx, prob, beta[:8], 100, 3, spins, noalloc=True)
        assert pbit.pbit_profile_variant(c.ctx) == timed != CLUSTER
        ref = oracle.anneal(graph_of(inst), beta[:8], 4, 3)
        assert np.array_equal(spins[:4].cpu().numpy(), ref.spins)
    finally:
        c.close()


def test_profile_counts_the_sweeps_that_ran():
    """The window of a launch whose workgroups did not meet is no half-sweep's time."""
    c = _impatient_context()
    try:
        prob = pbit.load_instance(c.ctx, synth.biclique_instance(300, seed=1, nb=200))
        pbit.pbit_profile_enable(c.ctx, 1)
        pbit.pbit_anneal(c.ctx, prob, synth.beta_linear(0.05, 2.0, 20), 40, 1)
        assert pbit.pbit_profile_variant(c.ctx) == 4  # sweeps in LDS, one launch
        ms, launches = pbit.pbit_profile_read(c.ctx, pbit.PBIT_BICLIQUE)
        assert launches == 40 and ms > 0
    finally:
        c.close()
