"""Batched biclique tiles on the FP4 matrix cores against the oracle, bit-exact, where their
loops end: K steps of 64 sites in every remainder of a ring of four, site blocks that fill no
wave and more than the 16 waves, ragged sides, replicas past one tile, threshold rows past the
16 held at a time, given spins, and fields at their largest."""
import os

import numpy as np
import pytest

import synth
from oracle import oracle
from paper_2510_23419_amd import pbit
from tests.test_bq_variants_gpu import _biclique_with_zeros
from tests.test_parity_gpu import graph_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = pbit.Context(0)
    yield c.ctx
    c.close()


def _check(ctx, inst, beta, R, seed, **kw):
    print("tiles", inst["J"].shape, "R", R, "S", len(beta), flush=True)
    prob = pbit.load_instance(ctx, inst)
    got = pbit.pbit_anneal_batch(ctx, [dict(problem=prob, beta=beta, n_replicas=R, seed=seed, **kw)])[0]
    pbit.pbit_unload_problem(ctx, prob)
    ref = oracle.anneal(graph_of(inst), beta, R, seed, **kw)
    assert np.array_equal(got.spins, ref.spins) and np.array_equal(got.energies, ref.energies)


@pytest.mark.parametrize("na,nb,R,S", [(1, 1, 1, 2), (64, 65, 33, 17), (129, 192, 31, 33), (257, 300, 64, 5),
                                       (321, 40, 70, 16), (600, 530, 40, 3), (31, 1100, 5, 4)])
def test_tiles_at_their_edges(ctx, na, nb, R, S):
    _check(ctx, _biclique_with_zeros(na, nb, seed=na + nb) if min(na, nb) > 8 else
           synth.biclique_instance(na, seed=3, nb=nb), synth.beta_linear(0.05, 2.0, S), R, seed=na)


def test_tiles_given_spins_and_offsets(ctx):
    inst = _biclique_with_zeros(100, 90, seed=4)
    _check(ctx, inst, synth.beta_linear(0.05, 2.0, 6), 40, seed=9, init_spins=synth.random_spins(40, 190, seed=2),
           sweep_offset=7, replica_offset=8)


@pytest.mark.parametrize("n", [700, 1500])
def test_largest_fields_are_exact(ctx, n):
    """All couplings +1 and all spins alike: |I| = n, through a batch and the per-instance call."""
    inst = synth.ferro_biclique(n)
    beta, R = np.full(16, 1e-4), 32
    init = np.ones((R, 2 * n), np.int8)
    init[1::2] = -1
    ref = oracle.anneal(graph_of(inst), beta, R, 5, init_spins=init)
    prob = pbit.load_instance(ctx, inst)
    outs = [pbit.pbit_anneal(ctx, prob, beta, R, 5, init_spins=init),
            pbit.pbit_anneal_batch(ctx, [dict(problem=prob, beta=beta, n_replicas=R, seed=5, init_spins=init)])[0]]
    pbit.pbit_unload_problem(ctx, prob)
    for got in outs:
        assert np.array_equal(got.spins, ref.spins) and np.array_equal(got.energies, ref.energies)


def test_longest_side_of_the_bit_kernel_is_exact():
    """128 x 524160, the longest side the FP4 bit kernel takes.  Partial sums reach 524160, the most that
    can cancel to a field whose decision is open (the float accumulators are exact to 2^20), and the
    fields of some hundreds that are left have to decide as in the int8 kernel with int32 sums."""
    na, nb, R = 128, 524160, 8
    rng = np.random.default_rng(1)
    J = np.ones((na, nb), np.int8)
    J[:, nb // 2:] = -1
    J[rng.random((na, nb), dtype=np.float32) < 2e-4] = 0
    spins = np.full((R, na + nb), -1, np.int8)
    spins[rng.random((R, na + nb), dtype=np.float32) < 5e-4] = 1
    inst = {"kind": "biclique", "dims": (na, nb), "J": J, "h": None}
    got = {}
    for variant in ("3", "2"):
        old = os.environ.get("PBIT_BQ_VARIANT")
        os.environ["PBIT_BQ_VARIANT"] = variant
        try:
            c = pbit.Context(0)
        finally:
            if old is None:
                del os.environ["PBIT_BQ_VARIANT"]
            else:
                os.environ["PBIT_BQ_VARIANT"] = old
        print("longest side, kernel", variant, flush=True)
        with c:
            out = pbit.pbit_anneal(c.ctx, pbit.load_instance(c.ctx, inst), [0.006, 0.006], R, 3, init_spins=spins)
            assert pbit.pbit_profile_variant(c.ctx) == int(variant)
            got[variant] = (out.spins, out.energies)
    field = J.sum(1, dtype=np.int64)  # of spins +1; the fields that decide are far below the partial sums
    assert np.abs(field).max() < 2000
    assert np.array_equal(got["3"][0], got["2"][0]) and np.array_equal(got["3"][1], got["2"][1])
