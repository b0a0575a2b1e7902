"""The spawning kernel's rejection bounds, queues and tile lists, bit for bit against the
oracle: shares of double excitations on both sides of 1/2 and at 0 and 1, integrals over
many orders of magnitude and with zeros, acceptance probabilities above 1, the widest one-
and two-word systems, spin-coupled and point-group systems, tiles that fill their lists."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

pytestmark = pytest.mark.gpu


def _same(ham, prm, n, blocks=2, setup=None):
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    if setup is not None:
        setup(gpu.h)
    for _ in range(blocks):
        gpu.iterate(n)
        ref.iterate(n)
        dg, pg, _ = gpu.walkers()
        do, po, _ = ref.walkers()
        assert np.array_equal(dg, do) and np.array_equal(pg, po)
        eg, eo = gpu.estimates(), ref.estimates()
        for k in ("n_walkers", "attempts", "spawns", "merged", "aborted", "born", "ref_pop"):
            assert eg[k] == eo[k], k
    gpu.close()
    ref.close()


def _molecule(m, na, nb, seed, **more):
    ham = S.synthetic_molecule(m, na, nb, seed)
    prm = S.Params(tau=3e-3, initiator_threshold=2, target_walkers=10**9, initial_walkers=2000,
                   initial_shift=2.0, seed=seed, **more)
    return ham, prm


@pytest.mark.parametrize("p_double", [0.0, 0.2, 0.4999, 0.5, 0.9, 1.0])
def test_share_of_doubles(p_double):
    ham, prm = _molecule(12, 3, 3, 31)
    ham.p_double = p_double
    print(f"[gpu] spawn: p_double {p_double}", flush=True)
    _same(ham, prm, 10)


@pytest.mark.parametrize("scale", [1e-6, 1.0, 30.0])
@pytest.mark.parametrize("p_double", [0.3, 0.95])
def test_range_of_integrals(scale, p_double):
    ham, prm = _molecule(10, 3, 2, 32)
    rng = np.random.default_rng(1)
    ham.eri = ham.eri * scale * 10.0 ** rng.uniform(-7, 0, size=ham.eri.size)
    ham.eri[rng.random(ham.eri.size) < 0.3] = 0.0
    ham.p_double = p_double
    prm.initial_shift = 1.0
    print(f"[gpu] spawn: integrals x {scale}, p_double {p_double}", flush=True)
    _same(ham, prm, 8)


@pytest.mark.parametrize("tau", [0.05, 0.5])
def test_several_walkers_per_spawn(tau):
    ham, prm = _molecule(8, 2, 2, 33)
    prm.tau, prm.initial_walkers, prm.initial_shift = tau, 200, 0.0
    print(f"[gpu] spawn: tau {tau}", flush=True)
    _same(ham, prm, 3)


@pytest.mark.parametrize("m,ne,words", [(32, 4, 0), (32, 4, 2), (33, 4, 0), (64, 4, 0), (2, 1, 0), (2, 2, 0)])
def test_widths(m, ne, words):
    ham, prm = _molecule(m, (ne + 1) // 2, ne // 2, 34)
    prm.det_words = words
    print(f"[gpu] spawn: {ne} electrons in {m} orbitals, words {words}", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    gpu.iterate(8)
    ref.iterate(8)
    (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
    dg, do = dg.reshape(len(pg), -1), do.reshape(len(po), -1)
    w = min(dg.shape[1], do.shape[1])
    assert np.array_equal(dg[:, :w], do[:, :w]) and np.array_equal(pg, po)
    assert gpu.estimates()["spawns"] == ref.estimates()["spawns"]
    gpu.close()
    ref.close()


@pytest.mark.parametrize("mode", ["hphf", "group", "group_level", "level"])
def test_general_variant(mode):
    irr = np.array([0, 1, 2, 3, 0, 1, 2, 3, 0, 1, 2, 3]) if mode.startswith("group") else None
    ham = S.synthetic_molecule(12, 3, 3, 35, irreps=irr)
    prm = S.Params(tau=3e-3, initiator_threshold=2, target_walkers=10**9, initial_walkers=2000,
                   initial_shift=2.0, seed=9, hphf=1 if mode == "hphf" else 0,
                   space=S.SPACE_EXCITATION if "level" in mode else 0, max_excitation=4)
    print(f"[gpu] spawn: {mode}", flush=True)
    _same(ham, prm, 12)


@pytest.mark.parametrize("limit", [32, 64, 1000, -1])
def test_lists_that_fill(limit):
    """60000 walkers on the reference in tiles of 64: far more than the lists hold (one tile
    each, two, 31), or all listed, spread over several lists."""
    ham = S.hubbard_ring(8, 4.0)
    prm = S.Params(tau=0.01, shift_update_every=1, target_walkers=80000, initial_walkers=60000, seed=6)

    def setup(h):
        F.fciqmc_set_test_options(h, 1, limit, 0)
        F.fciqmc_set_launch(h, 64, 256, 64)
    print(f"[gpu] spawn: tile lists of {limit} in all", flush=True)
    _same(ham, prm, 6, 2, setup)
