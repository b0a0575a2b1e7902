"""Double excitations that are null, bit for bit against the oracle: an attempt whose type
word picks a double that cannot be drawn spawns nothing, and is no single either."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

pytestmark = pytest.mark.gpu

COUNTS = ("n_walkers", "attempts", "spawns", "merged", "aborted", "born", "ref_pop")


def _words0(det):
    return det if det.ndim == 1 else det[:, 0]


@pytest.mark.parametrize("form", ["plain", "group", "two_words", "two_words_group"])
@pytest.mark.parametrize("p_double", [0.3, 0.6, 1.0])
def test_one_electron(p_double, form):
    """One electron has no double excitation: with an explicit share of doubles that share
    of the attempts is null."""
    irr = np.array([0, 1, 0, 1, 0, 0]) if form.endswith("group") else None
    ham = S.synthetic_molecule(6, 1, 0, 41, irreps=irr)
    ham.p_double = p_double
    prm = S.Params(tau=0.05, target_walkers=10**9, initial_walkers=2000, initial_shift=1.0, seed=7,
                   det_words=2 if form.startswith("two_words") else 0)
    print(f"[gpu] one electron, p_double {p_double}, {form}", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    gpu.iterate(10)
    ref.iterate(10)
    (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
    assert np.array_equal(_words0(dg), _words0(do)) and np.array_equal(pg, po)
    eg, eo = gpu.estimates(), ref.estimates()
    for k in COUNTS:
        assert eg[k] == eo[k], k
    assert (eg["total_spawns"] > 0) == (p_double < 1.0)
    gpu.close()
    ref.close()


def _pairs_without_target(ham):
    """Pairs of the reference's electrons for which no empty orbital has an empty partner."""
    nso, ref = 2 * ham.n_orb, int(ham.ref_det)
    irr = [0] * ham.n_orb if ham.orb_irrep is None else [int(x) for x in ham.orb_irrep]
    occ = [p for p in range(nso) if (ref >> p) & 1]
    emp = [p for p in range(nso) if not (ref >> p) & 1]
    none = 0
    for i, p in enumerate(occ):
        for q in occ[i + 1:]:
            g = irr[p >> 1] ^ irr[q >> 1]
            none += not any(a != b and sorted((a & 1, b & 1)) == sorted((p & 1, q & 1)) and
                            irr[a >> 1] ^ irr[b >> 1] == g for a in emp for b in emp)
    return none


def _group_system(seed, words, hphf=0):
    """Six electrons in ten orbitals; more than half of the reference's pairs have no target."""
    ham = S.synthetic_molecule(10, 3, 3, seed, irreps=np.array([2, 5, 7, 3, 3, 3, 3, 5, 3, 4]))
    ham.p_double = 0.9
    prm = S.Params(tau=5e-3, initiator_threshold=1, target_walkers=10**9, initial_walkers=3000,
                   initial_shift=2.0, seed=seed, det_words=words, hphf=hphf)
    return ham, prm


def _filled_system(seed, words):
    """Every spin-up orbital filled: without a point group, no pair with a spin-up electron
    has a target."""
    ham = S.synthetic_molecule(5, 5, 2, seed)
    ham.p_double = 0.9
    prm = S.Params(tau=5e-3, target_walkers=10**9, initial_walkers=3000, initial_shift=2.0, seed=seed,
                   det_words=words)
    return ham, prm


@pytest.mark.parametrize("words", [0, 2])
@pytest.mark.parametrize("form", ["group", "group_functions", "filled"])
def test_pairs_without_target(form, words):
    ham, prm = _filled_system(42, words) if form == "filled" else \
        _group_system(42, words, 1 if form == "group_functions" else 0)
    assert _pairs_without_target(ham) > 0
    print(f"[gpu] pairs without target: {form}, words {words}", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    for _ in range(2):
        gpu.iterate(8)
        ref.iterate(8)
        (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
        assert np.array_equal(_words0(dg), _words0(do)) and np.array_equal(pg, po)
        eg, eo = gpu.estimates(), ref.estimates()
        for k in COUNTS:
            assert eg[k] == eo[k], k
    gpu.close()
    ref.close()


@pytest.mark.parametrize("words", [0, 2])
def test_pairs_without_target_in_a_batch(words):
    """One workgroup spawns for systems of different point groups: the bounds of all but one
    are read from memory."""
    sy = [_group_system(43, words), _filled_system(44, words), _group_system(45, words),
          _group_system(46, words)]
    assert all(_pairs_without_target(ham) > 0 for ham, _ in sy)
    print(f"[gpu] pairs without target in a batch, words {words}", flush=True)
    h = F.fciqmc_batch_create(len(sy), [a for a, _ in sy], [b for _, b in sy], F.current_stream())
    F.fciqmc_set_launch(h, 1, 256, 4)
    refs = [O.Oracle(a, b) for a, b in sy]
    for _ in range(2):
        F.fciqmc_batch_iterate(h, 6)
        for slot, ref in enumerate(refs):
            ref.iterate(6)
            (d, p, _), (do, po, _) = F.fciqmc_batch_slot_walkers(h, slot), ref.walkers()
            assert np.array_equal(_words0(d), _words0(do)) and np.array_equal(p, po), slot
    for ref in refs:
        ref.close()
    F.fciqmc_free(h)
