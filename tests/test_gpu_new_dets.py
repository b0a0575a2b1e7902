"""Diagonal elements of determinants that enter the list, bit for bit against the oracle
(they decide the deaths of the following iterations): electron counts around the batches of
four in which the pair sums are loaded, and launches whose windows alternate between
systems, so that the queue of new determinants is emptied at a change of system."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

pytestmark = pytest.mark.gpu


def _molecule(na, nb, seed):
    ham = S.synthetic_molecule(9, na, nb, seed)
    prm = S.Params(tau=4e-3, initiator_threshold=0, target_walkers=10**9, initial_walkers=400,
                   initial_shift=1.0, seed=seed)
    return ham, prm


@pytest.mark.parametrize("words", [0, 2])
@pytest.mark.parametrize("na,nb", [(1, 0), (1, 1), (2, 1), (3, 2), (3, 3), (4, 5)])
def test_electron_counts(na, nb, words):
    ham, prm = _molecule(na, nb, 60 + 10 * na + nb)
    prm.det_words = words
    print(f"[gpu] new determinants: {na}+{nb} electrons, words {words}", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    for _ in range(2):
        gpu.iterate(12)
        ref.iterate(12)
        dg, pg, _ = gpu.walkers()
        do, po, _ = ref.walkers()
        assert np.array_equal(dg if words == 0 else dg[:, 0], do if do.ndim == 1 else do[:, 0])
        assert np.array_equal(pg, po)
    gpu.close()
    ref.close()


def test_systems_alternate():
    sy = [_molecule(2, 2, 91), _molecule(4, 3, 92), _molecule(1, 1, 93), _molecule(3, 3, 94),
          _molecule(5, 5, 95)]
    print("[gpu] new determinants: five systems in one batch", flush=True)
    h = F.fciqmc_batch_create(5, [a for a, _ in sy], [b for _, b in sy], F.current_stream())
    F.fciqmc_set_launch(h, 64, 256, 2)     # two workgroups: each meets several systems
    F.fciqmc_batch_iterate(h, 24)
    for slot, (ham, prm) in enumerate(sy):
        ref = O.Oracle(ham, prm)
        ref.iterate(24)
        d, p, _ = F.fciqmc_batch_slot_walkers(h, slot)
        do, po, _ = ref.walkers()
        assert np.array_equal(d, do) and np.array_equal(p, po), slot
        ref.close()
    F.fciqmc_free(h)


@pytest.mark.parametrize("m,na,nb", [(32, 31, 1), (32, 16, 17), (20, 1, 0), (33, 2, 1), (40, 20, 21),
                                     (64, 64, 63)])
def test_table_edges(m, na, nb):
    """Electron counts at the ends of the words of four in which the sums run, up to all
    spin orbitals but one, in tables of up to 64 spin orbitals and of more; and where no
    determinant's terms fit the workgroup's memory at once (127 electrons)."""
    ham = S.synthetic_molecule(m, na, nb, 11)
    prm = S.Params(tau=4e-3, initiator_threshold=0, target_walkers=10**9, initial_walkers=6000,
                   initial_shift=1.0, seed=3 * m + na)
    print(f"[gpu] new determinants: {na}+{nb} electrons in {m} orbitals", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    gpu.iterate(5)
    ref.iterate(5)
    (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
    assert len(pg) > (5 if na + nb == 1 else 40)
    assert np.array_equal(dg, do) and np.array_equal(pg, po)
    gpu.close()
    ref.close()
