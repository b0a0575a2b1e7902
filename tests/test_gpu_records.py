"""Spawn records in the slots of their children's buckets, bit for bit against the oracle:
one slot per bucket and counts around the 64 records a wavefront merges in one round (the
buckets then hold up to several hundred, merged in rounds), with iterations abandoned and
re-run where the slots overflow; one and two words per determinant; a list that starts on
the reference, whose children's buckets receive most of the records."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

pytestmark = pytest.mark.gpu


def _run(ham, prm, slots, blocks, n):
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    if slots:
        buckets = gpu.estimates()["table_slots"] // 256
        F.fciqmc_set_test_options(gpu.h, 0, -1, slots * buckets)
    for _ in range(blocks):
        gpu.iterate(n)
        ref.iterate(n)
        dg, pg, _ = gpu.walkers()
        do, po, _ = ref.walkers()
        assert np.array_equal(dg if dg.ndim == 1 else dg[:, 0], do if do.ndim == 1 else do[:, 0])
        assert np.array_equal(pg, po)
        eg, eo = gpu.estimates(), ref.estimates()
        for k in ("n_walkers", "spawns", "merged", "aborted", "born", "ref_pop", "shift"):
            assert eg[k] == eo[k], k
    e = gpu.estimates()
    gpu.close()
    ref.close()
    return e


@pytest.mark.parametrize("words", [0, 2])
@pytest.mark.parametrize("slots", [1, 63, 64, 65])
def test_slots_per_bucket(slots, words):
    ham, prm, _ = S.workload("hubbard8")
    prm.det_capacity, prm.target_walkers, prm.det_words = 4096, 30000, words
    print(f"[gpu] records: {slots} slots per bucket, words {words}", flush=True)
    e = _run(ham, prm, slots, 3, 40)
    assert e["redos"] > 0


def test_list_on_the_reference():
    ham = S.hubbard_ring(10, 4.0)
    prm = S.Params(tau=0.01, shift_update_every=1, target_walkers=60000, initial_walkers=60000,
                   seed=5)
    print("[gpu] records: 60000 walkers on the reference", flush=True)
    e = _run(ham, prm, 0, 2, 20)
    assert e["redos"] == 0       # the slots are planned from the largest population


@pytest.mark.parametrize("words", [0, 2])
def test_crowded_buckets(words):
    """A list of many buckets whose records crowd into a few (walkers on the reference of a
    ring: each of its neighbours is sent a thousand): the crowded buckets' slots beyond
    everybody's, and the iterations re-run until their counts are known."""
    ham = S.hubbard_ring(10, 4.0)
    prm = S.Params(tau=0.01, initiator_threshold=0, target_walkers=10**9, initial_walkers=100_000,
                   det_capacity=1 << 21, seed=9, det_words=words)
    print(f"[gpu] records: crowded buckets, words {words}", flush=True)
    e = _run(ham, prm, 0, 3, 5)
    assert 1 <= e["redos"] <= 4


def test_crowded_batch():
    """The same beside systems that are not crowded, through a change of the batch."""
    ring, mol = S.hubbard_ring(10, 4.0), S.synthetic_molecule(8, 3, 3, 4)
    sy = [(mol, S.Params(tau=4e-3, initiator_threshold=0, target_walkers=10**9, initial_walkers=500,
                         seed=1)),
          (ring, S.Params(tau=0.01, initiator_threshold=0, target_walkers=10**9,
                          initial_walkers=60_000, det_capacity=1 << 21, seed=2)),
          (ring, S.Params(tau=0.01, initiator_threshold=0, target_walkers=10**9,
                          initial_walkers=90_000, det_capacity=1 << 20, seed=3))]
    print("[gpu] records: crowded systems in a batch", flush=True)
    h = F.fciqmc_batch_create(3, [a for a, _ in sy], [b for _, b in sy], F.current_stream())
    refs = [O.Oracle(a, b) for a, b in sy]
    for n, drop in ((4, False), (5, True), (4, False)):
        F.fciqmc_batch_iterate(h, n)
        for slot, ref in enumerate(refs):
            if ref is None:
                continue
            ref.iterate(n)
            d, p, _ = F.fciqmc_batch_slot_walkers(h, slot)
            do, po, _ = ref.walkers()
            assert np.array_equal(d, do) and np.array_equal(p, po), slot
        if drop:
            F.fciqmc_batch_retire(h, 0)
            refs[0].close()
            refs[0] = None
    for ref in refs[1:]:
        ref.close()
    F.fciqmc_free(h)


def test_slots_when_the_list_grows():
    """Few buckets with thousands of slots each (a start on the reference) that become
    thousands of buckets: a list is loaded that needs them, and the solve goes on."""
    ham = S.synthetic_molecule(20, 4, 4, 12)
    prm = S.Params(tau=2e-3, initiator_threshold=3, target_walkers=10**9, initial_walkers=200_000,
                   det_capacity=1024, seed=21)
    print("[gpu] records: slots of a list that grows", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    for n in (2, 3):
        gpu.iterate(n)
        ref.iterate(n)
        F.fciqmc_reserve(gpu.h, 1 << (22 if n == 2 else 25))
        (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
        assert np.array_equal(dg, do) and np.array_equal(pg, po)
    gpu.iterate(2)
    ref.iterate(2)
    (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
    assert np.array_equal(dg, do) and np.array_equal(pg, po)
    gpu.close()
    ref.close()


@pytest.mark.parametrize("words", [0, 2])
def test_after_a_buffer_that_does_not_fit(words):
    """A record buffer no device has room for is refused; the solve then goes on with one of
    its own size."""
    ham, prm, _ = S.workload("hubbard8")
    prm.det_words = words
    print(f"[gpu] records: a buffer that does not fit, words {words}", flush=True)
    gpu, ref = F.Solver(ham, prm, F.current_stream()), O.Oracle(ham, prm)
    for n in (20, 20):
        gpu.iterate(n)
        ref.iterate(n)
        (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
        assert np.array_equal(dg if dg.ndim == 1 else dg[:, 0], do if do.ndim == 1 else do[:, 0])
        assert np.array_equal(pg, po)
        with pytest.raises(F.FciqmcError) as e:
            F.fciqmc_set_test_options(gpu.h, 1, -1, 1 << 40)
        assert e.value.code == -2
    gpu.iterate(5)
    ref.iterate(5)
    (dg, pg, _), (do, po, _) = gpu.walkers(), ref.walkers()
    assert np.array_equal(pg, po) and len(dg) == len(do)
    gpu.close()
    ref.close()
