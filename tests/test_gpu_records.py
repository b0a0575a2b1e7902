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
