"""Walker lists read out and loaded back, against numpy's sort: lengths around a wavefront,
a run and a workgroup of the sort, an odd and an even number of its digits, one and two
words, lists longer than the caller's arrays; and what a loaded list may hold."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

pytestmark = pytest.mark.gpu


def _lists(m, na, nb, n, rng):
    """n different determinants (as integers, in drawn order, the reference among them) and
    their populations."""
    ref = sum(1 << (2 * i) for i in range(na)) | sum(2 << (2 * i) for i in range(nb))
    dets = {ref}
    while len(dets) < n:
        a, b = rng.permutation(m)[:na], rng.permutation(m)[:nb]
        dets.add(sum(1 << (2 * int(i)) for i in a) | sum(2 << (2 * int(i)) for i in b))
    dets = [int(d) for d in dets]
    dets = [dets[i] for i in rng.permutation(n)]
    pop = rng.integers(1, 9, size=n) * rng.choice([-1, 1], size=n)
    return dets, pop.astype(np.int32), ref


def _array(dets, words):
    lo = np.array([d & (2**64 - 1) for d in dets], np.uint64)
    if words == 1:
        return lo
    return np.stack([lo, np.array([d >> 64 for d in dets], np.uint64)], axis=1)


def _solver(m, na, nb, **more):
    ham = S.synthetic_molecule(m, na, nb, 7)
    prm = S.Params(tau=1e-3, initiator_threshold=3, target_walkers=10**6, initial_walkers=10,
                   seed=3, **more)
    return F.Solver(ham, prm, F.current_stream()), ham, prm


@pytest.mark.parametrize("m,na,nb,words", [(9, 4, 4, 1), (20, 5, 5, 1), (30, 5, 4, 1), (9, 4, 4, 2),
                                           (36, 5, 5, 2), (64, 4, 4, 2)])
def test_read_out_sorted(m, na, nb, words):
    sv, _, _ = _solver(m, na, nb, det_words=words if 2 * m <= 64 else 0)
    rng = np.random.default_rng(m + words)
    for n in (1, 2, 63, 65, 1023, 1024, 1025, 4097, 9000):
        print(f"[gpu] lists: {m} orbitals, {words} words, {n} determinants", flush=True)
        dets, pop, ref = _lists(m, na, nb, n, rng)
        sv.load_walkers(_array(dets, words), pop)
        order = sorted(range(n), key=lambda i: dets[i])
        want = _array([dets[i] for i in order], words)
        wpop = pop[order]
        wflag = ((np.abs(wpop) > 3) | (np.array([dets[i] for i in order], object) == ref))
        det, p, f = sv.walkers()
        assert np.array_equal(det, want) and np.array_equal(p, wpop)
        assert np.array_equal(f, wflag.astype(np.uint32))
        # arrays shorter than the list take its first entries; each array may be missing
        k = max(1, n // 3)
        kd, kp = np.zeros(k * words, np.uint64), np.zeros(k, np.int32)
        fn = F.lib().fciqmc_walkers
        assert fn(sv.h, F._ptr(kd), None, None, k) == n
        assert fn(sv.h, None, F._ptr(kp), None, k) == n
        assert fn(sv.h, None, None, None, n) == n and fn(sv.h, F._ptr(kd), None, None, 0) == n
        assert np.array_equal(kd, want[:k].ravel()) and np.array_equal(kp, wpop[:k])
    sv.close()


@pytest.mark.parametrize("order", ["ascending", "drawn"])
@pytest.mark.parametrize("words", [1, 2])
def test_load(order, words):
    """Entries without walkers are left out, also when they are no determinants of the
    system or repeat others; without one on the reference it is added; the solve goes on as
    the oracle's."""
    m = 9
    sv, ham, prm = _solver(m, 3, 4, det_words=words)
    rng = np.random.default_rng(5)
    dets, pop, ref = _lists(m, 3, 4, 1500, rng)
    if order == "ascending":
        dets = sorted(dets)
    for has_ref in (True, False):
        print(f"[gpu] lists: load, {order}, {words} words, reference {has_ref}", flush=True)
        use, up = list(dets), pop.copy()
        if not has_ref:
            up[use.index(ref)] = 0
        if order == "drawn":
            use += [use[3], 0, ref, ref, 2**63 + 1]
            up = np.concatenate([up, np.zeros(5, np.int32)])
        sv.load_walkers(_array(use, words), up, iteration=4, shift=0.5)
        keep = {d: int(p) for d, p in zip(use, up) if p}
        e = sv.estimates()
        assert e["n_dets"] == len(keep) and e["n_walkers"] == sum(map(abs, keep.values()))
        assert e["ref_pop"] == keep.get(ref, 0)
        ref_run = O.Oracle(ham, prm)
        ks = sorted(keep)
        od = ref_run.walkers()[0]
        ref_run.load_walkers(_array(ks, od.ndim), np.array([keep[d] for d in ks], np.int32),
                             iteration=4, shift=0.5)
        sv.iterate(6)
        ref_run.iterate(6)
        (dg, pg, _), (do, po, _) = sv.walkers(), ref_run.walkers()
        assert np.array_equal(dg if dg.ndim == 1 else dg[:, 0], do if do.ndim == 1 else do[:, 0])
        assert np.array_equal(pg, po)
        ref_run.close()
    sv.close()


@pytest.mark.parametrize("words", [1, 2])
def test_load_refused(words):
    """What a list may not hold is named by the first entry that holds it, and a refused list
    leaves the solve as it was."""
    m = 9
    sv, _, _ = _solver(m, 3, 4, det_words=words, space=S.SPACE_EXCITATION, max_excitation=3)
    rng = np.random.default_rng(6)
    dets, pop, ref = _lists(m, 3, 4, 1200, rng)
    inside = [i for i, d in enumerate(dets) if bin(d & ~ref).count("1") <= 3]
    out = next(d for d in dets if bin(d & ~ref).count("1") > 3)
    dets, pop = [dets[i] for i in inside], pop[inside]
    sv.load_walkers(_array(dets, words), pop)
    before = sv.walkers()
    lowest = np.iinfo(np.int32).min
    bad = {"wrong electron counts": (0b111, 1), "population out of range": (dets[1], lowest),
           "outside the restricted space": (out, 2), "duplicate": (dets[7], 3)}
    for what, (d, p) in bad.items():
        for tail in ([], [(0b1, 1), (out, lowest)]):
            if tail and what == "duplicate":
                continue     # (looked for last)
            print(f"[gpu] lists: refused, {what}", flush=True)
            nd = dets + [d] + [t for t, _ in tail]
            np_ = np.concatenate([pop, np.array([p] + [q for _, q in tail], np.int32)])
            with pytest.raises(F.FciqmcError, match=what):
                sv.load_walkers(_array(nd, words), np_)
            for a, b in zip(before, sv.walkers()):
                assert np.array_equal(a, b)
    sv.close()
