"""Performance cases: what a user of the library has it do, through its public calls.

A case is a dict of plain values:

  kind       "iterate"     a running solve advanced by `iters` iterations, then its
                           estimates and the log of those iterations
             "solve"       one whole solve of a small system: create, iterate, read the
                           estimates and the walker list, free
             "batch"       `systems` independent solves of ragged sizes in one handle,
                           advanced together
             "serve"       a burst of requests through the continuous-batching server
             "checkpoint"  the walker list of a running solve read out and loaded back
  shape      "ring" (Hubbard ring at half filling, plain FCIQMC), "mol" (synthetic
             molecule, initiator rule) or "band" (24 electrons in 30 orbitals with a
             12-orbital band at the Fermi level, initiator rule)
  orbitals, electrons, walkers, iters
  spin       1: spin-coupled functions (even S)
  level      > 0: the space truncated at that excitation level
  irreps     > 1: an abelian point group with that many labels

Every Hamiltonian and random-number key is drawn from the seed. A state's walkers are
grown on the GPU the way a program does it: from walkers on the reference at a raised
shift, then with the shift varying.
"""
import math

import numpy as np

from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import serve
from paper_1305_6981_amd import systems as S

# Estimates that describe the state (the others are times and table layout).
ESTIMATES = ("iteration", "n_walkers", "n_dets", "ref_pop", "attempts", "spawns", "merged",
             "aborted", "born", "total_attempts", "total_spawns", "n_samples", "n_var", "n_prev",
             "shift", "e_ref", "p_double", "proj_num", "e_proj_inst", "e_proj_mean",
             "e_proj_err", "shift_mean", "shift_err", "shift_varying", "status")


def _case(name, kind, shape, orbitals, electrons, walkers, iters, **more):
    c = {"kind": kind, "shape": shape, "orbitals": orbitals, "electrons": electrons,
         "walkers": walkers, "iters": iters, "spin": 0, "level": 0, "irreps": 1, "systems": 1}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A program that looks at the estimates after every iteration of a small solve:
        # the smallest call, all latency.
        _case("ring8_step", "iterate", "ring", 8, 8, 10_000, 1),
        # A small solve from start to end, as a test or a scan over U/t runs it.
        _case("ring8_solve", "solve", "ring", 8, 8, 10_000, 256),
        # An ordinary lattice solve on one GPU: plain FCIQMC, single excitations only, the
        # shift updated every iteration.
        _case("ring14", "iterate", "ring", 14, 14, 300_000, 64),
        # The 10-electron molecule at its full walker number.
        _case("mol20_1e7", "iterate", "mol", 20, 10, 10_000_000, 64),
        # The transition-metal-dimer shape at a serving size.
        _case("band30_3e6", "iterate", "band", 30, 24, 3_000_000, 64),
        # The same at the headline size.
        _case("band30_1e8", "iterate", "band", 30, 24, 100_000_000, 32),
        # Spin-coupled functions: the general spawning path, with a second element per attempt.
        _case("band30_spin", "iterate", "band", 30, 24, 10_000_000, 32, spin=1),
        # More than 64 spin orbitals: two-word determinants.
        _case("mol36_two_words", "iterate", "mol", 36, 10, 2_000_000, 64),
        # A point group and a truncated space (CISDTQ).
        _case("mol20_group_level4", "iterate", "mol", 20, 10, 1_000_000, 64, irreps=4, level=4),
        # 64 independent solves in one handle, rings and molecules of ragged sizes.
        _case("batch64", "batch", "mix", 26, 14, 1_000_000, 32, systems=64),
        # A burst of requests served by continuous batching: admission, shared launches,
        # retirement, walker lists returned.
        _case("serve12", "serve", "mix", 20, 10, 300_000, 128, systems=12),
        # A checkpoint written and read back.
        _case("checkpoint_1e6", "checkpoint", "band", 30, 24, 2_000_000, 0),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("iterate", "step", "solve", "batch", "serve", "checkpoint"),
                       (10, 2, 2, 2, 1, 2))[0]
    shape = rng.choice(("ring", "mol", "mol", "band"))
    if kind == "batch":
        return _case(None, "batch", "mix", 26, 14, _log_uniform(rng, 50_000, 1_000_000),
                     rng.randint(8, 32), systems=rng.randint(2, 64))
    if kind == "serve":
        return _case(None, "serve", "mix", 20, 10, _log_uniform(rng, 20_000, 300_000),
                     rng.randint(40, 128), systems=rng.randint(3, 12))
    if kind == "checkpoint":
        return _case(None, "checkpoint", "band", 30, 24, _log_uniform(rng, 20_000, 2_000_000), 0)
    if kind == "solve":
        sites = 2 * rng.randint(3, 5)
        return _case(None, "solve", "ring", sites, sites, _log_uniform(rng, 2_000, 50_000),
                     rng.randint(64, 256))
    iters = rng.randint(1, 3) if kind == "step" else rng.randint(16, 64)
    if shape == "ring":
        sites = 2 * rng.randint(3, 8)
        hi = 40_000 if sites < 10 else 1_000_000
        return _case(None, "iterate", "ring", sites, sites, _log_uniform(rng, 3_000, hi), iters)
    if shape == "band":
        return _case(None, "iterate", "band", 30, 24, _log_uniform(rng, 300_000, 40_000_000),
                     min(iters, 32), spin=rng.choice((0, 0, 1)), level=0)
    orbitals = rng.randint(14, 40)
    spin, level, irreps = rng.choice(((0, 0, 1), (0, 0, 1), (0, 0, 4), (0, 4, 1), (1, 0, 1)))
    return _case(None, "iterate", "mol", orbitals, 2 * rng.randint(4, 6),
                 _log_uniform(rng, 20_000, 10_000_000 if orbitals <= 32 else 3_000_000), iters,
                 spin=spin, level=level, irreps=irreps)


# ---------------------------------------------------------------------------


def _system(case, seed):
    """(Hamiltonian, parameters, growth shift) of a case's system."""
    rng = np.random.default_rng([5, seed])
    key = int(rng.integers(1, 1 << 40))
    hseed = int(rng.integers(1, 1 << 30))
    m, ne, walkers = case["orbitals"], case["electrons"], case["walkers"]
    more = dict(target_walkers=walkers, seed=key, avg_start=0, hphf=case["spin"],
                space=S.SPACE_EXCITATION if case["level"] else 0, max_excitation=case["level"])
    if case["shape"] == "ring":
        ham = S.hubbard_ring(m, float(rng.uniform(2.0, 8.0)))
        return ham, S.Params(tau=0.01, shift_update_every=1, initial_walkers=max(10, walkers // 4),
                             **more), 0.0
    if case["shape"] == "band":
        ham = S.synthetic_molecule(m, ne // 2, ne // 2, hseed, orb_energy=S.band_energies(m))
        return ham, S.Params(tau=5e-4, shift_damping=0.5, initiator_threshold=3,
                             initial_walkers=max(100, walkers // 1000), **more), 40.0
    irr = None
    if case["irreps"] > 1:
        irr = rng.integers(0, case["irreps"], size=m)
    ham = S.synthetic_molecule(m, ne // 2, ne // 2, hseed, irreps=irr)
    return ham, S.Params(tau=1e-3, shift_damping=0.5, initiator_threshold=3,
                         initial_walkers=max(100, walkers // 20), **more), 10.0


def _grown(case, seed):
    """A running solve at its walker number, the shift varying."""
    ham, prm, raised = _system(case, seed)
    prm.initial_shift = raised
    sv = F.Solver(ham, prm, F.current_stream())
    done = 0
    while done < 4000:
        e = sv.estimates()
        if e["n_walkers"] >= prm.target_walkers:
            break
        n = 20 if e["n_walkers"] * 4 < prm.target_walkers else 4
        sv.iterate(n)
        done += n
    if raised > 0.0:
        e = sv.estimates()
        sv.set_shift(e["proj_num"] / e["ref_pop"] if e["ref_pop"] else 0.0, 1)
    for _ in range(4):
        sv.iterate(32)
    return sv


class _Batch:
    """A batch handle, freed with its owner."""

    def __init__(self, hams, prms):
        self.n = len(hams)
        self.h = F.fciqmc_batch_create(self.n, hams, prms, F.current_stream())

    def __del__(self):
        try:
            F.fciqmc_free(self.h)
        except Exception:
            pass


def _mix(n, walkers, seed):
    """Ragged independent solves: rings of 10-16 sites and molecules from 10 electrons in 16
    orbitals to 14 in 26, walker targets log-uniform over two decades up to `walkers`."""
    rng = np.random.default_rng([6, seed])
    hams, prms = [], []
    for i in range(n):
        target = int(round(walkers * 10 ** rng.uniform(-2.0, 0.0)))
        key = int(rng.integers(1, 1 << 40))
        if i % 2 == 0:
            hams.append(S.hubbard_ring(int(rng.choice([10, 12, 14, 16])), float(rng.uniform(2.0, 8.0))))
            prms.append(S.Params(tau=0.01, shift_update_every=1, target_walkers=target,
                                 initial_walkers=max(10, target // 4), seed=key))
        else:
            m, ne = int(rng.integers(16, 27)), 2 * int(rng.integers(5, 8))
            hams.append(S.synthetic_molecule(m, ne // 2, ne // 2, int(rng.integers(1, 1 << 30))))
            prms.append(S.Params(tau=1e-3, initiator_threshold=3, target_walkers=target,
                                 initial_walkers=max(10, target // 4), seed=key))
    return hams, prms


def _requests(n, walkers, iters, seed):
    """Requests of the serving shapes: the 8-site ring and the 10-electron molecule, each
    starting with half its walker target on the reference."""
    rng = np.random.default_rng([7, seed])
    out = []
    for i in range(n):
        target = int(round(walkers * 10 ** rng.uniform(-1.5, 0.0)))
        key = int(rng.integers(1, 1 << 40))
        if rng.integers(0, 2) == 0:
            ham = S.hubbard_ring(8, float(rng.uniform(2.0, 8.0)))
            prm = S.Params(tau=0.01, shift_update_every=1, target_walkers=target,
                           initial_walkers=max(10, target // 2), seed=key)
        else:
            ham = S.synthetic_molecule(20, 5, 5, int(rng.integers(1, 1 << 30)))
            prm = S.Params(tau=1e-3, initiator_threshold=3, target_walkers=target,
                           initial_walkers=max(10, target // 2), seed=key)
        out.append(serve.Request(ham, prm, 0.0, int(iters), i))
    return out


class _Lists:
    """Arrays that walker lists are collected in (unused entries are zero), as a program
    that keeps snapshots of one size holds them."""

    def __init__(self, cap):
        self.det = np.zeros(cap, np.int64)
        self.pop = np.zeros(cap, np.int32)
        self.flags = np.zeros(cap, np.int32)

    def collect(self, lists):
        n = 0
        for det, pop, flags in lists:
            m = n + len(det)
            self.det[n:m] = det.view(np.int64)
            self.pop[n:m] = pop
            self.flags[n:m] = flags.view(np.int32)
            n = m
        return {"n": n, "det": self.det, "pop": self.pop, "flags": self.flags}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        ham, prm, _ = _system(case, seed)
        return {"case": case, "ham": ham, "prm": prm,
                "lists": _Lists(_dimension(case["orbitals"], case["electrons"]))}
    if kind == "batch":
        b = _Batch(*_mix(case["systems"], case["walkers"], seed))
        for _ in range(4):
            F.fciqmc_batch_iterate(b.h, case["iters"])
        return {"case": case, "batch": b}
    if kind == "serve":
        return {"case": case, "lists": _Lists(case["systems"] * case["walkers"]),
                "requests": _requests(case["systems"], case["walkers"], case["iters"], seed)}
    if kind == "checkpoint":
        return {"case": case, "solver": _grown(case, seed), "lists": _Lists(2 * case["walkers"])}
    return {"case": case, "solver": _grown(case, seed)}


def _numbers(e):
    return {k: e[k] for k in ESTIMATES}


def _log(h, last, n):
    recs = F.fciqmc_history(h, 0, last - n + 1, n)
    return {k: np.array([r[k] for r in recs]) for k in recs[0]}


def run(state):
    case = state["case"]
    kind, n = case["kind"], case["iters"]
    if kind == "iterate":
        sv = state["solver"]
        sv.iterate(n)
        e = sv.estimates()
        return {"estimates": _numbers(e), "log": _log(sv.h, e["iteration"], n) if n > 3 else None}
    if kind == "solve":
        sv = F.Solver(state["ham"], state["prm"], F.current_stream())
        sv.iterate(n)
        e = sv.estimates()
        out = state["lists"].collect([sv.walkers()])
        sv.close()
        out["estimates"] = _numbers(e)
        return out
    if kind == "batch":
        b = state["batch"]
        F.fciqmc_batch_iterate(b.h, n)
        es = [F.fciqmc_batch_slot_estimators(b.h, i) for i in range(b.n)]
        return {k: np.array([e[k] for e in es]) for k in ESTIMATES}
    if kind == "serve":
        server = serve.SolveServer(max_slots=8, chunk_iters=64, tol=1e-3, min_samples=256,
                                   keep_walkers=True)
        res = sorted(server.run(state["requests"]).results, key=lambda r: r.tag)
        out = {k: np.array([float(getattr(r, k)) for r in res])
               for k in ("e_proj", "e_proj_err", "shift_energy")}
        out.update({k: np.array([int(getattr(r, k)) for r in res])
                    for k in ("iterations", "attempts", "converged", "failed")})
        out.update(state["lists"].collect([r.walkers for r in res]))
        return out
    # checkpoint: read out, load back (what a restart does), return what was written
    sv = state["solver"]
    e = sv.estimates()
    det, pop, flags = sv.walkers()
    sv.load_walkers(det, pop, iteration=e["iteration"], shift=e["shift"], n_prev=e["n_prev"],
                    varying=e["shift_varying"], n_var=e["n_var"])
    return state["lists"].collect([(det, pop, flags)])


def _dimension(m, ne):
    return math.comb(m, ne // 2) ** 2


def work(case):
    """One pass: per iteration, every occupied determinant's entry (20 bytes) read and its
    population (4) written, one spawn record (16 bytes) written and read for each of the
    few per cent of attempts that spawn; 252 operations per attempt (random numbers,
    excitation, matrix element, acceptance) and 77 per determinant (death)."""
    m, ne, w = case["orbitals"], case["electrons"], case["walkers"]
    if case["kind"] in ("batch", "serve"):
        w = case["systems"] * w * 0.2
        dets = 0.2 * w
    else:
        dets = min(0.5 * w, _dimension(m, ne))
    if case["kind"] == "checkpoint":
        # 16 bytes per determinant out, 12 in and 20 written to the list
        return {"bytes": 48.0 * dets, "flops": float(ne * ne) * dets}
    it = case["iters"]
    return {"bytes": it * (24.0 * dets + 32.0 * 0.03 * w), "flops": it * (252.0 * w + 77.0 * dets)}


def _reference_energy(ham):
    """<D0|H|D0> in float64 from the integrals."""
    occ = [p for p in range(2 * ham.n_orb) if (int(ham.ref_det) >> p) & 1]

    def tri(i, j):
        return i * (i + 1) // 2 + j if i >= j else j * (j + 1) // 2 + i

    def eri(p, q, r, s):
        return ham.eri[tri(tri(p >> 1, q >> 1), tri(r >> 1, s >> 1))]

    terms = [ham.e_core] + [ham.h1[p >> 1, p >> 1] for p in occ]
    for i, p in enumerate(occ):
        for q in occ[i + 1:]:
            terms.append(eri(p, p, q, q) - (eri(p, q, q, p) if (p ^ q) & 1 == 0 else 0.0))
    return math.fsum(terms)


def _p_double(ham):
    """Allowed doubles over all allowed excitations of the reference."""
    if ham.p_double >= 0.0:
        return float(ham.p_double)
    irr = np.zeros(ham.n_orb, int) if ham.orb_irrep is None else np.asarray(ham.orb_irrep, int)
    n = 2 * ham.n_orb
    occ = [p for p in range(n) if (int(ham.ref_det) >> p) & 1]
    emp = [p for p in range(n) if not (int(ham.ref_det) >> p) & 1]
    label = [(int(irr[p >> 1]), p & 1) for p in range(n)]

    def pairs(orbs):
        c = {}
        for i, p in enumerate(orbs):
            for q in orbs[i + 1:]:
                k = (label[p][0] ^ label[q][0], label[p][1] + label[q][1])
                c[k] = c.get(k, 0) + 1
        return c

    singles = sum(label[p] == label[a] for p in occ for a in emp)
    po, pe = pairs(occ), pairs(emp)
    doubles = sum(v * pe.get(k, 0) for k, v in po.items())
    return doubles / (singles + doubles)


def exact(case, seed):
    """The outputs that follow from the inputs alone: the reference energy and the share of
    double excitations (the rest is the random walk itself, whole numbers mostly)."""
    kind = case["kind"]
    if kind in ("iterate", "solve"):
        ham = _system(case, seed)[0]
        est = {k: None for k in ESTIMATES}
        est["e_ref"], est["p_double"] = _reference_energy(ham), _p_double(ham)
        if kind == "solve":
            return {"estimates": est, "n": None, "det": None, "pop": None, "flags": None}
        return {"estimates": est, "log": None}
    if kind == "batch":
        hams = _mix(case["systems"], case["walkers"], seed)[0]
        out = {k: None for k in ESTIMATES}
        out["e_ref"] = np.array([_reference_energy(h) for h in hams])
        out["p_double"] = np.array([_p_double(h) for h in hams])
        return out
    return None
