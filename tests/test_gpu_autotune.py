"""Autotuning that fails leaves the launch shape as it was."""
import pytest

from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

pytestmark = pytest.mark.gpu


def test_failed_trial_restores_the_launch_shape():
    """At tau (H_ii - E_0 - S) = 1 every walker on the reference dies in the first iteration,
    so the first trial stops with an error."""
    ham = S.synthetic_molecule(4, 2, 2, 53)
    prm = S.Params(tau=0.01, target_walkers=10**9, initial_walkers=50, initial_shift=-100.0, seed=3)
    ham.h1 *= 0.0
    ham.eri *= 0.0
    print("[gpu] autotune: a trial that fails", flush=True)
    sv = F.Solver(ham, prm, F.current_stream())
    before = F.fciqmc_get_launch(sv.h)
    with pytest.raises(F.FciqmcError) as e:
        F.fciqmc_autotune(sv.h, 1)
    assert e.value.code == -5
    assert F.fciqmc_get_launch(sv.h) == before
    sv.close()
