"""The tuner's candidate lists (no GPU): no two entries of a list are the same launches."""
import pytest

from paper_2301_02387_amd import tune

# schedule bits that the library accepts without effect (mh.h, mh_tune)
POISSON_IDLE, ORBITAL_IDLE = 8, 4


@pytest.mark.parametrize("name,idle", [("POI_CANDIDATES", POISSON_IDLE), ("POI_CANDIDATES_WIDE", POISSON_IDLE),
                                       ("POI_CANDIDATES_BATCH", POISSON_IDLE), ("ORB_CANDIDATES", ORBITAL_IDLE),
                                       ("ORB_CANDIDATES_BATCH", ORBITAL_IDLE)])
def test_candidates_are_different_launches(name, idle):
    """A bit without effect is set in none, so equal launches are timed once and
    the schedule that is reported holds only choices that were made."""
    cands = getattr(tune, name)
    assert all(not sched & idle for sched, _ in cands)
    # long rows by waves with bit 5 whatever bit 2 says
    keys = [(sched | 4 if sched & 32 else sched, grid) for sched, grid in cands]
    assert len(set(keys)) == len(keys)
