"""The interaction counts of the FP64 walk in rounds with each number of waves
and workgroups per item, at the sizes where they change: an entry dropped or
counted twice where workgroups share an item would show."""
import pytest

from paper_1110_4876_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    # sixteen waves: four workgroups an item up to 32 items, two up to 128,
    # whole items to 256, then the last four of each eighth shared by two
    ("items_33", lambda: inputs.plummer(32 * 64 + 1, seed=1, quadrupole=True, theta=0.6), 1, 0.0),
    ("items_128", lambda: inputs.sheet(128 * 64, seed=2, theta=0.6), 1, 500.0),
    ("items_129", lambda: inputs.sheet(128 * 64 + 1, seed=2, theta=0.6), 4, 500.0),
    ("items_257", lambda: inputs.plummer(256 * 64 + 1, seed=3, theta=0.7), 1, 0.0),
    ("items_400", lambda: inputs.sheet(400 * 64 - 5, seed=4, theta=0.7), 1, 1234.5),
    ("waves16_543_items", lambda: inputs.plummer(543 * 64, seed=5, theta=0.8), 1, 0.0),
    # eight waves, the last eight shared
    ("waves8_544_items", lambda: inputs.plummer(543 * 64 + 1, seed=5, theta=0.8), 1, 0.0),
    ("waves8_1000_items", lambda: inputs.sheet(1000 * 64 - 1, seed=6, theta=0.8), 8, 1234.5),
]


@pytest.mark.parametrize("name,maker,leaf,t", CASES, ids=[c[0] for c in CASES])
def test_counts_match_oracle(orc, name, maker, leaf, t):
    # (forces to 1e-12 of the rms as for the walk's other schedules, and the
    # oracle's counts exactly)
    from test_gpu_walk_rounds import test_rounds_match_oracle
    test_rounds_match_oracle(orc, name, maker, leaf, t, 0)
