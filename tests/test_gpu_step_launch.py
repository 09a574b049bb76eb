"""A step in one launch (attention, instruction score and the eviction by it) at the edges of its forms: one strip of instruction rows
and several, both numbers of key tiles, the most candidates, first steps that keep everything and first steps that evict.  The same
bits as the launches apart, twice over one workspace; a second document of another size on it finds its counters as it needs them."""

import pytest

import paper_2406_12018_amd as api
from test_gpu_fused_launches import test_merged_launches_give_the_bits_of_the_launches_apart as same_bits

pytestmark = pytest.mark.gpu

# dtype, L, Hq, Hkv, d, chunk, T, budget, instruction rows, options
CASES = [
    ("bf16", 1, 4, 4, 128, 64, 300, 100, 32, {}),               # one strip of 32 rows per head
    ("bf16", 1, 8, 4, 64, 130, 700, 129, 17, {}),               # two strips, the second of two rows; the first step evicts
    ("bf16", 1, 32, 8, 128, 100, 500, 37, 64, {}),              # eight strips
    ("bf16", 2, 16, 2, 128, 33, 200, 400, 70, {}),              # nothing is evicted
    ("bf16", 1, 8, 2, 128, 500, 2100, 780, 40, {}),             # 1280 candidates
    ("bf16", 1, 8, 2, 64, 500, 2100, 781, 40, {}),              # 1281
    ("bf16", 1, 4, 1, 64, 700, 4000, 1860, 30, dict(start_size=3)),  # 2560, the most
    ("bf16", 1, 8, 1, 128, 200, 1100, 300, 21, dict(score_mode=api.SCORE_ACCUMULATED)),  # sums of the first step are carried on
    ("bf16", 3, 8, 2, 128, 96, 500, 150, 16, dict(position_shift=1)),
    ("bf16", 1, 21, 3, 128, 150, 900, 200, 33, {}),             # eight strips of each of three units: over all XCDs
    ("bf16", 5, 20, 5, 64, 100, 700, 130, 40, {}),
    ("bf16", 16, 8, 4, 64, 98, 500, 65, 40, {}),                # 256 workgroups of the attention behind 192 of the score
    ("bf16", 1, 128, 32, 128, 64, 300, 70, 96, {}),             # 384 strips of 32 rows would be more than the compute units: 64 rows each
    ("bf16", 1, 64, 8, 128, 512, 2000, 768, 192, {}),           # the same, 1280 candidates
    ("bf16", 33, 16, 4, 64, 32, 150, 60, 12, {}),               # one strip of 64 rows per unit, 48 of them there
    ("bf16", 1, 48, 6, 64, 256, 1100, 700, 256, dict(position_shift=1)),
    ("f32", 1, 4, 1, 64, 32, 300, 64, 8, {}),
    ("f32", 2, 4, 2, 128, 60, 300, 125, 9, dict(start_size=2)),
    ("f32", 1, 2, 2, 64, 212, 900, 300, 30, dict(score_mode=api.SCORE_ACCUMULATED)),  # 512 candidates, 150 KB kept: gather apart
    ("f32", 1, 2, 1, 128, 20, 90, 200, 16, dict(position_shift=1)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c[:9]))
def test_step_in_one_launch(case):
    same_bits(case)
    same_bits(case)
