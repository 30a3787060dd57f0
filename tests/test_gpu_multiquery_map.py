"""Several queries per sequence: the readers of a split share an XCD.  Counts that do not divide by eight, one and two head
groups, against the oracle."""
import pytest

import test_gpu_multiquery as mq
from test_gpu_parity import shape

pytestmark = pytest.mark.gpu

MAPS = {
    "map_21_rows": (shape(64, 32, 128, 8, 1536, "bf16"), [300, 190, 77], 7, [0, 1, 3]),
    "map_two_head_groups": (shape(64, 40, 128, 8, 256, "bf16"), [260, 33, 150], 3, [0, 1, 2]),
    "map_three_head_groups": (shape(64, 72, 128, 4, 128, "bf16"), [190], 2, [0, 5]),
    # more work-groups than compute units, dealt out in runs: a prompt's own queries (with a rest behind the last turn), sequences
    # sorted by length, two head groups
    "map_own_prompt": (shape(64, 32, 128, 16, 256, "bf16"), [300], 300, [1]),
    "map_own_prompts_two_head_groups": (shape(64, 40, 128, 8, 256, "bf16"), [129, 129], 129, [1]),
    "map_sorted": (shape(64, 32, 128, 8, 256, "bf16"), [400 - 31 * i for i in range(12)], 8, [3]),
    "map_r16": (shape(64, 32, 128, 16, 1024, "bf16"), [210, 100], 2, [0, 4]),
}
mq.CASES.update(MAPS)


@pytest.mark.parametrize("name", list(MAPS))
def test_readers_of_a_split(name):
    mq.test_multiquery_matches_oracle(name)
