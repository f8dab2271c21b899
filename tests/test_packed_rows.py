"""Query tiles whose 128 columns are (row, head) pairs: group sizes that do
not divide 128, row counts whose pairs end just before, at and after a
wavefront (32) and a workgroup (128), and tiles whose last workgroups are
empty, forward and backward against the oracle."""
import pytest
import torch

from paper_2609_33133_amd import inputs as I
from paper_2609_33133_amd.api import REPLAY_FUSED, REPLAY_SPLIT

from gpu_helpers import assert_close, oracle, run_shared

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (prompt lens, branch lens, hq, hkv, d): pairs per tile = rows x group
CASES = [
    ([43, 129], [[1, 10, 11, 42, 43], [127, 128]], 3, 1, 128),       # g = 3: 30, 33, 126, 129, 384 pairs
    ([127], [[4, 5, 6, 18, 19, 128]], 14, 2, 128),                   # g = 7: 28, 35, 42, 126, 133 pairs
    ([64, 65], [[2, 8, 9], [31, 32, 33, 130]], 16, 1, 64),           # g = 16: 8 rows a workgroup
    ([33], [[1, 31, 32, 33, 97, 128, 129]], 2, 2, 64),               # g = 1: a tile is one workgroup
    ([257, 70], [[1, 3, 191], [64]], 128, 1, 64),                        # g = 128: one row a workgroup
    ([20], [[1, 2, 50]], 129, 1, 64),                                # g > 128: a row spans two workgroups
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_pairs_against_oracle(case):
    ps, rs, hq, hkv, d = CASES[case]
    gi = I.make_inputs(I.custom_shape(ps, rs, hq, hkv, d), seed=300 + case, qk_mult=1.0)
    ref = oracle(gi)
    for mode in (REPLAY_FUSED, REPLAY_SPLIT):
        got, _ = run_shared(gi, mode=mode)
        assert_close(got, ref, f"pairs {case} mode {mode}")
