"""The per-group replay-forward mode rule (AUGTREE_REPLAY_AUTO): host logic
only, no GPU. Its decisions on shapes whose two modes were timed on an
MI355X (replay_fwd alone) agree with the faster mode wherever the two differ
by more than 10 %:

    heads      P      G   R      fused us  split us
    32/8/128   32768  16  16       597       525
    32/8/128   32768  16  32       605       535
    32/8/128   32768  16  64       611       575
    32/8/128   32768  16  96       770       790
    32/8/128   32768  16  128      959       982
    32/8/128   16384  32  32       611       312
    32/8/128   16384  32  64       627       512
    32/8/128   16384  32  96       776       789
    32/8/128   16384  32  160     1547      1292
    32/8/128   8192   64  8        503       149
    32/8/128   8192   64  32       633       286
    32/8/128   8192   64  200     1658      1700
    32/8/128   4096   8   4096    2927      3273
    8/2/128    8192   64  16       153       138
    28/4/128   8192   64  32       356       241
    28/4/128   8192   64  200     1380      1469
    16/4/64    16384  32  64       264       220
    16/4/64    16384  32  96       281       292
    8/8/128    8192   64  40       165       143

(8192, 64, 200) with 32 / 8 heads is a near tie the rule gives to SPLIT.
"""
import numpy as np
import pytest

from paper_2609_33133_amd import api
from paper_2609_33133_amd import inputs as I
from paper_2609_33133_amd.api import GroupBatch

TIMED = [((32768, 16, 16), 1), ((32768, 16, 64), 1), ((8192, 64, 8), 1),
         ((8192, 64, 32), 1), ((8192, 64, 200), 1), ((4096, 8, 4096), 0)]
# (hq, hkv, d), (P, G, R), split: short branches whose (row, head) pairs fill one, two or three of a tile's workgroups,
# full and ragged tiles, other head layouts
H32, H8, H28, H64, H1 = (32, 8, 128), (8, 2, 128), (28, 4, 128), (16, 4, 64), (8, 8, 128)
TIMED_PACKED = [(H32, (32768, 16, 32), 1), (H32, (32768, 16, 96), 0), (H32, (32768, 16, 128), 0),
                (H32, (16384, 32, 32), 1), (H32, (16384, 32, 64), 1), (H32, (16384, 32, 96), 0),
                (H32, (16384, 32, 160), 1), (H8, (8192, 64, 16), 1), (H28, (8192, 64, 32), 1),
                (H28, (8192, 64, 200), 0), (H64, (16384, 32, 64), 1), (H64, (16384, 32, 96), 0),
                (H1, (8192, 64, 40), 1)]


@pytest.mark.parametrize("shape,split", TIMED)
def test_rule_matches_timed_winner(shape, split):
    P, G, R = shape
    b = GroupBatch.from_shape(I.custom_shape([P], [[R] * G], 32, 8, 128))
    assert api.replay_split_groups(b).tolist() == [split]


@pytest.mark.parametrize("heads,shape,split", TIMED_PACKED)
def test_rule_counts_the_workgroups_that_run(heads, shape, split):
    P, G, R = shape
    b = GroupBatch.from_shape(I.custom_shape([P], [[R] * G], *heads))
    assert api.replay_split_groups(b).tolist() == [split]


def test_rule_is_per_group():
    s = I.custom_shape([4096, 32768, 2048], [[4096] * 8, [16] * 16, [3000, 1]], 32, 8, 128)
    got = api.replay_split_groups(GroupBatch.from_shape(s)).tolist()
    assert got[:2] == [0, 1]
    assert got[2] in (0, 1)


def test_workloads_stay_fused():
    # the headline workloads' branches are long: the rule keeps them fused
    for name in ("balanced", "prompt", "response"):
        b = GroupBatch.from_shape(I.config_shape(name))
        assert not api.replay_split_groups(b).any(), name


def test_bad_descriptor_reported():
    b = GroupBatch(np.array([0, 5], np.int32), np.array([0, 1], np.int32), np.array([0, 0], np.int32), 2, 1, 64)
    with pytest.raises(Exception):
        api.replay_split_groups(b)
