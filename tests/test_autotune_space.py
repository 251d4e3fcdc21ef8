"""The tuner times no setting twice under two names (CPU)."""

from paper_2605_04864_amd import _lib as L
from paper_2605_04864_amd import autotune


def test_values_the_tuner_times():
    space = autotune.search_space((1, 4))
    assert list(space) == ["streams", *autotune.KNOB_ORDER] and space["streams"] == [1, 4]
    assert space["sort_fused"] == [0, 1]  # 2 takes the same passes as 0
    for k in autotune.KNOB_ORDER:
        assert space[k][0] == 0 and len(set(space[k])) == len(space[k])
        assert set(space[k]) <= set(L.TUNE[k][1])


def test_sort_fused_2_is_still_accepted():
    try:
        autotune.set_knobs({"sort_fused": 2})
        assert autotune.get_knobs()["sort_fused"] == 2
    finally:
        autotune.reset_knobs()
