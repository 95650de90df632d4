"""Host checks of the attention kernel's placement (no GPU needed): every query
group of every (batch, head) pair runs once, and the XCDs' shares of the work
are even, whatever the number of pairs."""
import numpy as np
import pytest

import paper_2503_05130_amd as ie

PAIRS = [1, 2, 3, 4, 7, 8, 9, 12, 13, 16, 20, 25, 31, 64, 100, 384]
GROUPS = [1, 2, 3, 5, 8, 18, 32, 33, 64]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n_cu", [256, 64, 12])
def test_placement(causal, n_cu):
    for pairs in PAIRS:
        for groups in GROUPS:
            place = ie.test_attention_place(pairs, groups, causal, n_cu)
            xcd = np.arange(len(place)) % 8
            g, p = place.T
            assert len(g) == pairs * groups and np.unique(p * groups + g).size == len(g)
            assert 0 <= g.min() and g.max() < groups and 0 <= p.min() and p.max() < pairs
            # an XCD has at most one group's work more than an even share
            work = place[:, 0] + 1 if causal else np.ones(len(place))
            share = np.bincount(xcd, weights=work, minlength=8)
            assert share.max() <= work.sum() / 8 + work.max(), (pairs, groups)
            # where 8 divides the pairs, a pair's K and V stay in one XCD's L2
            if pairs % 8 == 0:
                assert np.array_equal(xcd, p % 8)


@pytest.mark.parametrize("pairs,groups,n_cu", [(16, 32, 256), (12, 64, 256), (9, 24, 64), (2, 64, 256)])
def test_heavy_and_light_groups_take_turns(pairs, groups, n_cu):
    """A causal grid goes heaviest first in rows of one workgroup per CU of the XCD, every other row reversed."""
    place = ie.test_attention_place(pairs, groups, True, n_cu)
    for x in range(8):
        g = place[x::8, 0]
        rows = [g[i:i + n_cu // 8] for i in range(0, len(g), n_cu // 8)]
        for i, row in enumerate(rows):
            assert np.all(np.diff(row[::-1] if i % 2 else row) <= 0)
        for a, b in zip(rows, rows[1:]):
            assert a.min() >= b.max()


def test_bad_arguments():
    for args in [(0, 1, True, 256), (1, 0, True, 256), (1, 1, True, 0), (65536, 1, False, 256), (1, 1025, False, 256)]:
        with pytest.raises(ie.IefwdError) as e:
            ie.test_attention_place(*args)
        assert e.value.status == ie.EINVAL
