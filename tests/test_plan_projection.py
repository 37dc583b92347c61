"""How projection tiles are dealt to the XCDs (CPU only): every tile once, and the full rounds of a first launch are full rounds
on the XCD that gets the most tiles, too."""
import pytest

from plan_lib import projection_first_features, projection_group, projection_tiles

KINDS = [(256, 256, 1), (128, 128, 2), (128, 128, 1), (128, 64, 1), (64, 64, 2), (64, 32, 2), (32, 32, 2)]


def deal(m, n, m_per):
    """tiles per XCD by the kernels' rule: workgroup ids go to the eight XCDs in turn"""
    m_groups = -(-m // m_per)
    xcds = [[] for _ in range(8)]
    for block in range(8 * m_per * (-(-m_groups * n // 8))):
        grp = block // 8 // m_per * 8 + block % 8
        tm, tn = grp % m_groups * m_per + block // 8 % m_per, grp // m_groups
        if tm < m and tn < n:
            xcds[block % 8].append((tm, tn))
    return xcds


@pytest.mark.parametrize("tokens,hidden_in,features", [(2772, 7040, 6656), (5488, 4416, 3712), (2641, 3392, 6784), (4096, 8192, 6144),
                                                       (1219, 7424, 6784), (1, 64, 384), (6260, 3136, 5760), (8192, 8192, 9216)])
def test_tiles_are_dealt_once_and_evenly(tokens, hidden_in, features):
    first, *second = projection_tiles(tokens, hidden_in, features)
    f_first = projection_first_features(tokens, hidden_in, features)
    for i, (tile, f) in enumerate([(first, f_first)] + [(t, features - f_first) for t in second]):
        m, n = -(-tokens // tile[0]), -(-f // tile[1])
        xcds = deal(m, n, projection_group(tokens, KINDS.index(tile), f))
        assert sorted(t for x in xcds for t in x) == [(tm, tn) for tm in range(m) for tn in range(n)]
        if second and i == 0:
            slots = 32 * tile[2]
            rounds = -(-m * n // (8 * slots))
            assert max(map(len, xcds)) <= rounds * slots, (tile, m, n, rounds)
