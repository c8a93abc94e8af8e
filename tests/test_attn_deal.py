"""How the work items of a bf16 self-attention, longest first, are dealt to the eight XCDs (block b runs on XCD b mod 8)."""
import pytest

import paper_2501_09253_amd as ps


def _dealt(items, group):
    blocks = 8 * group * -(-items // (8 * group))
    return [ps.lib().pserve_test_attn_item(b, group) for b in range(blocks)]


@pytest.mark.parametrize("group", [1, 3, 8])
@pytest.mark.parametrize("items", [1, 40, 64, 65, 520, 1160])
def test_every_item_once(items, group):
    dealt = _dealt(items, group)
    assert sorted(dealt) == list(range(len(dealt)))


@pytest.mark.parametrize("group", [1, 3, 8])
@pytest.mark.parametrize("rounds", [2, 8])
def test_equal_shares_of_falling_cost(rounds, group):
    """Over two rounds every XCD gets the same (dealt one way, the first one gets more than the last in every round)."""
    items = 8 * group * rounds
    dealt = _dealt(items, group)
    assert len({sum(items - it for it in dealt[x::8]) for x in range(8)}) == 1
