"""How a tower step launches its backward pass, by its sizes."""
import pytest

from paper_2201_05500_amd.binding_mlp import ctr_debug_mlp_backward_plan as plan
from tests.test_gpu_tower_backward import TOWERS


@pytest.mark.parametrize("in_dim,hidden,batch", [(624, [400, 200, 80], 1000), (72, [136, 64], 264), (8, [8], 8), (256, [128, 64], 4104)])
def test_a_gradient_over_the_input_waits_for_the_first_weight_gradient(in_dim, hidden, batch):
    """In one launch the two would read and write the same memory."""
    assert plan(in_dim, hidden, batch)[1][0] == 1
    kept, paired, weight_ranges, input_ranges = plan(in_dim, hidden, batch, in_place=True)
    assert paired == (0,) + plan(in_dim, hidden, batch)[1][1:]
    assert kept == 2 and min(weight_ranges + input_ranges) >= 1


def test_towers_compared_bit_by_bit_take_every_route():
    """(kept, first layer or above, paired, weight gradient split, input gradient split) of each layer: a change of the cost
    rule must not drop a route from the GPU test unnoticed."""
    taken = set()
    for tower in TOWERS:
        kept, *layers = plan(*tower)
        taken |= {(kept, l > 0, bool(p), w > 1, i > 1) for l, (p, w, i) in enumerate(zip(*layers))}
    no, yes = False, True
    paired = {(2, up, yes, split, no) for up in (no, yes) for split in (no, yes)}
    kept = {(2, up, no, *split) for up in (no, yes) for split in ((no, no), (no, yes), (yes, no))}
    first_kept = {(1, no, no, yes, no), (1, yes, no, no, no), (1, yes, no, yes, no), (1, yes, no, yes, yes)}
    nothing_kept = {(0, up, no, *split) for up in (no, yes) for split in ((no, no), (yes, no), (yes, yes))}
    assert taken >= paired | kept | first_kept | nothing_kept


@pytest.mark.parametrize("bad", [(0, [8], 8), (8, [], 8), (8, [12], 8), (8, [8], 0), (8, [8], 12), (8, [8], (1 << 20) + 8)])
def test_refused_sizes(bad):
    with pytest.raises(ValueError):
        plan(*bad)
