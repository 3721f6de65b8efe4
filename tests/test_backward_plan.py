"""How a tower step launches its backward pass, by its sizes."""
import pytest

from paper_2201_05500_amd.binding_mlp import ctr_debug_mlp_backward_plan as plan


@pytest.mark.parametrize("in_dim,hidden,batch", [(624, [400, 200, 80], 1000), (72, [136, 64], 264), (8, [8], 8), (256, [128, 64], 4104)])
def test_a_gradient_over_the_input_waits_for_the_first_weight_gradient(in_dim, hidden, batch):
    """In one launch the two would read and write the same memory."""
    assert plan(in_dim, hidden, batch)[1][0] == 1
    kept, paired, weight_ranges, input_ranges = plan(in_dim, hidden, batch, in_place=True)
    assert paired == (0,) + plan(in_dim, hidden, batch)[1][1:]
    assert kept == 2 and min(weight_ranges + input_ranges) >= 1


@pytest.mark.parametrize("bad", [(0, [8], 8), (8, [], 8), (8, [12], 8), (8, [8], 0), (8, [8], 12), (8, [8], (1 << 20) + 8)])
def test_refused_sizes(bad):
    with pytest.raises(ValueError):
        plan(*bad)
