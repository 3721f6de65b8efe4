"""The sums over the batch of a tower step (bias gradients, the output layer's gradients, the loss) at the edges of
column tiles, row slices and the number of layers.

A sample of zeros has zero activations (biases start at 0) and passes no gradient back, so with one sample of the batch
not zero every gradient but the output bias's is that sample's, whichever row it stands in: the same bits for every
row.  The output bias's gradient is the sum of sigmoid(z) - y over the batch, of which each term but one is 1/2: exact
to a few roundings of a sum of B terms, at most B 2^-24 relative."""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("in_dim,hidden,B", [(8, [8], 8), (64, [128, 136], 72), (24, [264, 8, 120], 520),
                                             (16, [8] * 6, 1000), (64, [32], 4104), (200, [1024, 48], 64),
                                             (8, [65536, 8, 65536, 8, 65536], 8)])  # sums in more than one launch
def test_gradient_of_one_sample_is_the_same_in_every_row(in_dim, hidden, B):
    import torch
    from paper_2201_05500_amd.binding_mlp import CtrMlp
    sample = np.random.default_rng(B).standard_normal(in_dim).astype(np.float32)
    per = (B + 63) // 64
    rows = sorted({r for r in (0, 1, 7, 8, per - 1, per, B // 2, B - per, B - 1) if 0 <= r < B})
    first = None
    for r in rows:
        tower = CtrMlp(in_dim, hidden, init_seed=3)
        pooled = np.zeros((B, in_dim), np.float32)
        pooled[r] = sample
        st, loss, _ = tower.step(0, torch.from_numpy(pooled).cuda(), torch.zeros(B, device="cuda:0"))
        assert st == 0
        e = tower.export()
        tower.close()
        if first is None:
            oracle = M.MlpOracle(in_dim, hidden, init_seed=3)
            oloss, _ = oracle.step(0, pooled, np.zeros(B, np.float32))
            assert abs(float(loss.cpu()[0]) - float(oloss)) <= 1e-5 * float(oloss)
            # bf16 roundings of one sample's activations: a few times 2^-8 of its gradient
            d = np.linalg.norm(e["m"].astype(np.float64) - oracle.m[0])
            assert d <= 2e-2 * np.linalg.norm(oracle.m[0].astype(np.float64))
            first = e
        assert np.array_equal(e["m"][:-1], first["m"][:-1]), r
        assert abs(e["m"][-1] - oracle.m[0][-1]) <= (B * 2.0 ** -24 + 1e-6) * abs(oracle.m[0][-1]), r
