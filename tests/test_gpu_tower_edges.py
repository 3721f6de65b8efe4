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
                                             (8, [65536, 8, 65536, 8, 65536], 8),   # sums in more than one launch
                                             (32, [504], 72), (32, [512], 72), (32, [520], 8), (16, [64, 1544], 136)])
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


@pytest.mark.parametrize("kstep", [False, True])
@pytest.mark.parametrize("width", [1024, 1032])  # a remainder of 1 parameter behind the groups of 4; widths on both sides
def test_dense_step_of_large_towers(width, kstep):
    """Towers of 2.1 M parameters and more update 4 parameters per thread.  From the moments a step left, its model
    step follows in binary64, rounded once: x - lr m / sqrt(den), with the tower's own second moment, the shared
    denominator of the k-step method, or (merge step) not at all; and the bf16 copy that the products read is the
    rounded parameter."""
    import torch
    from paper_2201_05500_amd.binding import CTR_OK, CTR_STEP_LOCAL, CTR_STEP_MERGE_PENDING
    from paper_2201_05500_amd.binding_mlp import CtrMlp
    in_dim, B, W, lr, b1, b2 = 2048, 64, 2 if kstep else 1, 1e-3, 0.9, 0.999
    tower = CtrMlp(in_dim, [width], init_seed=4, n_replicas=W, kstep=kstep, lr=lr, beta1=b1, beta2=b2)
    assert tower.n_params >= 4 * 256 * 2048 and tower.n_params % 4 == 1
    f32 = lambda a: np.float64(np.float32(a))
    rng = np.random.default_rng(width)
    ran = {CTR_STEP_LOCAL: 0, CTR_STEP_MERGE_PENDING: 0}
    for step in range(4):
        mode = CTR_STEP_MERGE_PENDING if kstep and step % 2 else CTR_STEP_LOCAL
        for r in range(W):
            before = tower.export(r)
            pooled = torch.from_numpy(rng.standard_normal((B, in_dim)).astype(np.float32) * np.float32(0.1)).cuda()
            labels = torch.from_numpy((rng.random(B) < 0.3).astype(np.float32)).cuda()
            st, _, _ = tower.step(r, pooled, labels, mode=mode)
            assert st == CTR_OK
            after = tower.export(r)
            ran[mode] += 1
            m0, v0, m, v = (a.astype(np.float64) for a in (before["m"], before["v"], after["m"], after["v"]))
            # m and v were made from one gradient: from m's, to a rounding of m, follows v
            g = (m - f32(b1) * m0) / (1.0 - f32(b1))
            slack = 2.0 ** -23 * (np.abs(m) + np.abs(m0)) / (1.0 - f32(b1))   # of g
            want = f32(b2) * v0 + (1.0 - f32(b2)) * g * g
            assert (np.abs(v - want) <= 2.0 ** -22 * want + (1.0 - f32(b2)) * (2 * np.abs(g) * slack + slack * slack)).all()
            assert np.count_nonzero(g) > 0.2 * g.size
            if mode == CTR_STEP_MERGE_PENDING:
                assert np.array_equal(after["params"], before["params"])
            else:
                den = before["vhat"].astype(np.float64) if kstep else v
                x = before["params"].astype(np.float64) - f32(lr) * m / np.sqrt(den)
                # binary64, rounded once: the last bit of a rounding that falls between two values
                assert (np.abs(after["params"] - x) <= 2.0 ** -24 * np.abs(x) * (1 + 1e-6) + 1e-45).all()
            st, logits = tower.forward(r, pooled)
            assert st == CTR_OK
            assert tower.load(r, params=after["params"], pending=mode == CTR_STEP_MERGE_PENDING) == CTR_OK
            st, again = tower.forward(r, pooled)
            assert st == CTR_OK and torch.equal(logits, again)
        if kstep and step % 2:
            assert tower.kstep_merge() == CTR_OK
    assert ran[CTR_STEP_LOCAL] >= 4 and (not kstep or ran[CTR_STEP_MERGE_PENDING] == 4)


@pytest.mark.parametrize("width,B,most_us", [(65536, 512, 450), (16384, 8, 130)])
def test_step_of_a_wide_last_layer(width, B, most_us):
    """One wave per sample walks the last hidden layer forward and back: 8 columns per lane and request, or its chain
    is the step (measured 250 and 82 us; 919 and 187 with a column per lane and request)."""
    import torch
    from paper_2201_05500_amd.binding_mlp import CtrMlp
    t = CtrMlp(64, [width])
    x = torch.randn((B, 64), device="cuda:0").to(torch.bfloat16)
    y, g, loss = torch.zeros(B, device="cuda:0"), torch.empty((B, 64), device="cuda:0"), torch.empty(1, device="cuda:0")
    took = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            assert t.step(0, x, y, grad_pooled=g, loss=loss)[0] == 0
        b.record()
        torch.cuda.synchronize()
        took.append(a.elapsed_time(b) * 200.0)
    assert sorted(took)[3] <= most_us, took
