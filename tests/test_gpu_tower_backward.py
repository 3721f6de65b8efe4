"""The backward pass of a tower step, bit by bit: a step launches a layer's two products together or apart, finishes split
products at once or leaves their partial sums to the optimizer, as the sizes have it; every gradient must be the one
that the products give on their own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _product(a_kc, b_kc, A, B, M, N, K, room):
    import torch
    from paper_2201_05500_amd import binding_mlp as BM
    C = torch.empty((M, N), dtype=torch.float32, device="cuda:0")
    assert BM.ctr_mlp_gemm(a_kc, b_kc, A.data_ptr(), A.shape[1], B.data_ptr(), B.shape[1], M, N, K, C.data_ptr(), N,
                           room.data_ptr(), room.numel() * 4, torch.cuda.current_stream().cuda_stream) == 0
    return C


# tests/test_backward_plan.py says which routes these take
TOWERS = [
    # small ones (all layers paired, the weight gradients split and not), one whose first layer is not paired, one layer only,
    # and one whose partial sums do not fit beside each other
    (8, [8], 8), (72, [136, 64], 264), (624, [400, 200, 80], 1000), (256, [128, 64], 4104), (3200, [1024, 512, 256], 4096),
    (64, [72, 40, 24, 16, 8, 8], 520), (4800, [1024, 512], 16384), (2048, [4096], 2048),
    # split weight gradients of layers that are not paired, left to the optimizer; the upper layer alone not paired
    (640, [264], 16384), (64, [512, 256], 16384), (16, [1840, 1792], 1816),
    # split input gradients behind kept sums
    (64, [2048], 64), (16, [16, 1800], 8),
    # only the first layer's partial sums kept: above it unsplit weight gradients, split input gradients
    (352, [408, 1360, 128], 4184), (184, [1592, 8, 1200], 5408),
    # nothing kept: split weight gradients and not, split input gradients, of the first layer and above
    (64, [856, 424], 8032), (8, [1896, 1096], 3944), (784, [1176, 248, 128], 6000), (240, [896, 8, 1672], 6152),
    (232, [144, 1560, 544], 4776)]


@pytest.mark.parametrize("in_dim,hidden,B", TOWERS)
@pytest.mark.parametrize("grad_bf16", [False, True])
def test_gradients_are_those_of_the_products(in_dim, hidden, B, grad_bf16):
    import torch
    from paper_2201_05500_amd.binding_mlp import CtrMlp
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(in_dim + B)
    x = torch.randn((B, in_dim), generator=gen, device="cuda:0").to(torch.bfloat16)
    y = (torch.rand(B, generator=gen, device="cuda:0") < 0.3).float()
    tower = CtrMlp(in_dim, hidden, init_seed=5)
    params = torch.from_numpy(tower.export()["params"]).cuda()
    widths = [in_dim] + list(hidden) + [1]
    room = torch.empty(min(max(max(a * b for a, b in zip(widths, widths[1:-1])) * 4, 8 << 20), 128 << 20), device="cuda:0")
    W, at = [], 0
    for i, o in zip(widths, widths[1:]):
        W.append(params[at:at + i * o].view(i, o).to(torch.bfloat16).contiguous())  # biases begin at 0
        at += i * o + o
    acts = [x]
    for i, o, w in zip(widths[:-2], widths[1:-1], W):
        acts.append(_product(True, False, acts[-1], w, B, o, i, room).clamp(min=0).to(torch.bfloat16))
    st, _, got = tower.step(0, x, y, grad_pooled=torch.empty((B, in_dim), dtype=torch.bfloat16 if grad_bf16 else torch.float32,
                                                              device="cuda:0"))
    assert st == 0
    # the logits before the step
    before = CtrMlp(in_dim, hidden, init_seed=5)
    st, logits = before.forward(0, x)
    assert st == 0
    z = logits.double()
    d = ((1.0 / (1.0 + torch.exp(-z)) - y.double()) / B).float()
    dz = torch.where(acts[-1] > 0, d[:, None] * W[-1].float().view(1, -1), torch.zeros((), device="cuda:0")).to(torch.bfloat16)
    m = torch.from_numpy(tower.export()["m"]).cuda()
    starts = np.cumsum([0] + [i * o + o for i, o in zip(widths, widths[1:])])
    omb1 = 1.0 - float(np.float32(0.9))
    for l in range(len(hidden) - 1, -1, -1):
        i, o = widths[l], widths[l + 1]
        dw = _product(False, False, acts[l], dz, i, o, B, room)
        have = m[starts[l]:starts[l] + i * o].view(i, o)
        assert torch.equal(have, (omb1 * dw.double()).float()), ("weights", l)
        db = omb1 * dz.double().sum(0)
        slack = B * 2.0 ** -24 * omb1 * dz.double().abs().sum(0) + 1e-30
        assert bool(((m[starts[l] + i * o:starts[l + 1]].double() - db).abs() <= slack).all()), ("biases", l)
        dh = _product(True, True, dz, W[l], B, i, o, room)
        if l:
            dz = torch.where(acts[l] > 0, dh, torch.zeros((), device="cuda:0")).to(torch.bfloat16)
    assert torch.equal(got, dh.to(got.dtype))


# towers whose first layer is paired (the second not) when nothing overlaps; the input at the beginning, in the middle and at the
# end of what the gradient overwrites, and over its beginning and end
@pytest.mark.parametrize("in_dim,hidden,B", [(624, [400, 200, 80], 1000), (72, [136, 64], 264), (8, [8], 8), (3200, [1024, 512, 256], 4096)])
@pytest.mark.parametrize("grad_bf16", [False, True])
@pytest.mark.parametrize("at", [-0.5, 0.0, 0.5, 1.0])
def test_gradient_over_the_input(in_dim, hidden, B, grad_bf16, at):
    import torch
    from paper_2201_05500_amd.binding_mlp import CtrMlp
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(in_dim + B)
    x = torch.randn((B, in_dim), generator=gen, device="cuda:0").to(torch.bfloat16)
    y = (torch.rand(B, generator=gen, device="cuda:0") < 0.3).float()
    grad_type = torch.bfloat16 if grad_bf16 else torch.float32
    n = B * in_dim
    apart, over = CtrMlp(in_dim, hidden, init_seed=5), CtrMlp(in_dim, hidden, init_seed=5)
    st, loss, want = apart.step(0, x, y, grad_pooled=torch.empty((B, in_dim), dtype=grad_type, device="cuda:0"))
    assert st == 0
    memory = torch.zeros(4 * n, dtype=torch.bfloat16, device="cuda:0")
    begin = n if at < 0 else 0                                            # of the gradient
    put = begin + int(at * n) // 8 * 8                                    # of the input
    pooled = memory[put:put + n].view(B, in_dim)
    pooled.copy_(x)
    place = memory[begin:begin + (n if grad_bf16 else 2 * n)]
    grad = (place if grad_bf16 else place.view(torch.float32)).view(B, in_dim)
    st, over_loss, got = over.step(0, pooled, y, grad_pooled=grad)
    assert st == 0 and got.data_ptr() == grad.data_ptr()
    assert torch.equal(got, want) and torch.equal(loss, over_loss)
    a, b = apart.export(), over.export()
    assert all(np.array_equal(a[k], b[k]) for k in ("params", "m", "v"))


# one of the 16-byte aligned places, 8 bytes beside it, 2 and 14
@pytest.mark.parametrize("in_dim,hidden,B", [(624, [400, 200, 80], 1000), (8, [8], 8), (3200, [1024, 512, 256], 4096), (1600, [256, 128], 16384)])
@pytest.mark.parametrize("beside", [0, 4, 1, 7])
def test_input_at_any_alignment(in_dim, hidden, B, beside):
    import torch
    from paper_2201_05500_amd.binding_mlp import CtrMlp
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(in_dim + B)
    x = torch.randn((B, in_dim), generator=gen, device="cuda:0").to(torch.bfloat16)
    y = (torch.rand(B, generator=gen, device="cuda:0") < 0.3).float()
    memory = torch.full((x.numel() + 16,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    pooled = memory[beside:beside + x.numel()].view(B, in_dim)
    pooled.copy_(x)
    assert x.data_ptr() % 16 == 0 and pooled.data_ptr() % 16 == 2 * beside
    results = []
    for p in (x, pooled):
        tower = CtrMlp(in_dim, hidden, init_seed=5)
        st, logits = tower.forward(0, p)
        assert st == 0
        st, loss, grad = tower.step(0, p, y)
        assert st == 0
        results.append([logits, loss, grad] + [torch.from_numpy(tower.export()[k]) for k in ("params", "m", "v")])
    assert all(torch.equal(a, b) for a, b in zip(*results))
