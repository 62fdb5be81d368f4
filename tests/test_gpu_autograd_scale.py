"""The fused wrapper's dW: the one pass that scales and rounds it against the two torch operations, to the bit, over
sizes with and without a remainder, special values, and the forms that still go through torch."""
import math

import pytest
import torch

from paper_2606_05597_amd.autograd import _scaled_to_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7, 8, 9, 2047, 2049, 65536 * 2048 + 2048 * 3 + 5])
@pytest.mark.parametrize("g", [1.0, -0.3, 1e-30])
def test_one_pass_matches_two(n, g):
    x = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    for i, v in enumerate([math.inf, -math.inf, math.nan, 0.0, -0.0, 3.4e38, 1e-40][:n]):
        x[i] = v
    up = torch.tensor(g, dtype=torch.float64, device="cuda")
    with torch.no_grad():
        got = _scaled_to_bf16(x, up)
    want = torch.mul(x, up.to(torch.float32)).to(torch.bfloat16)
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got.nan_to_num(), want.nan_to_num())


def test_other_forms_go_through_torch():
    x = torch.randn(16, 8, device="cuda")
    up = torch.tensor(0.5, dtype=torch.float64, device="cuda")
    want = (x * 0.5).to(torch.bfloat16)
    with torch.no_grad():
        assert torch.equal(_scaled_to_bf16(x.t().contiguous().t(), up), want)  # strided
        odd = torch.empty(16 * 8 + 1, device="cuda")[1:].view(16, 8).copy_(x)  # not 16-byte aligned
        assert torch.equal(_scaled_to_bf16(odd, up), want)
        ups = torch.tensor([0.5, 2.0], dtype=torch.float64, device="cuda")
        got = torch.func.vmap(lambda u: _scaled_to_bf16(x, u))(ups)  # batched upstream gradients
        assert torch.equal(got[0], want) and torch.equal(got[1], (x * 2).to(torch.bfloat16))
    up2 = up.clone().requires_grad_(True)  # a graph through the backward
    _scaled_to_bf16(x, up2).float().sum().backward()
    assert up2.grad is not None


def test_forward_mode_modes_and_lazy_negation_go_through_torch():
    from torch.autograd import forward_ad
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        def __init__(self):
            super().__init__()
            self.ops = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.ops.append(func.__name__)
            return func(*args, **(kwargs or {}))

    x = torch.randn(16, 8, device="cuda")
    up = torch.tensor(0.5, device="cuda")
    with torch.no_grad():
        with forward_ad.dual_level():  # the tangent of the upstream gradient reaches dW
            out = _scaled_to_bf16(x, forward_ad.make_dual(up, torch.tensor(2.0, device="cuda")))
            tangent = forward_ad.unpack_dual(out).tangent
            assert tangent is not None and torch.equal(tangent, (x * 2).to(torch.bfloat16))
        with Seen() as seen:
            _scaled_to_bf16(x, up)
        assert any("mul" in op for op in seen.ops)
        neg = torch._neg_view(up)  # -0.5 over memory that holds 0.5
        assert torch.equal(_scaled_to_bf16(x, neg), (x * -0.5).to(torch.bfloat16))


def test_function_modes_go_through_torch():
    from torch.overrides import TorchFunctionMode

    class Seen(TorchFunctionMode):
        def __init__(self):
            super().__init__()
            self.calls = []

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.calls.append(func.__name__)
            return func(*args, **(kwargs or {}))

    x = torch.randn(16, 8, device="cuda")
    up = torch.tensor(0.5, device="cuda")
    with torch.no_grad():
        with Seen() as seen:
            got = _scaled_to_bf16(x, up)
        assert "mul" in seen.calls and torch.equal(got, (x * 0.5).to(torch.bfloat16))


def test_an_upstream_gradient_without_memory():
    x = torch.randn(16, 8, device="cuda")
    zero = torch._efficientzerotensor((), device="cuda")  # known to be zero: no storage behind it
    with torch.no_grad():
        assert torch.equal(_scaled_to_bf16(x, zero) + 0, torch.zeros_like(x, dtype=torch.bfloat16))


@pytest.mark.parametrize("V", [65528, 65536])
def test_wrapper_scales_small_and_large_dw(V):
    import paper_2606_05597_amd as grpo
    T, H = 40, 64  # H V on both sides of the one pass's 2^22 elements
    gen = torch.Generator("cuda").manual_seed(4)
    h = torch.randn((T, H), device="cuda", generator=gen).to(torch.bfloat16)
    W = (torch.randn((H, V), device="cuda", generator=gen) / 8).to(torch.bfloat16)
    act = torch.randint(0, V, (T,), device="cuda", generator=gen, dtype=torch.int32)
    behave = torch.full((T,), -11.0, device="cuda")
    adv = torch.tensor([1.0, -1.0], device="cuda")
    sto = torch.tensor([0, 10, 25, T], dtype=torch.int32, device="cuda")
    tso = torch.tensor([0, 1, 3], dtype=torch.int32, device="cuda")
    _, dh, dw = grpo.fused_lmhead_grpo_blocked(h, W, act, behave, adv, sto, tso, 2)
    hp, Wp = h.clone().requires_grad_(True), W.clone().requires_grad_(True)
    loss = grpo.FusedLmHeadGrpoLoss.apply(hp, Wp, act, behave, adv, sto, tso, 2, {"schedule": "blocked"})
    (loss * 0.3).backward()
    g = torch.tensor(0.3, dtype=torch.float64, device="cuda")
    assert torch.equal(Wp.grad, torch.mul(dw, g.float()).to(torch.bfloat16))
    assert torch.equal(hp.grad, torch.mul(dh, g.to(torch.bfloat16)))
