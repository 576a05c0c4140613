"""Calls at the limits of the hardware's own sizes: reductions of more bytes than
a buffer descriptor's range covers (2^31 - 1), and launches of more threads than
HIP counts (2^32 - 1), were every token to take all the waves it usually does."""
import pytest
import torch

from gpu_helpers import dev, need_gpu
from paper_2510_00207_amd import _lib as L
from paper_2510_00207_amd.layer import MoELayer

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


def _rel(got, ref):
    return float((got.double() - ref.double()).norm() / ref.double().norm())


@pytest.mark.parametrize("R", [1, 2])
def test_weight_gradients_beyond_descriptor_range(R):
    """One expert of 140000 rows, H = 16384: 4.6 GB of dH in one chunk (past 2^32
    bytes), 2.3 GB in each of two (past 2^31). Every row is in the sums."""
    need_gpu()
    d = dev()
    T, M, H = 140000, 64, 16384
    g = torch.Generator(device=d).manual_seed(3)
    layer = MoELayer(T_total=T, M=M, H=H, E=1, k=1, R=R, f=1.0, device=d)
    for name, std in (("x", 1.0), ("dy", 1.0), ("w1", 0.1), ("w2", 0.1), ("w_gate", 0.1)):
        t = getattr(layer, name)
        t.copy_(torch.randn(t.shape, generator=g, device=d) * std)
    sc = torch.cuda.current_stream()
    layer.forward(sc, sc)
    layer.backward(sc, sc)
    torch.cuda.synchronize()
    w1, w2 = layer.w1[0].float(), layer.w2[0].float()
    dw1, dw2 = torch.zeros(M, H, device=d), torch.zeros(H, M, device=d)
    for t in range(0, T, 10000):
        x, dy = layer.x[t:t + 10000].float(), layer.dy[t:t + 10000].float()
        h = (x @ w1).requires_grad_()
        a = torch.nn.functional.gelu(h)
        (dh,) = torch.autograd.grad(a, h, dy @ w2.t().contiguous())
        dw1 += x.t().contiguous() @ dh
        dw2 += a.detach().t().contiguous() @ dy
    # h, a and dH are rounded to bf16 (2^-9 each); the rows past 2^31 bytes are half of
    # the sums
    assert _rel(layer.dw1[0], dw1) < 1e-2
    assert _rel(layer.dw2[0], dw2) < 1e-2


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_expert_weights_beyond_descriptor_range(act):
    """Experts' weights of 2 GiB and more each: x W1 (W3) of 40000 x 27136 with rows of
    every tile class, and a W2 of 27136 x 40000."""
    need_gpu()
    d = dev()
    M, H, cnt = 40000, 27136, [3, 0, 300]
    E, T = len(cnt), sum(cnt)
    HW = 2 * H if act == "swiglu" else H
    g = torch.Generator(device=d).manual_seed(5)
    n = lambda *sh, std=1.0: torch.randn(*sh, generator=g, device=d, dtype=BF) * std
    w1, w2 = n(E, M, H, std=0.005), n(E, H, M, std=0.005)
    w3 = n(E, M, H, std=0.005) if act == "swiglu" else None
    x = n(T, M)
    counts = torch.tensor(cnt, dtype=torch.int32, device=d)
    offsets = torch.tensor([0, 3, 3, 303], dtype=torch.int32, device=d)
    s = L.make_shape(T, M, H, E, 1, 300, L.BF16, L.SWIGLU if act == "swiglu" else L.GELU, L.PACKED)
    h, a, y = (torch.full((T, c), 5.0, dtype=BF, device=d) for c in (HW, H, M))
    L.flowmoe_expert_ffn(s, x, counts, offsets, w1, w3, w2, h, a, y)
    torch.cuda.synchronize()
    for e, r in ((0, slice(0, 3)), (2, slice(3, 303))):
        for j, w in enumerate((w1, w3) if act == "swiglu" else (w1,)):
            ref = sum(x[r, k:k + 8000].float() @ w[e, k:k + 8000].float() for k in range(0, M, 8000))
            # one rounding to bf16; the weight rows past 2^31 bytes are 1.1 % of the products
            assert _rel(h[r, j * H:(j + 1) * H], ref) < 4e-3
        ref = sum(a[r, k:k + 8000].float() @ w2[e, k:k + 8000].float() for k in range(0, H, 8000))
        assert _rel(y[r], ref) < 4e-3


def test_combine_of_many_tokens():
    """2^25 fp32 tokens of two segments each: 2^32 threads with a wave a segment. Few of
    the tokens have rows (in each, and in the last block); the others' are zeros."""
    need_gpu()
    d = dev()
    T, M, n = 1 << 25, 520, 1000
    s = L.make_shape(T, M, 8, 2, 1, n // 2, L.F32, L.GELU, L.PACKED)
    rows = L.flowmoe_rows_capacity(s)
    assert rows == n
    g = torch.Generator(device=d).manual_seed(9)
    tok = torch.randperm(T - 1, generator=g, device=d)[:n]
    tok[0] = T - 1
    slot = torch.full((T, 1), -1, dtype=torch.int32, device=d)
    slot[tok, 0] = torch.arange(n, dtype=torch.int32, device=d)
    w = torch.rand(T, 1, generator=g, device=d)
    src = torch.randn(n, M, generator=g, device=d)
    counts = torch.tensor([n // 2, n // 2], dtype=torch.int32, device=d)
    offsets = torch.tensor([0, n // 2, n], dtype=torch.int32, device=d)
    y = torch.empty(T, M, device=d)
    for weight, call in ((w[tok], lambda: L.flowmoe_combine(s, src, slot, w, y)),
                         (1.0, lambda: L.flowmoe_dispatch_bwd(s, src, slot, y))):
        y.fill_(7.0)
        call()
        assert torch.equal(y[tok], weight * src)
        y[tok] = 0
        assert not any(c.any() for c in y.chunk(64))
    y.fill_(0.5)
    y[tok] = torch.randn(n, M, generator=g, device=d)
    dys, dw = torch.full((n, M), 7.0, device=d), torch.full((T, 1), 7.0, device=d)
    L.flowmoe_combine_bwd(s, y, src, slot, w, counts, offsets, dys, dw)
    assert torch.equal(dys, w[tok] * y[tok])
    ref = (y[tok].double() * src.double()).sum(1)
    # 520 products summed in fp32, off by at most 2^-24 of their size each and at each sum
    assert (dw[tok, 0].double() - ref).abs().max() < 520 * 2.0 ** -22
    dw[tok] = 0
    assert not dw.any()


def test_f32_gate_of_many_tokens():
    """2^27 + 5 tokens at E = 64, eight a block of 256 threads: more than 2^32 threads."""
    need_gpu()
    d = dev()
    T, M, E = (1 << 27) + 5, 8, 64
    g = torch.Generator(device=d).manual_seed(9)
    x = torch.randn(T, M, generator=g, device=d)
    wg = torch.randn(M, E, generator=g, device=d)
    logits = torch.full((T, E), 7.0, device=d)
    idx = torch.full((T, 1), -5, dtype=torch.int32, device=d)
    w = torch.full((T, 1), 7.0, device=d)
    s = L.make_shape(T, M, 8, E, 1, 0, L.F32, L.GELU, L.PACKED)
    L.flowmoe_gate_topk(s, x, wg, None, logits, idx, w)
    torch.cuda.synchronize()
    assert bool((w == 1).all())  # (the softmax over one)
    for a in range(0, T, 1 << 24):
        lg, ix = logits[a:a + (1 << 24)], idx[a:a + (1 << 24)].long()
        assert torch.equal(lg.gather(1, ix)[:, 0], lg.max(1).values)
    for r in (slice(0, 4096), slice((1 << 27) - 4096, None)):
        ref = x[r].double() @ wg.double()
        assert (logits[r].double() - ref).abs().max() < 1e-5 * ref.abs().max()
