"""The plans of mid-size and large layers (4-neuron synced forward, synced backward in place
of a double-buffered one, workgroups in launch order) against even slices of the same
neurons, which take the narrow or the one-chunk plan: the same bit for bit.  Every size ends
in a partial workgroup; bit-packed rows leave a rest of a word."""
import itertools

import pytest

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 65, 900012),    # widef; synced backward
          ("f32", 71, 3000004),   # widef with partial chunks
          ("f32", 33, 450002),    # synced backward
          ("bf16", 40, 450002),   # the same
          ("f32", 13, 1300002),   # one chunk, launch order
          ("bf16", 7, 1300004),
          ("bf16", 40, 2200008),  # 32-step chunk and tail, launch order
          ("bf16", 70, 2200008)]  # several, synced in launch order


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


def _spikes(H, s, a, b, spk):
    torch = H.torch
    if spk != "bits":
        return (s[:, a:b] != 0).to(torch.uint8)
    n = torch.arange(a, b, device=s.device)
    return ((s[:, n >> 3] >> (n & 7).to(torch.uint8)) & 1).to(torch.uint8)


def _same(a, b):
    return (a.contiguous().view(-1) == b.contiguous().view(-1)).all() and a.dtype == b.dtype


@pytest.mark.parametrize("io,T,N", SHAPES, ids=str)
@pytest.mark.parametrize("reset,spk,segment", list(itertools.product(["hard", "soft"], ["u8", "bits", "io"], [False, True])))
def test_plan_equals_slices(H, io, T, N, reset, spk, segment):
    torch, layer = H.torch, H.layer
    cfg = layer.LifConfig(0.6, 0.9, v_reset=0.1, reset=reset, io=io, spk=spk)
    gen = torch.Generator(device=H.DEV).manual_seed(T * 7919 + N)
    x = torch.empty((T, N), dtype=cfg.dtype, device=H.DEV).normal_(0.5, 0.6, generator=gen)
    gs = torch.empty_like(x).normal_(generator=gen)
    state = torch.randn((2, N), device=H.DEV, generator=gen)

    def run(a, b):
        xs, gss = x[:, a:b].contiguous(), gs[:, a:b].contiguous()
        v_in = g_in = v_last = g_out = None
        if segment:
            v_in, g_in = state[0, a:b].clone(), state[1, a:b].clone()
            v_last, g_out = torch.empty_like(v_in), torch.empty_like(g_in)
        out = layer.alloc_forward(cfg, T, b - a, H.DEV, segment)
        spikes, saved, v = layer.forward(cfg, xs, out=out, v_in=v_in, v_last=v_last)
        gx = layer.backward(cfg, xs, saved, gss, v_in=v_in, g_in=g_in, g_out=g_out)
        return spikes, [t for t in (v, gx, v_last, g_out) if t is not None]

    spikes, whole = run(0, N)
    if spk == "bits":
        assert not _spikes(H, spikes, N, (N + 63) // 64 * 64, spk).any()   # padding bits are written as 0
    for a, b in ((0, 192), (N - 192, N)):
        s, part = run(a, b)
        assert torch.equal(_spikes(H, s, 0, b - a, spk), _spikes(H, spikes, a, b, spk))
        for p, q in zip(part, whole):
            assert _same(p, q[..., a:b])
    torch.cuda.synchronize()


@pytest.mark.parametrize("T,B,F", [(33, 1300, 1001)])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_gain_and_stack_in_launch_order(H, T, B, F, io):
    torch, layer = H.torch, H.layer
    cfg = layer.LifConfig(0.6, 0.9, v_reset=0.1, io=io, spk="io")
    gen = torch.Generator(device=H.DEV).manual_seed(5)
    y = (torch.rand((T, B * F), device=H.DEV, generator=gen) < 0.4).to(cfg.dtype)
    x = torch.empty((T, B * F), dtype=cfg.dtype, device=H.DEV).normal_(0.5, 0.6, generator=gen)
    gs = torch.empty_like(y).normal_(generator=gen)
    gains = torch.empty((2, F), device=H.DEV).uniform_(-0.4, 1.6, generator=gen)

    def run(b):                                       # the first b samples
        n = b * F
        ys, xs, gss = (t[:, :n].contiguous() for t in (y, x, gs))
        s1, saved, _ = layer.forward_gain(cfg, ys, gains[0].clone(), b, F)
        g1 = layer.backward_gain(cfg, ys, gains[0].clone(), saved, gss, b, F)
        s2, _, saved, _ = layer.stack_forward(cfg, xs, gains, b, F)
        return s1, g1, s2, layer.stack_backward(cfg, xs, gains, saved, gss, b, F)

    for part, whole in zip(run(2), run(B)):
        assert _same(part, whole[:, :2 * F])
