"""The plans of mid-size and large layers (4-neuron synced forward, synced backward in place
of a double-buffered one, 8 or 2 neurons per lane) against even slices of the same neurons,
which take the plans of small layers: every neuron the same bit for bit.  Every size ends in
a partial workgroup; bit-packed rows leave a rest of a word."""
import itertools

import pytest

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 65, 900012),    # widef; synced backward
          ("f32", 71, 3000004),   # widef with partial chunks
          ("f32", 33, 450002),    # synced backward
          ("bf16", 40, 450002),   # the same
          ("f32", 13, 1300002),   # one chunk
          ("bf16", 7, 1300004),
          ("bf16", 40, 2200008),  # 32-step chunk and tail, synced, 8 per lane forward
          ("bf16", 70, 2200008),  # several
          ("bf16", 40, 2208030)]  # N % 8 != 0, rounds half filled: 2 per lane


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


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
        out = H.sentinels(*layer.alloc_forward(cfg, T, b - a, H.DEV, segment))
        spikes, saved, v = layer.forward(cfg, xs, out=out, v_in=v_in, v_last=v_last)
        gx = layer.backward(cfg, xs, saved, gss, grad_x=torch.full_like(gss, float("nan")), v_in=v_in, g_in=g_in,
                            g_out=g_out)
        return spikes, [t for t in (v, gx, v_last, g_out) if t is not None]

    spikes, whole = run(0, N)
    if spk == "bits":
        assert not H.spike_columns(spikes, N, (N + 63) // 64 * 64, spk).any()   # padding bits are written as 0
    for a, b in H.even_slices(N):
        s, part = run(a, b)
        assert torch.equal(H.spike_columns(s, 0, b - a, spk), H.spike_columns(spikes, a, b, spk))
        for p, q in zip(part, whole):
            assert torch.equal(H.as_bytes(p), H.as_bytes(q[..., a:b]))


# more than 2^20 neurons and few enough that the workgroups of the last XCD are partial; N % 64 = 52
@pytest.mark.parametrize("T,B,F", [(33, 1300, 1001)])
@pytest.mark.parametrize("io,spk", list(itertools.product(["f32", "bf16"], ["u8", "bits", "io"])))
def test_gain_and_stack_equal_slices(H, T, B, F, io, spk):
    torch, layer = H.torch, H.layer
    cfg = layer.LifConfig(0.6, 0.9, v_reset=0.1, io=io, spk=spk)
    gen = torch.Generator(device=H.DEV).manual_seed(5)
    y = torch.rand((T, B * F), device=H.DEV, generator=gen) < 0.4
    x = torch.empty((T, B * F), dtype=cfg.dtype, device=H.DEV).normal_(0.5, 0.6, generator=gen)
    gs = torch.empty_like(x).normal_(generator=gen)
    gains = torch.empty((2, F), device=H.DEV).uniform_(-0.4, 1.6, generator=gen)

    def run(b0, b1):                                  # samples [b0, b1)
        a, b, nb = b0 * F, b1 * F, b1 - b0
        ys = H.pack_spikes(y[:, a:b], spk, cfg.dtype)
        xs, gss = (t[:, a:b].contiguous() for t in (x, gs))
        out = H.sentinels(*layer.alloc_forward(cfg, T, b - a, H.DEV))
        s1, saved, _ = layer.forward_gain(cfg, ys, gains[0].clone(), nb, F, out=out)
        nan = float("nan")
        g1 = layer.backward_gain(cfg, ys, gains[0].clone(), saved, gss, nb, F, grad_s_in=torch.full_like(gss, nan))
        s2, _, saved, _ = layer.stack_forward(cfg, xs, gains, nb, F)
        g2 = layer.stack_backward(cfg, xs, gains, saved, gss, nb, F, grad_x=torch.full_like(gss, nan))
        return (s1, s2), (g1, g2)

    spikes, grads = run(0, B)
    if spk == "bits":
        for s in spikes:
            assert not H.spike_columns(s, B * F, (B * F + 63) // 64 * 64, spk).any()
    step = 64                                         # 64,064 neurons: a narrow layer
    for b0 in range(0, B, step):
        b1 = min(B, b0 + step)
        part_s, part_g = run(b0, b1)
        for p, q in zip(part_s, spikes):
            assert torch.equal(H.spike_columns(p, 0, (b1 - b0) * F, spk), H.spike_columns(q, b0 * F, b1 * F, spk))
        for p, q in zip(part_g, grads):
            assert torch.equal(H.as_bytes(p), H.as_bytes(q[:, b0 * F:b1 * F]))
