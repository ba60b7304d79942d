"""Layers of few neurons and several chunks (one neuron per lane, one-wave workgroups, the
backward as a relay of waves) against the same neurons inside a wider layer, which takes the
general path: spikes, membranes, checkpoints, gradients and the handed-on segment state are
the same bit for bit.  Sizes: less than, exactly and just over a wave; the last narrow size;
tails of 1 .. K - 1 steps; fewer, as many and more chunks than the relay has waves."""
import itertools

import pytest

pytestmark = pytest.mark.gpu

NARROW_N = 5 * 256 * 64   # the largest layer that takes the narrow path

SHAPES = [(17, 2), (33, 1), (40, 64), (47, 65), (128, 66), (129, 63), (150, 1000), (289, 127), (33, NARROW_N),
          (40, NARROW_N - 1), (129, 64001), (300, 69148)]   # the last two: backward not as a relay


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("T,N", SHAPES, ids=str)
@pytest.mark.parametrize("reset,io,spk", list(itertools.product(["hard", "soft"], ["f32", "bf16"], ["u8", "bits", "io"])))
@pytest.mark.parametrize("segment", [False, True])
def test_dense(H, T, N, reset, io, spk, segment):
    torch, layer = H.torch, H.layer
    cfg = layer.LifConfig(0.6, 0.9, v_reset=0.1, reset=reset, io=io, spk=spk)
    wide = NARROW_N + 2 + N % 2                       # the same chunk length: N's parity
    gen = torch.Generator(device=H.DEV).manual_seed(T * 7919 + N)
    x = torch.empty((T, wide), dtype=cfg.dtype, device=H.DEV).normal_(0.5, 0.6, generator=gen)
    gs = torch.empty_like(x).normal_(generator=gen)
    state = torch.randn((2, wide), device=H.DEV, generator=gen)
    a = wide - N                                      # the wide layer's last N neurons

    def run(lo):
        n = wide - lo
        xs, gss = x[:, lo:].contiguous(), gs[:, lo:].clone().contiguous()
        if not segment:
            spikes, saved, v = layer.forward(cfg, xs, v_out=True)
            return spikes, saved, v, layer.backward(cfg, xs, saved, gss), ()
        v_in, g_in = state[0, lo:].clone(), state[1, lo:].clone()
        v_last, g_out = torch.empty_like(v_in), torch.empty_like(g_in)
        out = H.sentinels(*layer.alloc_forward(cfg, T, n, H.DEV, True))
        spikes, saved, v = layer.forward(cfg, xs, out=out, v_in=v_in, v_last=v_last)
        gx = layer.backward(cfg, xs, saved, gss, grad_x=gss, v_in=v_in, g_in=g_in, g_out=g_out)   # in place
        return spikes, saved, v, gx, (v_last, g_out)

    w, s = run(0), run(a)
    assert torch.equal(H.spike_columns(s[0], 0, N, spk), H.spike_columns(w[0], a, wide, spk))
    if spk == "bits" and N % 64:
        pad = H.spike_columns(s[0], N, (N + 63) // 64 * 64, spk)
        assert not pad.any()                          # padding bits are written as 0
    saved_w, saved_s = (t.view(torch.float32).view(-1, n) for t, n in ((w[1], wide), (s[1], N)))
    assert torch.equal(H.as_bytes(saved_s), H.as_bytes(saved_w[:, a:]))
    assert torch.equal(H.as_bytes(s[2]), H.as_bytes(w[2][:, a:]))
    assert torch.equal(H.as_bytes(s[3]), H.as_bytes(w[3][:, a:]))
    for narrow, whole in zip(s[4], w[4]):
        assert torch.equal(H.as_bytes(narrow), H.as_bytes(whole[a:]))


@pytest.mark.parametrize("T,B,F", [(17, 1, 2), (33, 3, 21), (40, 2, 33), (47, 7, 64), (150, 5, 200), (289, 16, 40),
                                   (97, 3, 21), (161, 5, 33), (48, 1631, 33), (300, 692, 100)])
@pytest.mark.parametrize("reset,io,spk", list(itertools.product(["hard", "soft"], ["f32", "bf16"], ["u8", "bits", "io"])))
def test_gain(H, T, B, F, reset, io, spk):
    torch, layer = H.torch, H.layer
    cfg = layer.LifConfig(0.6, 0.9, v_reset=0.1, reset=reset, io=io, spk=spk)
    Bw = NARROW_N // F + 1
    Bw += (Bw - B) % 2                                # the same parity of N
    N, wide = B * F, Bw * F
    gen = torch.Generator(device=H.DEV).manual_seed(T * 7919 + N)
    y = torch.rand((T, wide), device=H.DEV, generator=gen) < 0.4
    gs = torch.empty((T, wide), dtype=cfg.dtype, device=H.DEV).normal_(generator=gen)
    gain = torch.empty(F, device=H.DEV).uniform_(-0.4, 1.6, generator=gen)

    def run(b):
        lo = (Bw - b) * F
        ys, gss = H.pack_spikes(y[:, lo:], spk, cfg.dtype), gs[:, lo:].contiguous()
        out = H.sentinels(*layer.alloc_forward(cfg, T, b * F, H.DEV, True))
        spikes, saved, v = layer.forward_gain(cfg, ys, gain, b, F, out=out)
        gx = layer.backward_gain(cfg, ys, gain, saved, gss, b, F, grad_s_in=torch.full_like(gss, float("nan")))
        return H.spike_columns(spikes, 0, b * F, spk), saved.view(torch.float32).view(-1, b * F), v, gx

    for narrow, whole in zip(run(B), run(Bw)):
        assert torch.equal(H.as_bytes(narrow), H.as_bytes(whole[:, wide - N:]))
