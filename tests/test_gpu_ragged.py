"""bf16 layers whose N is no multiple of the lane width (unaligned rows, and a rest of N that
takes one neuron per lane) against even slices of the same neurons, which take the aligned
path: spikes, membranes, gradients and the handed-on segment state of every neuron are the
same bit for bit."""
import itertools

import pytest

pytestmark = pytest.mark.gpu

# N: 2 per lane (rest 1), 8 per lane in the forward and 4 in short backwards (rests 1, 2, 6, 63 bits)
SHAPES = [(3, 257), (12, 2097153), (16, 2097154), (20, 81927), (32, 513), (33, 262145), (40, 2097158), (72, 2097215),
          (100, 100003), (50, 2203833), (200, 2097155)]   # ... rounds half filled; backward without barriers


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("T,N", SHAPES, ids=str)
@pytest.mark.parametrize("reset,spk", list(itertools.product(["hard", "soft"], ["u8", "bits", "io"])))
@pytest.mark.parametrize("segment", [False, True])
def test_ragged_rows(H, T, N, reset, spk, segment):
    torch, layer = H.torch, H.layer
    cfg = layer.LifConfig(0.6, 0.9, v_reset=0.1, reset=reset, io="bf16", spk=spk)
    gen = torch.Generator(device=H.DEV).manual_seed(T * 7919 + N)
    x = torch.empty((T, N), dtype=cfg.dtype, device=H.DEV).normal_(0.5, 0.6, generator=gen)
    gs = torch.empty_like(x).normal_(generator=gen)
    state = torch.randn((2, N), device=H.DEV, generator=gen)

    def run(a, b):
        xs, gss = x[:, a:b].contiguous(), gs[:, a:b].clone().contiguous()
        v_in = g_in = v_last = g_out = None
        if segment:
            v_in, g_in = state[0, a:b].clone(), state[1, a:b].clone()
            v_last, g_out = torch.empty_like(v_in), torch.empty_like(g_in)
        out = H.sentinels(*layer.alloc_forward(cfg, T, b - a, H.DEV, True))
        spikes, saved, v = layer.forward(cfg, xs, out=out, v_in=v_in, v_last=v_last)
        gx = layer.backward(cfg, xs, saved, gss, grad_x=gss, v_in=v_in, g_in=g_in, g_out=g_out)   # in place
        return spikes, [t for t in (v, gx, v_last, g_out) if t is not None]

    spikes, whole = run(0, N)
    if spk == "bits":
        assert not H.spike_columns(spikes, N, (N + 63) // 64 * 64, spk).any()   # padding bits are written as 0
    for a, b in H.even_slices(N):
        s, part = run(a, b)
        assert torch.equal(H.spike_columns(s, 0, b - a, spk), H.spike_columns(spikes, a, b, spk))
        for p, q in zip(part, whole):
            assert torch.equal(H.as_bytes(p), H.as_bytes(q[..., a:b]))
