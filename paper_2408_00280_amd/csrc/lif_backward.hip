// Backward-kernel launchers for one I/O dtype, chosen at build time by SNNLIF_IO.  With
// SNNLIF_GAIN=1 (and SNNLIF_SPK) the unit holds the backward of the layer fed by the previous
// layer's spikes through a per-feature gain.
#include "lif_host.h"
#include "lif_kernels.h"

#if !defined(SNNLIF_IO)
#error "build with -DSNNLIF_IO=<snn_io>"
#endif
#ifndef SNNLIF_GAIN
#define SNNLIF_GAIN 0
#endif

namespace snnlif {
namespace {

// The relay's workgroups: a wave per chunk, up to kRelayWaves.
int relay_lanes(const Plan& p, int64_t T) {
    const int64_t chunks = (T + p.k - 1) / p.k;
    return kWave * int(chunks < kRelayWaves ? chunks : kRelayWaves);
}

}  // namespace

#if !SNNLIF_GAIN

template <int IO>
snn_status backward_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, const void* x,
                          const void* saved, const void* gs, void* gx, const float* v_in, const float* g_in,
                          float* g_out, hipStream_t s) {
    const float* sv = static_cast<const float*>(saved);
    const BwdSeg seg{v_in, g_in, g_out};
    auto go = [&](auto rst) {
        constexpr int R = decltype(rst)::value;
        auto row_walk = [&](auto V, auto K, auto PIPE, auto blk, auto sync, auto ragged) {
            constexpr int Vc = decltype(V)::value, Kc = decltype(K)::value, B = decltype(blk)::value;
            constexpr bool Pc = decltype(PIPE)::value, S = decltype(sync)::value, Q = decltype(ragged)::value;
            return launch_blk(lif_backward_kernel<IO, R, Vc, Kc, Pc, B, S, Q>, wide_grid<SNN_SPK_IO, Vc>(N, B), B, s, k,
                              T, N, x, sv, gs, gx, seg);
        };
        return backward_route<IO>(p, T, N, row_walk, [&](auto K) {
            return launch_blk(lif_backward_relay_kernel<IO, R, decltype(K)::value>, grid_for(N, kWave),
                              relay_lanes(p, T), s, k, T, N, x, sv, gs, gx, seg);
        });
    };
    return reset == SNN_RESET_SOFT ? go(IntC<SNN_RESET_SOFT>{}) : go(IntC<SNN_RESET_HARD>{});
}

template snn_status backward_entry<SNNLIF_IO>(int, const Plan&, const LifK&, int64_t, int64_t, const void*,
                                              const void*, const void*, void*, const float*, const float*, float*,
                                              hipStream_t);

#else

#if !defined(SNNLIF_SPK)
#error "build the gain unit with -DSNNLIF_SPK=<snn_spk>"
#endif

template <int IO, int SPK>
snn_status backward_gain_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, int64_t F,
                               const void* spikes_in, const float* gain, const void* saved, const void* gs,
                               void* gs_in, hipStream_t s) {
    const uint8_t* si = static_cast<const uint8_t*>(spikes_in);
    const float* sv = static_cast<const float*>(saved);
    auto go = [&](auto rst) {
        constexpr int R = decltype(rst)::value;
        auto row_walk = [&](auto V, auto K) {
            constexpr int Vc = decltype(V)::value, Kc = decltype(K)::value;
            return launch(lif_backward_gain_kernel<IO, SPK, R, Vc, Kc>, grid_for((N + Vc - 1) / Vc), s, k, T, N, F, si,
                          gain, p.row_bytes, sv, gs, gs_in);
        };
        return backward_gain_route<IO>(p, row_walk, [&](auto K) {
            return launch_blk(lif_backward_gain_relay_kernel<IO, SPK, R, decltype(K)::value>, grid_for(N, kWave),
                              relay_lanes(p, T), s, k, T, N, F, si, gain, p.row_bytes, sv, gs, gs_in);
        });
    };
    return reset == SNN_RESET_SOFT ? go(IntC<SNN_RESET_SOFT>{}) : go(IntC<SNN_RESET_HARD>{});
}

template snn_status backward_gain_entry<SNNLIF_IO, SNNLIF_SPK>(int, const Plan&, const LifK&, int64_t, int64_t,
                                                               int64_t, const void*, const float*, const void*,
                                                               const void*, void*, hipStream_t);

#endif

}  // namespace snnlif
