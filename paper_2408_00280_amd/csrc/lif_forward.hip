// Forward-kernel launchers for one (I/O dtype, spike format) pair, chosen at build time by
// SNNLIF_IO and SNNLIF_SPK so that the variants compile as parallel translation units.
// With SNNLIF_GAIN=1 the unit holds the layer fed by the previous layer's spikes through a
// per-feature gain instead of the layer fed by a dense input current.
#include "lif_host.h"
#include "lif_kernels.h"

#if !defined(SNNLIF_IO) || !defined(SNNLIF_SPK)
#error "build with -DSNNLIF_IO=<snn_io> -DSNNLIF_SPK=<snn_spk>"
#endif
#ifndef SNNLIF_GAIN
#define SNNLIF_GAIN 0
#endif

namespace snnlif {

#if !SNNLIF_GAIN

template <int IO, int SPK>
snn_status forward_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, const void* x,
                         void* spikes, void* saved, float* v_out, const float* v_in, float* v_last,
                         hipStream_t s) {
    uint8_t* sp = static_cast<uint8_t*>(spikes);
    float* sv = static_cast<float*>(saved);
    auto go = [&](auto rst) {
        return forward_route<IO>(p, T, N, [&](auto V, auto FB, auto K, auto PIPE, auto blk, auto ragged) {
            constexpr int R = decltype(rst)::value, Vc = decltype(V)::value, Fc = decltype(FB)::value;
            constexpr int Kc = decltype(K)::value, B = decltype(blk)::value;
            constexpr bool Pc = decltype(PIPE)::value, Q = decltype(ragged)::value;
            const dim3 g = forward_grid<SPK, Vc, Q>(N, B);
            return v_out ? launch_blk(lif_forward_kernel<IO, SPK, R, Vc, Fc, Kc, true, Pc, B, Q>, g, B, s, k, T, N, x,
                                      sp, p.row_bytes, sv, v_out, v_in, v_last)
                         : launch_blk(lif_forward_kernel<IO, SPK, R, Vc, Fc, Kc, false, Pc, B, Q>, g, B, s, k, T, N, x,
                                      sp, p.row_bytes, sv, v_out, v_in, v_last);
        });
    };
    return reset == SNN_RESET_SOFT ? go(IntC<SNN_RESET_SOFT>{}) : go(IntC<SNN_RESET_HARD>{});
}

template snn_status forward_entry<SNNLIF_IO, SNNLIF_SPK>(int, const Plan&, const LifK&, int64_t, int64_t,
                                                         const void*, void*, void*, float*, const float*, float*,
                                                         hipStream_t);

#else

template <int IO, int SPK>
snn_status forward_gain_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, int64_t F,
                              const void* spikes_in, const float* gain, void* spikes, void* saved, float* v_out,
                              hipStream_t s) {
    const uint8_t* si = static_cast<const uint8_t*>(spikes_in);
    uint8_t* sp = static_cast<uint8_t*>(spikes);
    float* sv = static_cast<float*>(saved);
    auto go = [&](auto rst) {
        return forward_gain_route<IO>(p, [&](auto V, auto FB, auto K, auto PIPE, auto blk) {
            constexpr int R = decltype(rst)::value, Vc = decltype(V)::value, Fc = decltype(FB)::value;
            constexpr int Kc = decltype(K)::value, B = decltype(blk)::value;
            constexpr bool Pc = decltype(PIPE)::value;
            const dim3 g = wide_grid<SPK, Vc>(N, B);
            return v_out ? launch_blk(lif_forward_gain_kernel<IO, SPK, R, Vc, Fc, Kc, true, Pc, B>, g, B, s, k, T, N, F,
                                      si, gain, sp, p.row_bytes, sv, v_out)
                         : launch_blk(lif_forward_gain_kernel<IO, SPK, R, Vc, Fc, Kc, false, Pc, B>, g, B, s, k, T, N,
                                      F, si, gain, sp, p.row_bytes, sv, v_out);
        });
    };
    return reset == SNN_RESET_SOFT ? go(IntC<SNN_RESET_SOFT>{}) : go(IntC<SNN_RESET_HARD>{});
}

template snn_status forward_gain_entry<SNNLIF_IO, SNNLIF_SPK>(int, const Plan&, const LifK&, int64_t, int64_t,
                                                              int64_t, const void*, const float*, void*, void*,
                                                              float*, hipStream_t);

#endif

}  // namespace snnlif
