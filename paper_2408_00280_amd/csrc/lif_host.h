// Host-side planning and launching for the fused LIF library: argument checks, the lane /
// chunk plan shared by forward and backward, and the per-translation-unit launchers.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "lif_common.h"

namespace snnlif {

inline snn_status check_cfg(const snn_lif_cfg* c) {
    if (c == nullptr) return SNN_E_NULL;
    if (!(c->decay >= 0.0f && c->decay <= 1.0f)) return SNN_E_PARAM;  // also rejects NaN
    if (!std::isfinite(c->v_th) || !std::isfinite(c->v_reset)) return SNN_E_PARAM;
    if (!(c->alpha > 0.0f) || !std::isfinite(c->alpha)) return SNN_E_PARAM;
    if (c->reset != SNN_RESET_HARD && c->reset != SNN_RESET_SOFT) return SNN_E_PARAM;
    if (c->io != SNN_IO_F32 && c->io != SNN_IO_BF16) return SNN_E_PARAM;
    if (c->spk != SNN_SPK_U8 && c->spk != SNN_SPK_BITS && c->spk != SNN_SPK_IO) return SNN_E_PARAM;
    return SNN_OK;
}

inline snn_status check_shape(int64_t T, int64_t N) {
    if (T < 0 || N < 0 || T > kMaxT || N > kMaxN) return SNN_E_SHAPE;
    if (T > 0 && N > kMaxTN / T) return SNN_E_SHAPE;
    return SNN_OK;
}

inline bool aligned_to(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline bool aligned(const void* p) { return aligned_to(p, 16); }

inline int64_t io_bytes(const snn_lif_cfg* c) { return c->io == SNN_IO_F32 ? 4 : 2; }

inline int64_t spike_row_bytes(const snn_lif_cfg* c, int64_t N) {
    return c->spk == SNN_SPK_U8 ? N : c->spk == SNN_SPK_BITS ? 8 * ((N + 63) / 64) : N * io_bytes(c);
}

// Neurons per lane in the forward (vf) and the backward (vb), steps per chunk (K, also the
// checkpoint interval, sized by the backward's register budget) and whether chunks are
// double-buffered.  The same choice drives both kernels and the checkpoint layout (which
// does not depend on the lane widths), so it depends only on (cfg, T, N).
struct Plan {
    int vf;
    int vb;
    int k;
    bool pipe;
    int blkf;        // workgroup sizes of the dense forward and backward kernels
    int blkb;
    bool syncb;      // the backward's kSyncBlock workgroups meet at a barrier after each chunk
    int rf;          // bf16 layers whose N is not a multiple of the widths above: the wider
    int rb;          // lanes that take their place, all but a rest of N (else 0)
    bool widef;      // fp32 forward: 4 neurons per lane, 4-row batches, kSyncBlock workgroups
    bool midsync;    // the backward of a double-buffered plan single-buffered in synced workgroups
    bool narrow;     // few neurons, several chunks: the forward with one neuron per lane in
                     // place of vf, in one-wave workgroups
    bool relay;      // the same: the backward as a relay of waves
    int64_t row_bytes;
};

// Steps per chunk for v neurons per backward lane: the backward keeps K membranes per
// neuron in VGPRs plus K rows of x and dL/dy (twice the rows when double-buffered).  Large
// bf16 layers (not double-buffered) take 32 steps at 2 neurons per lane instead: half the
// checkpoint traffic, and bf16 rows take half the registers (make_plan).
constexpr int chunk_steps(int v) { return v == 1 ? 32 : 16; }

// A layer of T <= K steps is one chunk and keeps no checkpoint; it runs with the shortest
// of these chunk lengths that holds T, so that registers sized for K steps do not cap the
// occupancy of short-lived waves.
constexpr int kShortChunks[] = {4, 8, 16};

// Lanes that fill the chip with 16 waves per CU (256 CUs x 16 x 64).
constexpr int64_t kFillLanes = int64_t(256) * 16 * 64;

// Workgroup size for layers of several chunks that are not double-buffered.  Rows lie
// 16-32 MiB apart, each in its own 2 MiB page, and a wave uses a few hundred bytes of each;
// as waves drift apart along a long walk, the pages in use at once outgrow the per-CU
// address-translation cache.  16 waves that start together and meet at a barrier after
// every chunk share the translations of the same rows' pages.  Measured against
// 256-lane workgroups: forward -4% (bf16, T = 256) to -6.5% (fp32, T = 128 and 256);
// fp32 backward -1.5% / -5% / -6.5% / -2.5% at T = 32 / 64 / 128 / 256 (N = 8.4M).  The
// bf16 backward (32-step chunks, one such workgroup per CU) with the barrier is 1.3-2.6%
// faster than without it at T = 64 / 96 / 128 / 192 in every run (21 runs, five boxes),
// but at T = 256 it ran 13% slower in about half the runs, so it takes the barrier only
// for layers of at most kSyncBf16Chunks chunks; without one it is a steady 1.5-3% faster
// than 256-lane workgroups.
// A 1024-lane workgroup allows 128 VGPRs per lane: the 8-neuron bf16 forward with spikes
// in the I/O dtype needs about 150 and spills some 40, yet still ran 2% / 5% faster than
// the spill-free 256-lane kernel at T = 64 / 256 (N = 2^24), so it keeps these workgroups.
constexpr int kSyncBlock = 1024;
constexpr int kSyncBf16Chunks = 6;

// A layer of several chunks with at most this many neurons (5 waves per CU at one neuron
// per lane) runs one neuron per lane, in workgroups of one wave, double-buffered, and its
// backward as a relay of waves (backward_relay): twice the lanes of the wider plan, and as
// many CUs as there are waves.  Its chunk length stays that of the wider plan.  Measured
// against 2 neurons per lane in 256-lane workgroups, fp32 forward: x[1000][8192] 52.5 ->
// 28.9 us, [200][16384] 14.2 -> 8.2 us, [200][65536] 19.0 -> 14.7 us, [200][80000] 20.1 ->
// 17.3 us, [200][98304] 21.6 -> 20.9 us (bf16 17.2 -> 19.6 us): hence the limit.
constexpr int64_t kNarrowN = 5 * int64_t(256) * 64;

constexpr int64_t kWaveN = int64_t(256) * 64;   // neurons of one wave per CU

// The narrow forward does not pay for all of them either.  Against the plan it replaces (2,900
// sizes, most 1.1-1.8 times as fast): bf16 bit spikes of even N, whose words one lane per wave
// stores, 0.83-1.0 beyond one wave of neurons per CU up to 64 steps, beyond three up to 128
// (x[44][77454] 0.83); fp32 spikes in the I/O dtype, many steps beyond three and a half waves
// per CU 0.86-1.0 ([389][76402] 0.86, odd [706][62503] 0.88; odd N past 66 workgroups of 1,024
// neurons 1.2-1.4).  Gain-fed layers, which it double-buffers and the other plan does not: bf16
// spikes in the I/O dtype as the bit spikes ([47][74240] 0.70), fp32 ones beyond four waves per
// CU (0.87-1.1, [536][79050] 0.87), and odd N of up to three 32-step chunks ([48][53805] 0.76,
// [93][62985] 0.72).
inline bool narrow_forward(const snn_lif_cfg* c, int64_t T, int64_t N, int k, bool gain) {
    const bool f32 = c->io == SNN_IO_F32, odd = k == chunk_steps(1);
    if (gain && odd && T <= 3 * k) return false;
    if (!f32 && !odd && c->spk == (gain ? SNN_SPK_IO : SNN_SPK_BITS))
        return N <= kWaveN || T > (N <= 3 * kWaveN ? 64 : 128);
    if (f32 && c->spk == SNN_SPK_IO && T > 8 * k)
        return N <= (gain && !odd ? 4 * kWaveN : 7 * kWaveN / 2) || (odd && N > 66 * 1024);
    return true;
}

// The relay keeps eight chunks of a workgroup's 64 neurons in flight, so with several
// workgroups to a CU a long walk touches more rows at once than the plan of few waves and
// two chunks: against that one (1,600 sizes) it is 1.1-5 times as fast on up to three waves of
// neurons per CU, whatever T, and on all narrow layers of few steps (fp32 100, bf16 250), but
// 0.75-1.0 beyond both (fp32 x[765][69148] 0.77, [176][80472] 0.91, bf16 [993][65778] 0.62,
// [816][57246] 0.92).  Chunks of 32 steps (odd N) hold more registers: two and a half waves
// per CU in fp32, three in bf16 (fp32 [932][42301] 0.91, [515][66958] 0.79, bf16 [256][64015]
// 0.83), or less than two chunks (fp32 [64][49863] gain-fed 0.80); past 66 workgroups of 1,024
// neurons it gains again (1.0-1.4; the plan it replaces then has two workgroups on some CUs).
inline bool relay_backward(const snn_lif_cfg* c, int64_t T, int64_t N, int k) {
    const bool f32 = c->io == SNN_IO_F32;
    if (k == chunk_steps(2)) return N <= 3 * kWaveN || T <= (f32 ? 100 : 250);
    return N <= (f32 ? 5 * kWaveN / 2 : 3 * kWaveN) || T < 64 || N > 66 * 1024;
}

// How many 256ths of its rounds a layer fills in synced workgroups of kSyncBlock lanes with
// v neurons each, one workgroup to a CU.
inline int64_t sync_fill(int64_t N, int v) {
    const int64_t wgs = (N / v + kSyncBlock - 1) / kSyncBlock, cus = 256;
    return wgs == 0 ? 0 : 256 * wgs / (((wgs + cus - 1) / cus) * cus);
}

// A layer whose plan double-buffers runs its backward in such workgroups where they fill four
// fifths of their rounds: fp32 T = 40, N = 450K / 900K 45.5 -> 40.1 / 87.6 -> 77.9 us, T = 256,
// N = 1M 589 -> 554 us, bf16 T = 96, N = 450K / 950K 63.4 -> 55.4 / 142 -> 117 us; less filled,
// fp32 T = 96, N = 1.15M (0.73) 272 -> 281 us.  Not up to two full chunks (170 sizes of T = 17 to
// 32: 1.01 times as fast on average and 0.79-1.16 each, [19][2096128] 109 -> 138 us); up to three
// (T = 33 to 48: 1.07, 0.93-1.2) not within 2^14 neurons of a multiple of 2^19, whose fp32 rows
// share memory channels ([44][2088960] bf16 0.93, [37][2096128] fp32 0.93); nor on rows exactly
// a multiple of 2 MiB ([96][2^19] fp32 0.89).
inline bool sync_backward(const snn_lif_cfg* c, int64_t T, int64_t N) {
    const int64_t span = int64_t(1) << 19, off = N % span, near = off < span - off ? off : span - off;
    return 5 * sync_fill(N, 2) >= 4 * 256 && (T > 48 || (T > 32 && near >= int64_t(1) << 14)) &&
           (N * io_bytes(c)) % (int64_t(2) << 20) != 0;
}

// The fp32 forward of long layers takes 4 neurons per lane and 4 rows at a time in such
// workgroups where they fill 0.85 of their rounds, 0.9 of two rounds: T = 200, N = 900K / 1M /
// 3M 190 -> 161 / 214 -> 182 / 604 -> 574 us, T = 64, N = 1M / 3M / 6M 58.2 -> 57.0 / 207 -> 194
// / 405 -> 390 us; less filled, T = 64, N = 1.5M / 2.2M (0.71 / 0.70) 91.5 -> 95.0 / 153 -> 160
// us; 0.85-0.9 of two rounds (69 sizes, rows of about 7 MiB) 1.00 times as fast on average and
// 0.84-1.15 each (T = 128, N = 1835008 0.84, T = 80, N = 1859968 106 -> 116 us), while one round
// and three to six gain 2-23% there.  Not on rows 16 MiB apart (T = 64, N = 2^22 260.6 -> 266.8
// us) nor for fewer steps (T = 32, N = 1.5M 45.0 -> 48.0 us).
inline bool wide_sync_forward(const snn_lif_cfg* c, int64_t T, int64_t N) {
    const bool two_rounds = N > 4 * kSyncBlock * int64_t(256) && N <= 8 * kSyncBlock * int64_t(256);
    return c->io == SNN_IO_F32 && T >= 64 && N % 4 == 0 && 100 * sync_fill(N, 4) >= (two_rounds ? 90 : 85) * 256 &&
           (N * 4) % (int64_t(16) << 20) != 0;
}

// bf16 layers of several chunks whose N is no multiple of 8 take 8 neurons per lane in the
// forward where the synced workgroups fill their rounds.  Even N, in place of 2 per lane, from
// 0.62, with byte spikes 0.9: bit spikes 1.05-1.35 times as fast, spikes in the I/O dtype
// 1.0-1.24, byte spikes 0.98-1.17; less filled, byte spikes 0.79-1.0 ([204][2448302] 340 -> 428
// us, [90][4288218] 268 -> 306 us), bit spikes [136][2149282] 187 -> 204 us.  Odd N, in place of
// one, always but for byte spikes under 0.62, where 8 per lane are 0.86-1.03 times as fast
// ([50][2203833] 78.8 -> 91.7 us) and 2 per lane 1.03-1.27.
inline bool ragged_forward_fills(const snn_lif_cfg* c, int64_t N) {
    const bool odd = N % 2 != 0, u8 = c->spk == SNN_SPK_U8;
    return 100 * sync_fill(N, 8) >= (odd ? (u8 ? 62 : 0) : (u8 ? 90 : 62)) * 256;
}

inline Plan make_plan(const snn_lif_cfg* c, int64_t T, int64_t N) {
    Plan p;
    // 2 neurons per lane (fp32 8-byte rows: 4 per lane measured 1% slower on large layers;
    // bf16 4-byte rows with 32-step chunks: faster than 4 per lane with 16-step chunks),
    // except bf16 layers of at most 16 steps that fill the chip: 4 per lane, 8-byte rows
    p.vb = N % 2 != 0 ? 1 : 2;
    if (c->io == SNN_IO_BF16 && T <= 16 && N % 4 == 0 && N / 4 >= kFillLanes) p.vb = 4;
    p.pipe = T > chunk_steps(p.vb) && N / p.vb < 4 * kFillLanes;
    p.k = chunk_steps(p.vb);
    if (!p.pipe && c->io == SNN_IO_BF16 && p.vb == 2) p.k = 32;
    if (T <= p.k) {
        for (int k : kShortChunks) {
            if (T <= k && k < p.k) {
                p.k = k;
                break;
            }
        }
    }
    // bf16 forward: 8 neurons per lane (16-byte rows, whole spike bytes) on large layers
    p.vf = (c->io == SNN_IO_BF16 && N % 8 == 0 && N / 8 >= kFillLanes) ? 8 : p.vb;
    const bool long_walk = !p.pipe && T > p.k;   // several chunks, not double-buffered
    p.blkf = long_walk && p.vf >= 2 ? kSyncBlock : kBlock;   // the lane widths measured
    p.blkb = long_walk && p.vb == 2 ? kSyncBlock : kBlock;
    p.syncb = c->io == SNN_IO_F32 || (T + p.k - 1) / p.k <= kSyncBf16Chunks;
    const bool small = T > p.k && N <= kNarrowN;
    p.narrow = small && narrow_forward(c, T, N, p.k, false);
    p.relay = small && relay_backward(c, T, N, p.k);
    // bf16 rows are read 2 (large layers 8 and 4) neurons per lane whatever N is, a vector
    // needing only its elements' alignment; 2-byte loads, and chunks of 32 single neurons
    // whose tail waits at every row, cost far more than unaligned vectors: forward / backward
    // of x[20][1010625] 25.3 -> 20.8 / 96.8 -> 30.0 us, [40][300001] 22.0 -> 15.0 / 66.7 -> 21.0
    // us, [17][3897755] (bit spikes) 50.2 -> 28.1 / 314 -> 88.6 us, [64][4000002] (bit spikes,
    // 8 instead of 2 per lane forward) 139 -> 112 us.  fp32 rows of odd N keep one neuron, a
    // dword, per lane.  So do few bf16 neurons, which leave lanes idle: narrow layers, and of
    // one-chunk layers as small the forward (350 sizes of 2-32 steps: two per lane 0.81-1.2
    // times as fast, 0.95 on average; [15][1587] 4.4 -> 5.2 us; up to 8 steps also to 2^17
    // neurons, 0.97 on average of 30 sizes, [7][90825] 3.2 -> 3.5 us) and the backward of a whole
    // chunk ([32][4929] 4.7 -> 6.1 us) or of less than four waves; the backward of a partial
    // chunk gains there too ([20][1201] 12.1 -> 9.7 us).
    p.rf = p.rb = 0;
    if (c->io == SNN_IO_BF16) {
        const int wf = N / 8 >= kFillLanes && (T <= p.k || ragged_forward_fills(c, N)) ? 8 : 2;
        const int wb = T <= 16 && N / 4 >= kFillLanes ? 4 : 2;
        const bool few = N <= kNarrowN;
        p.rf = N > (T <= 8 ? int64_t(1) << 17 : kNarrowN) && wf > p.vf ? wf : 0;
        p.rb = (!few || (T < p.k && N >= 4 * kWave)) && wb > p.vb ? wb : 0;
    }
    p.midsync = p.pipe && p.vb == 2 && sync_backward(c, T, N);
    p.widef = p.k == chunk_steps(2) && wide_sync_forward(c, T, N);
    p.row_bytes = spike_row_bytes(c, N);
    return p;
}

// The layer fed by the previous layer's spikes reads one spike word per lane and row (2-8
// bytes) where the dense layer reads an I/O row of 8-16 bytes, so double-buffering its
// chunks costs more in occupancy than it hides, but for the few lanes of a narrow layer
// (fp32 backward: 191 instead of 79 VGPRs, 2 instead of 6 waves per SIMD; forward 127
// instead of 69).  Its chunks are single-buffered at the dense layer's chunk length, so the
// checkpoint layout and snn_lif_saved_bytes stay the dense layer's.  At N = 2^19 (event
// timing, three alternating rounds): fp32 u8 spikes,
// T = 32: forward 10.2 instead of 10.5 us, backward 29.7-29.9 instead of 30.7-31.0 us; bf16
// bit spikes, T = 32: 11.1 instead of 11.8 us and 18.6 instead of 19.6-19.8 us; bf16 u8,
// T = 64: backward 32.8 instead of 35.7-36.0 us, forward within 1%.
inline Plan make_gain_plan(const snn_lif_cfg* c, int64_t T, int64_t N) {
    Plan p = make_plan(c, T, N);
    p.pipe = false;
    p.narrow = T > p.k && N <= kNarrowN && narrow_forward(c, T, N, p.k, true);
    return p;
}

// A stack of L layers fused across depth (lif_stack_*_kernel): 16-step chunks -- L
// membranes per neuron and step in the backward's VGPRs -- or the shortest of kShortChunks
// that holds a short layer.  One neuron per lane on layers of up to kStackNarrowN neurons:
// the 3-layer backward then needs 77 VGPRs instead of 151, twice the waves hide the
// latency of its load-then-compute chunks, and it ran 5-13% faster than with 2 neurons per
// lane at 2^18-2^20 neurons (x[32][B*4096], B = 64-256; 2 layers 2-7%; below 2^18 the two
// are within the run-to-run spread); beyond that the 8-byte rows of 2 neurons per lane (1
// when N is odd) are as fast or faster (B = 768-2048).
constexpr int kMaxStackLayers = 3;
constexpr int64_t kStackNarrowN = 4 * kFillLanes;

struct StackPlan {
    int v;
    int k;
    int64_t row_bytes;
};

inline StackPlan make_stack_plan(const snn_lif_cfg* c, int64_t T, int64_t N) {
    StackPlan p;
    p.v = N % 2 != 0 || N <= kStackNarrowN ? 1 : 2;
    p.k = 16;
    for (int k : kShortChunks) {
        if (T <= k && k < p.k) {
            p.k = k;
            break;
        }
    }
    p.row_bytes = spike_row_bytes(c, N);
    return p;
}

inline int64_t stack_saved_bytes(const StackPlan& p, int L, int64_t T, int64_t N) {
    const int64_t chunks = (T + p.k - 1) / p.k;
    return chunks > 1 ? (chunks - 1) * L * N * int64_t(sizeof(float)) : 0;
}

inline int64_t saved_bytes(const Plan& p, int64_t T, int64_t N) {
    const int64_t chunks = (T + p.k - 1) / p.k;
    return chunks > 1 ? (chunks - 1) * N * int64_t(sizeof(float)) : 0;
}

inline LifK kernel_consts(const snn_lif_cfg* c) {
    LifK k;
    k.k = c->decay;
    k.th = c->v_th;
    k.rest = c->v_reset;
    k.alpha = c->alpha;
    k.c_exp = float(-double(c->alpha) * 1.4426950408889634074);  // -alpha log2(e)
    k.kth = c->decay * c->v_th;
    return k;
}

inline dim3 grid_for(int64_t lanes, int blk = kBlock) { return dim3(unsigned((lanes + blk - 1) / blk)); }

// V-wide lanes over the whole vectors of N, and a workgroup for the rest, if any.
template <int SPK, int V>
dim3 wide_grid(int64_t N, int blk = kBlock) {
    const int64_t whole = whole_vectors<SPK, V>(N);
    return dim3(unsigned((whole / V + blk - 1) / blk + (whole < N)));
}

template <typename Tuple, size_t... I>
void fill_argv(Tuple& t, void** argv, std::index_sequence<I...>) {
    ((argv[I] = static_cast<void*>(&std::get<I>(t))), ...);
}

// Launch through hipLaunchKernel so the runtime's verdict is returned directly and the
// caller's sticky error state is left alone.
template <typename... P, typename... A>
snn_status launch_blk(void (*kernel)(P...), dim3 grid, int blk, hipStream_t stream, A... a) {
    static_assert(sizeof...(P) == sizeof...(A), "argument count");
    std::tuple<P...> args(a...);
    void* argv[sizeof...(P)];
    fill_argv(args, argv, std::index_sequence_for<P...>{});
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(blk), argv, 0, stream);
    return e == hipSuccess ? SNN_OK : SNN_E_LAUNCH;
}

template <typename... P, typename... A>
snn_status launch(void (*kernel)(P...), dim3 grid, hipStream_t stream, A... a) {
    return launch_blk(kernel, grid, kBlock, stream, a...);
}

template <int I>
using IntC = std::integral_constant<int, I>;

// Rows per load batch of the forward.  The forward never revisits a row, so it need not
// hold a whole 32-step chunk (the checkpoint interval) in registers: it loads 16 rows at a
// time and checkpoints after every second batch.
constexpr int forward_batch(int io, int v, int k, bool pipe) {
    return (!pipe && k > 16) ? 16 : k;
}

// Ragged layers (bf16): V neurons per lane, single-buffered chunks of the plan's length, in
// kSyncBlock workgroups (SYNC) where layers of their size take them.
template <int V, int K, bool SYNC, typename F>
snn_status ragged_blocks(bool sync_block, F&& f) {
    if constexpr (K == 32 && SYNC) {
        if (sync_block) return f(IntC<V>{}, IntC<K>{}, IntC<kSyncBlock>{});
    }
    return f(IntC<V>{}, IntC<K>{}, IntC<kBlock>{});
}

template <int V, bool SYNC, typename F>
snn_status ragged_variant(const Plan& p, bool sync_block, F&& f) {
    switch (p.k) {
        case 4: return ragged_blocks<V, 4, SYNC>(sync_block, f);
        case 8: return ragged_blocks<V, 8, SYNC>(sync_block, f);
        case 16: return ragged_blocks<V, 16, SYNC>(sync_block, f);
        case 32: if constexpr (V != 4) return ragged_blocks<V, 32, SYNC>(sync_block, f);
                 break;
    }
    return SNN_E_UNSUPPORTED;
}

// The chunk lengths of a narrow layer: those of the plans of 2 neurons (even N) and of 1.
template <typename F>
snn_status narrow_variant(const Plan& p, F&& f) {
    switch (p.k) {
        case chunk_steps(2): return f(IntC<chunk_steps(2)>{});
        case chunk_steps(1): return f(IntC<chunk_steps(1)>{});
    }
    return SNN_E_UNSUPPORTED;
}

// Calls f(V, K, PIPE) -- std::integral_constant / bool_constant tags -- with the lane width
// and chunk length the plan chose for the forward (vf) or the backward (vb): the
// combinations a kernel translation unit instantiates.
template <int IO, int V, typename F>
snn_status chunk_variant(const Plan& p, F&& f) {
    if (p.pipe) {   // few lanes: none wider than 2
        if constexpr (V <= 2) {
            constexpr int K = chunk_steps(V);
            if (p.k == K) return f(IntC<V>{}, IntC<K>{}, std::true_type{});
        }
        return SNN_E_UNSUPPORTED;   // no plan pairs another chunk with these lanes
    }
    switch (p.k) {   // the long chunks, and the single-chunk layers of kShortChunks
        case 4: return f(IntC<V>{}, IntC<4>{}, std::false_type{});
        case 8: return f(IntC<V>{}, IntC<8>{}, std::false_type{});
        case 16: return f(IntC<V>{}, IntC<16>{}, std::false_type{});
        case 32: if constexpr (V == 1 || (IO == SNN_IO_BF16 && V != 4)) return f(IntC<V>{}, IntC<32>{}, std::false_type{});
                 break;
    }
    return SNN_E_UNSUPPORTED;
}

// Lane widths: 2 or 1; bf16 also 4 (short layers) and 8 (the forward of large layers).
template <int IO, typename F>
snn_status forward_variant(const Plan& p, F&& f) {
    switch (p.vf) {
        case 8: if constexpr (IO == SNN_IO_BF16) return chunk_variant<IO, 8>(p, f); break;
        case 4: if constexpr (IO == SNN_IO_BF16) return chunk_variant<IO, 4>(p, f); break;
        case 2: return chunk_variant<IO, 2>(p, f);
        case 1: return chunk_variant<IO, 1>(p, f);
    }
    return SNN_E_UNSUPPORTED;
}

template <int IO, typename F>
snn_status backward_variant(const Plan& p, F&& f) {
    switch (p.vb) {
        case 4: if constexpr (IO == SNN_IO_BF16) return chunk_variant<IO, 4>(p, f); break;
        case 2: return chunk_variant<IO, 2>(p, f);
        case 1: return chunk_variant<IO, 1>(p, f);
    }
    return SNN_E_UNSUPPORTED;
}

// The kernels of a plan: each of the following calls its functor with the tags of the one
// kernel that the plan launches, and is the only place where the plan's switches are weighed
// against each other.
//
// The dense forward: f(V, FB, K, PIPE, BLK, RAGGED) -- neurons per lane, rows per load batch,
// steps per chunk, double-buffered, workgroup size, N no multiple of V.
template <int IO, typename F>
snn_status forward_route(const Plan& p, int64_t T, int64_t N, F&& f) {
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr int kLong = IO == SNN_IO_F32 ? chunk_steps(2) : 32;   // the chunk of layers not double-buffered
    if (p.narrow) return narrow_variant(p, [&](auto K) { return f(IntC<1>{}, K, K, yes, IntC<kWave>{}, no); });
    if constexpr (IO == SNN_IO_F32) {
        if (p.widef) return f(IntC<4>{}, IntC<4>{}, IntC<chunk_steps(2)>{}, no, IntC<kSyncBlock>{}, no);
    } else {
        auto ragged = [&](auto V, auto K, auto blk) {
            constexpr int FB = forward_batch(IO, decltype(V)::value, decltype(K)::value, false);
            return f(V, IntC<FB>{}, K, no, blk, yes);
        };
        const bool sync_block = T > p.k && N / 2 >= 4 * kFillLanes;
        if (p.rf == 8) return ragged_variant<8, true>(p, sync_block, ragged);
        if (p.rf == 2) return ragged_variant<2, false>(p, false, ragged);   // fewer than fill the chip
    }
    return forward_variant<IO>(p, [&](auto V, auto K, auto PIPE) -> snn_status {
        constexpr int Vc = decltype(V)::value, Kc = decltype(K)::value;
        constexpr bool Pc = decltype(PIPE)::value;
        constexpr IntC<forward_batch(IO, Vc, Kc, Pc)> FB{};
        if constexpr (!Pc && Vc >= 2 && Kc == kLong) {
            if (p.blkf == kSyncBlock) return f(V, FB, K, PIPE, IntC<kSyncBlock>{}, no);
        }
        // bf16 layers of odd N and several chunks are narrow or ragged; a single 32-step chunk
        // of even N takes 8 neurons per lane
        if constexpr (IO == SNN_IO_BF16 && ((Vc == 1 && Pc) || (Vc == 2 && Kc == 32))) return SNN_E_UNSUPPORTED;
        else return f(V, FB, K, PIPE, IntC<kBlock>{}, no);
    });
}

// The dense backward: f(V, K, PIPE, BLK, SYNC, RAGGED), SYNC for the barriers, or relay(K).
template <int IO, typename F, typename G>
snn_status backward_route(const Plan& p, int64_t T, int64_t N, F&& f, G&& relay) {
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr int kLong = IO == SNN_IO_F32 ? chunk_steps(2) : 32;
    if (p.relay) return narrow_variant(p, relay);
    if constexpr (IO == SNN_IO_BF16) {
        auto ragged = [&](auto V, auto K, auto blk) {
            if constexpr (decltype(blk)::value == kSyncBlock) {
                if (p.syncb) return f(V, K, no, blk, yes, yes);
            }
            return f(V, K, no, blk, no, yes);
        };
        const bool sync_block = T > p.k && N / 2 >= 4 * kFillLanes;
        if (p.rb == 4) return ragged_variant<4, false>(p, false, ragged);   // one chunk
        if (p.rb == 2) return ragged_variant<2, true>(p, sync_block, ragged);
    }
    if (p.midsync) return f(IntC<2>{}, IntC<chunk_steps(2)>{}, no, IntC<kSyncBlock>{}, yes, no);
    return backward_variant<IO>(p, [&](auto V, auto K, auto PIPE) {
        if constexpr (!decltype(PIPE)::value && decltype(V)::value == 2 && decltype(K)::value == kLong) {
            if (p.blkb == kSyncBlock) {
                if constexpr (IO == SNN_IO_BF16) {
                    if (!p.syncb) return f(V, K, PIPE, IntC<kSyncBlock>{}, no, no);
                }
                return f(V, K, PIPE, IntC<kSyncBlock>{}, yes, no);
            }
        }
        return f(V, K, PIPE, IntC<kBlock>{}, no, no);
    });
}

// The gain-fed layer, single-buffered but for the narrow forward: f(V, FB, K, PIPE, BLK), and
// f(V, K) or relay(K).
template <int IO, typename F>
snn_status forward_gain_route(const Plan& p, F&& f) {
    if (p.narrow)
        return narrow_variant(p, [&](auto K) { return f(IntC<1>{}, K, K, std::true_type{}, IntC<kWave>{}); });
    return forward_variant<IO>(p, [&](auto V, auto K, auto PIPE) -> snn_status {
        if constexpr (decltype(PIPE)::value) {
            return SNN_E_UNSUPPORTED;
        } else {
            constexpr IntC<forward_batch(IO, decltype(V)::value, decltype(K)::value, false)> FB{};
            return f(V, FB, K, PIPE, IntC<kBlock>{});
        }
    });
}

template <int IO, typename F, typename G>
snn_status backward_gain_route(const Plan& p, F&& f, G&& relay) {
    if (p.relay) return narrow_variant(p, relay);
    return backward_variant<IO>(p, [&](auto V, auto K, auto PIPE) -> snn_status {
        if constexpr (decltype(PIPE)::value) return SNN_E_UNSUPPORTED;
        else return f(V, K);
    });
}

// The dense forward's grid.  A workgroup's neurons are whole words of bit-packed spikes, so
// the lanes that complete the last word are in the last workgroup.
template <int SPK, int V, bool RAGGED>
dim3 forward_grid(int64_t N, int blk) {
    static_assert(kBlock % kWave == 0 && kSyncBlock % kWave == 0);
    if constexpr (RAGGED) return wide_grid<SPK, V>(N, blk);
    else return grid_for((N + V - 1) / V, blk);
}

// v_in / v_last / g_in / g_out: the segment state of a sequence split along time (each may
// be null; see snn_lif_forward_seg and snn_lif_backward_seg).
template <int IO, int SPK>
snn_status forward_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, const void* x,
                         void* spikes, void* saved, float* v_out, const float* v_in, float* v_last,
                         hipStream_t s);

template <int IO>
snn_status backward_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, const void* x,
                          const void* saved, const void* gs, void* gx, const float* v_in, const float* g_in,
                          float* g_out, hipStream_t s);

// The layer fed by the previous layer's spikes (format SPK, u8 or bits) through a per-feature
// gain of F features.
template <int IO, int SPK>
snn_status forward_gain_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, int64_t F,
                              const void* spikes_in, const float* gain, void* spikes, void* saved, float* v_out,
                              hipStream_t s);

template <int IO, int SPK>
snn_status backward_gain_entry(int reset, const Plan& p, const LifK& k, int64_t T, int64_t N, int64_t F,
                               const void* spikes_in, const float* gain, const void* saved, const void* gs,
                               void* gs_in, hipStream_t s);

// The stack fused across depth: gains is [L-1][F]; hidden and v_out may be null.
template <int IO, int SPK>
snn_status stack_forward_entry(int reset, int L, const StackPlan& p, const LifK& k, int64_t T, int64_t N, int64_t F,
                               const void* x, const float* gains, void* spikes, void* hidden, void* saved,
                               float* v_out, hipStream_t s);

template <int IO>
snn_status stack_backward_entry(int reset, int L, const StackPlan& p, const LifK& k, int64_t T, int64_t N, int64_t F,
                                const void* x, const float* gains, const void* saved, const void* gs, void* gx,
                                hipStream_t s);

snn_status gain_forward_entry(const snn_lif_cfg* c, int64_t T, int64_t N, int64_t F, const void* spikes,
                              int64_t row_bytes, const float* gain, void* x_next, hipStream_t s);

snn_status gain_backward_entry(const snn_lif_cfg* c, int64_t T, int64_t N, int64_t F, const void* gx_next,
                               const float* gain, void* gs, hipStream_t s);

snn_status serial_forward_entry(const snn_lif_cfg* c, const LifK& k, int64_t N, const void* x_t,
                                const float* v_prev, float* v_t, void* spikes_t, hipStream_t s);

snn_status serial_backward_entry(const snn_lif_cfg* c, const LifK& k, int64_t N, const float* v_t, const void* gs_t,
                                 const float* g_next, void* gx_t, float* g_out, hipStream_t s);

}  // namespace snnlif
