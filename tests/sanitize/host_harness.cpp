// Host-only driver for AddressSanitizer / UndefinedBehaviorSanitizer runs, built with g++
// (no GPU code): the library's argument checks and lane/chunk planners (lif_host.h), and the
// CPU oracle (oracle/lif_oracle.c, built with gcc beside it).  Every plan the planner can
// return must map to an instantiated kernel variant, cover every neuron and size its
// checkpoint buffer without overflow; the oracle runs on ragged, empty and non-finite
// inputs.  Exit status 0 when every invariant holds (the sanitizers abort on their own
// findings).
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <limits>
#include <vector>

#include "lif_host.h"

extern "C" {
#include "lif_oracle.h"
}

using namespace snnlif;

static int failures = 0;

#define CHECK(cond)                                                                  \
    do {                                                                             \
        if (!(cond)) {                                                               \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            ++failures;                                                              \
        }                                                                            \
    } while (0)

static snn_lif_cfg cfg(float decay, float th, int reset, int io, int spk) {
    snn_lif_cfg c;
    c.decay = decay;
    c.v_th = th;
    c.v_reset = 0.0f;
    c.alpha = 4.0f;
    c.reset = reset;
    c.io = io;
    c.spk = spk;
    return c;
}

static void check_cfgs() {
    const float nan = std::numeric_limits<float>::quiet_NaN(), inf = std::numeric_limits<float>::infinity();
    CHECK(check_cfg(nullptr) == SNN_E_NULL);
    snn_lif_cfg c = cfg(0.5f, 1.0f, SNN_RESET_HARD, SNN_IO_F32, SNN_SPK_U8);
    CHECK(check_cfg(&c) == SNN_OK);
    for (float d : {-0.01f, 1.01f, nan, inf, -inf}) {
        snn_lif_cfg b = c;
        b.decay = d;
        CHECK(check_cfg(&b) == SNN_E_PARAM);
    }
    for (float d : {0.0f, 1.0f}) {
        snn_lif_cfg b = c;
        b.decay = d;
        CHECK(check_cfg(&b) == SNN_OK);
    }
    for (float v : {nan, inf, -inf}) {
        snn_lif_cfg b = c;
        b.v_th = v;
        CHECK(check_cfg(&b) == SNN_E_PARAM);
        b = c;
        b.v_reset = v;
        CHECK(check_cfg(&b) == SNN_E_PARAM);
    }
    for (float a : {0.0f, -1.0f, nan, inf}) {
        snn_lif_cfg b = c;
        b.alpha = a;
        CHECK(check_cfg(&b) == SNN_E_PARAM);
    }
    for (int e : {-1, 2, 1 << 30, std::numeric_limits<int>::min()}) {
        snn_lif_cfg b = c;
        b.reset = e;
        CHECK(check_cfg(&b) == SNN_E_PARAM);
        b = c;
        b.io = e;
        CHECK(check_cfg(&b) == SNN_E_PARAM);
        b = c;
        b.spk = e + 1;   // 3 and up are out of range; 0..2 are formats
        if (e + 1 < 0 || e + 1 > 2) CHECK(check_cfg(&b) == SNN_E_PARAM);
    }
}

static void check_shapes() {
    CHECK(check_shape(0, 0) == SNN_OK);
    CHECK(check_shape(-1, 1) == SNN_E_SHAPE);
    CHECK(check_shape(1, -1) == SNN_E_SHAPE);
    CHECK(check_shape(kMaxT, 1) == SNN_OK);
    CHECK(check_shape(kMaxT + 1, 1) == SNN_E_SHAPE);
    CHECK(check_shape(1, kMaxN) == SNN_OK);
    CHECK(check_shape(1, kMaxN + 1) == SNN_E_SHAPE);
    CHECK(check_shape(int64_t(1) << 13, kMaxN) == SNN_OK);          // T N = 2^44
    CHECK(check_shape((int64_t(1) << 13) + 1, kMaxN) == SNN_E_SHAPE);
    CHECK(check_shape(kMaxT, kMaxN) == SNN_E_SHAPE);
    CHECK(check_shape(std::numeric_limits<int64_t>::max(), 2) == SNN_E_SHAPE);
    CHECK(check_shape(2, std::numeric_limits<int64_t>::max()) == SNN_E_SHAPE);
}

// What is launched: the functors below take the place of the launchers and check the one
// kernel and grid that each route picks.

// The lanes of grid x blk workgroups, v neurons each, cover `end` and no workgroup more.
static void check_grid(dim3 grid, int blk, int v, int64_t end) {
    CHECK(grid.y == 1 && grid.z == 1);
    CHECK(int64_t(grid.x) * blk * v >= end);
    CHECK((int64_t(grid.x) - 1) * blk * v < end);
}

// wide_grid: whole vectors (whole spike words), and one workgroup for a rest smaller than it.
template <int SPK, int V>
static void check_wide_grid(dim3 grid, int blk, int64_t N) {
    const int64_t whole = whole_vectors<SPK, V>(N), rest = N - whole;
    CHECK(whole >= 0 && rest >= 0 && rest < blk && whole % V == 0);
    if (SPK == SNN_SPK_BITS && V > 1) CHECK(whole % kWave == 0);
    if (rest == 0) return check_grid(grid, blk, V, whole);
    CHECK(whole % V == 0 && grid.x >= 1);
    if (whole == 0) CHECK(grid.x == 1);
    else check_grid(dim3(grid.x - 1), blk, V, whole);
}

template <int SPK>
struct ForwardProbe {
    const Plan& p;
    int64_t T, N;
    template <typename V, typename FB, typename K, typename P, typename B, typename Q>
    snn_status operator()(V, FB, K, P, B, Q) const {
        constexpr int v = V::value, blk = B::value;
        CHECK(K::value == p.k && p.k % FB::value == 0);           // checkpoints after whole batches
        if (P::value) CHECK(FB::value == K::value && T > p.k);
        if (blk > kBlock) CHECK(!P::value && T > p.k);            // barriers: several chunks
        const dim3 g = forward_grid<SPK, v, Q::value>(N, blk);
        if (Q::value) {
            check_wide_grid<SPK, v>(g, blk, N);
        } else {
            CHECK(N % v == 0);                                    // lanes never straddle the row end
            check_grid(g, blk, v, SPK == SNN_SPK_BITS ? p.row_bytes * 8 : N);   // every spike word written
        }
        return SNN_OK;
    }
};

struct BackwardProbe {
    const Plan& p;
    int64_t T, N;
    template <typename V, typename K, typename P, typename B, typename S, typename Q>
    snn_status operator()(V, K, P, B, S, Q) const {
        constexpr int v = V::value, blk = B::value;
        CHECK(K::value == p.k);                                   // reads the forward's checkpoints
        if (P::value) CHECK(T > p.k);
        if (S::value) CHECK(blk > kBlock && !P::value && T > p.k);
        if (!Q::value) CHECK(N % v == 0);
        check_wide_grid<SNN_SPK_IO, v>(wide_grid<SNN_SPK_IO, v>(N, blk), blk, N);
        return SNN_OK;
    }
};

struct RelayProbe {
    const Plan& p;
    int64_t T, N;
    template <typename K>
    snn_status operator()(K) const {
        CHECK(K::value == p.k && T > p.k);                        // at least two waves take turns
        check_grid(grid_for(N, kWave), kWave, 1, N);
        return SNN_OK;
    }
};

template <int SPK>
struct GainForwardProbe {
    const Plan& p;
    int64_t N;
    template <typename V, typename FB, typename K, typename P, typename B>
    snn_status operator()(V, FB, K, P, B) const {
        CHECK(K::value == p.k && p.k % FB::value == 0 && N % V::value == 0);
        check_wide_grid<SPK, V::value>(wide_grid<SPK, V::value>(N, B::value), B::value, N);
        return SNN_OK;
    }
};

struct GainBackwardProbe {
    const Plan& p;
    int64_t N;
    template <typename V, typename K>
    snn_status operator()(V, K) const {
        CHECK(K::value == p.k && N % V::value == 0);
        check_grid(grid_for((N + V::value - 1) / V::value), kBlock, V::value, N);
        return SNN_OK;
    }
};

template <int IO, int SPK>
static void check_routes(const snn_lif_cfg& c, int64_t T, int64_t N) {
    const Plan p = make_plan(&c, T, N), gp = make_gain_plan(&c, T, N);
    const snn_status st[] = {forward_route<IO>(p, T, N, ForwardProbe<SPK>{p, T, N}),
                             backward_route<IO>(p, T, N, BackwardProbe{p, T, N}, RelayProbe{p, T, N}),
                             forward_gain_route<IO>(gp, GainForwardProbe<SPK>{gp, N}),
                             backward_gain_route<IO>(gp, GainBackwardProbe{gp, N}, RelayProbe{gp, T, N})};
    for (snn_status s : st) {
        if (s != SNN_OK)
            std::fprintf(stderr, "no kernel: route %d io %d spk %d T %lld N %lld vf %d vb %d k %d\n", int(&s - st), IO,
                         SPK, (long long)T, (long long)N, p.vf, p.vb, p.k);
        CHECK(s == SNN_OK);
    }
    const StackPlan sp = make_stack_plan(&c, T, N);
    if (sp.v == 2) check_wide_grid<SPK, 2>(wide_grid<SPK, 2>(N), kBlock, N);
    else check_wide_grid<SPK, 1>(wide_grid<SPK, 1>(N), kBlock, N);
}

static void check_plan(const snn_lif_cfg& c, int64_t T, int64_t N) {
    const Plan p = make_plan(&c, T, N);
    CHECK(p.vf == 1 || p.vf == 2 || p.vf == 4 || p.vf == 8);
    CHECK(p.vb == 1 || p.vb == 2 || p.vb == 4);
    CHECK(N % p.vb == 0 && N % p.vf == 0);
    CHECK(p.k == 4 || p.k == 8 || p.k == 16 || p.k == 32);
    CHECK(p.blkf == kBlock || p.blkf == kSyncBlock);
    CHECK(p.blkb == kBlock || p.blkb == kSyncBlock);
    if (p.blkf == kSyncBlock) CHECK(!p.pipe && T > p.k);
    if (p.blkb == kSyncBlock) CHECK(!p.pipe && T > p.k && p.vb == 2);
    // one plan takes the place of vf, one that of vb, with the chunks it reads checkpoints by
    CHECK(int(p.narrow) + int(p.widef) + int(p.rf > 0) <= 1);
    CHECK(int(p.relay) + int(p.midsync) + int(p.rb > 0) <= 1);
    if (p.widef) CHECK(p.k == 16 && N % 4 == 0 && c.io == SNN_IO_F32);
    if (p.midsync) CHECK(p.k == 16 && p.vb == 2 && p.pipe);
    if (p.rb == 4) CHECK(p.k <= 16);
    if (p.narrow || p.relay) CHECK(T > p.k && N <= kNarrowN);
    CHECK(p.row_bytes == spike_row_bytes(&c, N));
    const int64_t chunks = (T + p.k - 1) / p.k;
    CHECK(saved_bytes(p, T, N) == (chunks > 1 ? (chunks - 1) * N * 4 : 0));
    CHECK(saved_bytes(p, T, N) <= 4 * T * N);
    // the gain-fed layer: single-buffered chunks of the same length, so the same checkpoints
    const Plan gp = make_gain_plan(&c, T, N);
    CHECK(!gp.pipe && gp.k == p.k && gp.vf == p.vf && gp.vb == p.vb);
    CHECK(saved_bytes(gp, T, N) == saved_bytes(p, T, N));
    switch (c.io * 4 + c.spk) {
        case SNN_IO_F32 * 4 + SNN_SPK_U8: check_routes<SNN_IO_F32, SNN_SPK_U8>(c, T, N); break;
        case SNN_IO_F32 * 4 + SNN_SPK_BITS: check_routes<SNN_IO_F32, SNN_SPK_BITS>(c, T, N); break;
        case SNN_IO_F32 * 4 + SNN_SPK_IO: check_routes<SNN_IO_F32, SNN_SPK_IO>(c, T, N); break;
        case SNN_IO_BF16 * 4 + SNN_SPK_U8: check_routes<SNN_IO_BF16, SNN_SPK_U8>(c, T, N); break;
        case SNN_IO_BF16 * 4 + SNN_SPK_BITS: check_routes<SNN_IO_BF16, SNN_SPK_BITS>(c, T, N); break;
        case SNN_IO_BF16 * 4 + SNN_SPK_IO: check_routes<SNN_IO_BF16, SNN_SPK_IO>(c, T, N); break;
    }
    const StackPlan s = make_stack_plan(&c, T, N);
    CHECK((s.v == 1 || s.v == 2) && N % s.v == 0);
    CHECK(s.k == 4 || s.k == 8 || s.k == 16);
    for (int L = 2; L <= kMaxStackLayers; ++L) {
        const int64_t sc = (T + s.k - 1) / s.k;
        CHECK(stack_saved_bytes(s, L, T, N) == (sc > 1 ? (sc - 1) * L * N * 4 : 0));
    }
}

static uint64_t rng_state = 0x9E3779B97F4A7C15ull;

static double uniform() {   // xorshift64*, for test inputs only
    rng_state ^= rng_state >> 12;
    rng_state ^= rng_state << 25;
    rng_state ^= rng_state >> 27;
    return double((rng_state * 0x2545F4914F6CDD1Dull) >> 11) / double(uint64_t(1) << 53);
}

static void check_all(int64_t T, int64_t N) {
    if (check_shape(T, N) != SNN_OK) return;
    for (int io : {SNN_IO_F32, SNN_IO_BF16})
        for (int spk : {SNN_SPK_U8, SNN_SPK_BITS, SNN_SPK_IO}) check_plan(cfg(0.5f, 1.0f, SNN_RESET_HARD, io, spk), T, N);
}

static void check_plans() {
    const int64_t wave = int64_t(256) * 64;
    std::vector<int64_t> Ns = {1, 2, 3, 7, 63, 64, 65, 1000, 4096, 4097, 131072, 524288, 1000000, 8388608,
                               (int64_t(1) << 22) + 2, 16777216, (int64_t(1) << 24) + 8, (int64_t(1) << 24) + 1,
                               int64_t(1) << 28, kMaxN - 1, kMaxN};
    // around the lines of the plans: waves of neurons per CU, filled rounds of synced
    // workgroups, lanes that fill the chip
    for (int64_t line : {wave, 5 * wave / 2, 3 * wave, 7 * wave / 2, int64_t(66) * 1024, kNarrowN, int64_t(1) << 17,
                         int64_t(891289), int64_t(419430), int64_t(1) << 20, int64_t(1) << 21, int64_t(1) << 22})
        for (int64_t d : {-4, -3, -2, -1, 0, 1, 2, 3, 4, 8, 64}) Ns.push_back(line + d);
    const int64_t Ts[] = {1, 2, 3, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 40, 48, 49, 63, 64, 65, 96, 100, 101, 128, 129,
                          192, 193, 250, 251, 256, 257, 1000};
    for (int64_t N : Ns)
        for (int64_t T : Ts) check_all(T, N);
    for (int i = 0; i < 20000; ++i)
        check_all(int64_t(std::exp(uniform() * std::log(1200.0))), int64_t(std::exp(uniform() * std::log(4e7))));
}

// Sizes at which a plan lost against the general one: the rules keep them on the latter.
static Plan plan_of(int io, int spk, int64_t T, int64_t N) {
    const snn_lif_cfg c = cfg(0.5f, 1.0f, SNN_RESET_HARD, io, spk);
    return make_plan(&c, T, N);
}

static void check_synced_backward_rule() {
    // one full chunk and a tail, two full chunks
    for (int64_t T : {17, 19, 22, 24, 28, 32})
        for (int64_t N : {848294, 1375558, 1572862, 2096128}) CHECK(!plan_of(SNN_IO_F32, SNN_SPK_U8, T, N).midsync);
    // two or three chunks next to a multiple of 2^19 neurons, on either side
    for (int64_t N : {516096, 524290, 1564672, 2088960, 2096128})
        for (int64_t T : {33, 44, 48}) CHECK(!plan_of(SNN_IO_BF16, SNN_SPK_U8, T, N).midsync);
    // where it gains
    for (int64_t N : {450000, 900000, 990000}) CHECK(plan_of(SNN_IO_F32, SNN_SPK_U8, 40, N).midsync);
    for (int64_t N : {450000, 524284, 1000000, 2097146}) CHECK(plan_of(SNN_IO_BF16, SNN_SPK_U8, 96, N).midsync);
}

static void check_wide_forward_rule() {
    for (int64_t N : {1785856, 1819112, 1835004, 1835008, 1859968})   // 0.85-0.9 of two rounds
        for (int64_t T : {64, 128, 200}) CHECK(!plan_of(SNN_IO_F32, SNN_SPK_IO, T, N).widef);
    for (int64_t N : {892476, 935124, 1000000, 1966080, 2097148, 2752512, 3000000})
        CHECK(plan_of(SNN_IO_F32, SNN_SPK_IO, 128, N).widef);
}

static void check_ragged_rule() {
    for (int spk : {SNN_SPK_U8, SNN_SPK_BITS, SNN_SPK_IO}) {
        for (int64_t T : {2, 3, 15, 16, 20, 31, 32})        // few neurons: one per lane forward
            for (int64_t N : {69, 1587, 5463, 65281, 81919}) CHECK(plan_of(SNN_IO_BF16, spk, T, N).rf == 0);
        for (int64_t T : {4, 8, 16, 32})                    // and in the backward of a whole chunk
            for (int64_t N : {75, 741, 4929, 61155}) CHECK(plan_of(SNN_IO_BF16, spk, T, N).rb == 0);
        for (int64_t T : {2, 15, 20}) CHECK(plan_of(SNN_IO_BF16, spk, T, 145).rb == 0);
        for (int64_t T : {3, 15, 20, 31}) CHECK(plan_of(SNN_IO_BF16, spk, T, 1201).rb == 2);
        for (int64_t T : {2, 5, 8}) CHECK(plan_of(SNN_IO_BF16, spk, T, 131071).rf == 0);
        // 8 per lane over several chunks where they fill the chip
        CHECK(plan_of(SNN_IO_BF16, spk, 146, 2208030).rf == 0);
        CHECK(plan_of(SNN_IO_BF16, spk, 90, 4288218).rf == (spk == SNN_SPK_U8 ? 0 : 8));
        CHECK(plan_of(SNN_IO_BF16, spk, 64, 4000002).rf == 8 && plan_of(SNN_IO_BF16, spk, 20, 2208030).rf == 8);
        CHECK(plan_of(SNN_IO_BF16, spk, 50, 2203833).rf == (spk == SNN_SPK_U8 ? 2 : 8));
        CHECK(plan_of(SNN_IO_BF16, spk, 173, 2884353).rf == 8);
        for (int64_t T : {9, 20, 33, 400}) {
            const Plan p = plan_of(SNN_IO_BF16, spk, T, 81921);
            CHECK(p.rf == 2 && p.rb == 2);
        }
    }
}

struct NarrowCase {
    int io, spk;
    int64_t T, N;
    bool dense, gain;
};

static void check_narrow_forward_rule() {
    const NarrowCase cases[] = {
        {SNN_IO_BF16, SNN_SPK_BITS, 44, 77454, false, true},  {SNN_IO_BF16, SNN_SPK_BITS, 26, 57140, false, true},
        {SNN_IO_BF16, SNN_SPK_BITS, 128, 49154, false, true}, {SNN_IO_BF16, SNN_SPK_BITS, 129, 49154, true, true},
        {SNN_IO_BF16, SNN_SPK_BITS, 64, 49152, false, true},  {SNN_IO_BF16, SNN_SPK_BITS, 65, 49152, true, true},
        {SNN_IO_BF16, SNN_SPK_BITS, 17, 16384, true, true},   {SNN_IO_BF16, SNN_SPK_IO, 47, 74240, true, false},
        {SNN_IO_BF16, SNN_SPK_IO, 26, 33820, true, false},    {SNN_IO_BF16, SNN_SPK_IO, 200, 74240, true, true},
        {SNN_IO_F32, SNN_SPK_IO, 389, 76402, false, false},   {SNN_IO_F32, SNN_SPK_IO, 128, 76402, true, true},
        {SNN_IO_F32, SNN_SPK_IO, 389, 65536, false, true},    {SNN_IO_BF16, SNN_SPK_IO, 93, 62985, true, false},
        {SNN_IO_F32, SNN_SPK_IO, 706, 62503, false, false},   {SNN_IO_F32, SNN_SPK_IO, 786, 81919, true, true},
        {SNN_IO_F32, SNN_SPK_U8, 48, 53805, true, false},     {SNN_IO_F32, SNN_SPK_U8, 97, 53805, true, true},
        {SNN_IO_F32, SNN_SPK_U8, 1000, 8192, true, true},     {SNN_IO_BF16, SNN_SPK_U8, 1000, 81920, true, true}};
    for (const NarrowCase& r : cases) {
        const snn_lif_cfg c = cfg(0.5f, 1.0f, SNN_RESET_HARD, r.io, r.spk);
        CHECK(make_plan(&c, r.T, r.N).narrow == r.dense);
        CHECK(make_gain_plan(&c, r.T, r.N).narrow == r.gain);
    }
}

struct RelayCase {
    int io;
    int64_t T, N;
    bool relay;
};

static void check_relay_rule() {
    const RelayCase cases[] = {
        // many steps of more than three waves per CU (two and a half: fp32, odd N)
        {SNN_IO_F32, 765, 69148, false}, {SNN_IO_F32, 176, 80472, false}, {SNN_IO_F32, 983, 54130, false},
        {SNN_IO_BF16, 993, 65778, false}, {SNN_IO_BF16, 890, 78730, false}, {SNN_IO_BF16, 816, 57246, false},
        {SNN_IO_F32, 932, 42301, false}, {SNN_IO_F32, 515, 66958, false}, {SNN_IO_F32, 122, 64023, false},
        {SNN_IO_F32, 64, 49863, false}, {SNN_IO_BF16, 256, 64015, false}, {SNN_IO_BF16, 165, 64357, false},
        // where it gains: up to there, few steps, and odd N past two workgroups on some CUs
        {SNN_IO_F32, 1000, 49152, true}, {SNN_IO_F32, 100, 81920, true}, {SNN_IO_BF16, 250, 81920, true},
        {SNN_IO_F32, 1000, 40959, true}, {SNN_IO_F32, 63, 64001, true}, {SNN_IO_F32, 786, 81919, true},
        {SNN_IO_BF16, 1000, 49151, true}, {SNN_IO_BF16, 400, 76001, true}, {SNN_IO_F32, 17, 2, true}};
    for (const RelayCase& r : cases)
        for (int spk : {SNN_SPK_U8, SNN_SPK_BITS, SNN_SPK_IO}) {
            const snn_lif_cfg c = cfg(0.5f, 1.0f, SNN_RESET_HARD, r.io, spk);
            CHECK(make_plan(&c, r.T, r.N).relay == r.relay);
            CHECK(make_gain_plan(&c, r.T, r.N).relay == r.relay);
        }
}

// ---------------------------------------------------------------- the oracle

static void run_oracle(int64_t T, int64_t B, int64_t F, int soft, bool nonfinite) {
    const int64_t N = B * F, TN = T * N;
    lif_oracle_params p = {0.75f, 1.0f, 0.125f, 4.0f, soft};
    // exact-size heap buffers, so any access past an end is reported
    std::vector<float> x(TN), v(TN), xs(3 * TN), vs(3 * TN), xn(TN), gains(2 * F);
    std::vector<uint8_t> y(TN), ys(3 * TN);
    std::vector<double> gy(TN), gx(TN), ge(TN), gr(TN), sg(3 * TN), se(3 * TN), sr(3 * TN), gn(N);
    for (int64_t i = 0; i < TN; ++i) {
        x[i] = float(2.0 * uniform() - 0.3);
        gy[i] = 2.0 * uniform() - 1.0;
    }
    if (nonfinite && TN >= 3) {
        x[0] = std::numeric_limits<float>::quiet_NaN();
        x[TN / 2] = std::numeric_limits<float>::infinity();
        x[TN - 1] = -std::numeric_limits<float>::infinity();
    }
    for (int64_t f = 0; f < 2 * F; ++f) gains[f] = float(0.5 + 1.5 * uniform());
    for (int64_t n = 0; n < N; ++n) gn[n] = uniform();
    lif_oracle_forward(&p, T, N, x.data(), nullptr, nullptr, y.data(), v.data());
    lif_oracle_backward(&p, T, N, v.data(), y.data(), gy.data(), nullptr, nullptr, gn.data(), gx.data(), ge.data(),
                        gr.data());
    lif_oracle_backward(&p, T, N, v.data(), y.data(), gy.data(), ge.data(), gr.data(), nullptr, gx.data(),
                        ge.data(), nullptr);
    lif_oracle_gain_forward(T, B, F, y.data(), gains.data(), xn.data());
    lif_oracle_gain_backward(T, B, F, gx.data(), ge.data(), gr.data(), gains.data(), gy.data(), ge.data(), gr.data());
    for (int L = 1; L <= 3; ++L) {
        lif_oracle_stack_forward(&p, L, T, B, F, x.data(), gains.data(), xs.data(), ys.data(), vs.data());
        CHECK(lif_oracle_stack_backward(&p, L, T, B, F, vs.data(), ys.data(), gains.data(), gy.data(), L & 1,
                                        sg.data(), se.data(), sr.data()) == 0);
    }
    if (!nonfinite)
        for (int64_t i = 0; i < TN; ++i) CHECK(se[i] >= std::fabs(sg[i]));
}

int main() {
    check_cfgs();
    check_shapes();
    check_plans();
    check_synced_backward_rule();
    check_wide_forward_rule();
    check_narrow_forward_rule();
    check_relay_rule();
    check_ragged_rule();
    const int64_t shapes[][3] = {{0, 1, 1}, {1, 0, 3}, {1, 1, 1}, {2, 3, 5}, {17, 2, 33}, {40, 3, 7}, {5, 1, 1000}};
    for (const auto& s : shapes)
        for (int soft = 0; soft < 2; ++soft)
            for (int nf = 0; nf < 2; ++nf) run_oracle(s[0], s[1], s[2], soft, nf != 0);
    if (failures) {
        std::fprintf(stderr, "%d check(s) failed\n", failures);
        return 1;
    }
    std::printf("host harness: all checks passed\n");
    return 0;
}
