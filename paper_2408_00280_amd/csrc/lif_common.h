// Constants and the kernel-argument struct shared by the host and device code of the
// fused LIF library.
#pragma once
#include <climits>
#include <cstdint>

#include "snn_lif.h"

namespace snnlif {

constexpr int kBlock = 256;  // 4 wave64 per workgroup
constexpr int kWave = 64;

constexpr int64_t kMaxT = INT32_MAX;
constexpr int64_t kMaxN = int64_t(1) << 31;
constexpr int64_t kMaxTN = int64_t(1) << 44;

// The neurons that lanes of V take in layers whose N need not be whole vectors (ragged bf16
// layers) and in the gain-fed layers and stacks: whole vectors, and whole words of bit-packed
// spikes (a word of 64 neurons is shared by several lanes).  The few that are left go to one
// workgroup of one neuron per lane, the first in the grid so that its long walk starts with
// the others; no lane is guarded.
template <int SPK, int V>
constexpr int64_t whole_vectors(int64_t N) {
    constexpr int64_t unit = SPK == SNN_SPK_BITS && V > 1 ? kWave : V;
    return N / unit * unit;
}

// Whether a gain-fed layer or a stack, whose N is a multiple of V, can have such a rest.
template <int SPK, int V>
constexpr bool has_rest() { return SPK == SNN_SPK_BITS && V > 1; }

// Kernel-side hyper-parameters.
struct LifK {
    float k;      // decay k_tau
    float th;     // V_th
    float rest;   // V_rest
    float alpha;  // surrogate sharpness
    float c_exp;  // -alpha * log2(e): e^{-alpha |u|} = 2^{c_exp |u|}
    float kth;    // k * V_th (soft-reset backward)
};

}  // namespace snnlif
