// stab_device.h -- structures shared by the kernels and the host side of libstab.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace stabdev {

// Most 64-bit column words a lane of the deterministic-measurement wave keeps in registers.
constexpr int kMaxWordsPerLane = 4;
// Most 64-row bands of a half: up to it a half-band fits in LDS, and the block's form of k_plan's
// elimination holds a chunk's words in registers (16 waves of 10).
constexpr int kMaxBands = 160;

struct Geom {
    int n;    // qubits
    int Wc;   // column words per row and component: ceil(n / 64)
    int Wr;   // 64-row bands per half: ceil(n / 64)
    int NR;   // rows per half, padded: 64 * Wr
    int RS;   // row stride in words: 2 * Wc (x words, then z words)
    int NB;   // bands (and sign words) per tableau: 2 * Wr
    int S;    // tableau copies
    int B;    // shots
    int bpc;  // shots per copy (B / S)
    int rev;  // 1: kernels take their blocks in reverse order (a determinism check)
};

// Block index along x (y) in the order the kernels take blocks: reversed when g.rev is set, so a
// run with the flag changes which work each dispatched workgroup does and the order in which the
// work reaches the device; the results must not change.
__device__ __forceinline__ int blk_x(const Geom& g) { return g.rev ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x; }
__device__ __forceinline__ int blk_y(const Geom& g) { return g.rev ? (int)gridDim.y - 1 - (int)blockIdx.y : (int)blockIdx.y; }

// One noise instruction of a segment.
struct NoiseDesc {
    uint64_t instr;        // instruction index (Philox counter word 0)
    uint64_t t0, t1, t2;   // thresholds
    int kind;              // DEP1, DEP2 or PAULI1
    int toff;              // first target in the segment's noise target array
    int units;             // targets (DEP1, PAULI1) or pairs (DEP2)
    int bucket;            // event bucket (= item.w of the noise item; consecutive noise layers share one)
};

// Work counters are striped over this many addresses (by block) to keep atomics uncontended.
constexpr int kCounterStripes = 32;
constexpr int kNumCounters = 12;

__device__ __forceinline__ void count_add(unsigned long long* counters, int idx, unsigned long long v)
{
    if (counters) atomicAdd(&counters[idx * kCounterStripes + (blockIdx.x & (kCounterStripes - 1))], v);
}

// Gates of a layer: at most a qubit each.
constexpr int kGateBits = 14, kGateMask = (1 << kGateBits) - 1;
static_assert(64 * kMaxBands <= kGateMask, "gate counts of an item");

struct SegArgs {
    // {0 | Xs << 1 | Ys << 15, first gate, gate count | Ss << 14, CXs | Hs << 14} or {1, first event slot,
    // event capacity, bucket}
    const int4* items;
    int nitems;
    int nlds;              // items whose descriptors the kernel keeps in LDS (past the sign accumulators)
    const uint32_t* gates; // i0 | i1 << 16, i = the qubit's pair in the staged tile (i1 = i0 for one qubit);
                           // an item's gates 0, h, 1, h + 1, ... with h = half of them, rounded up
    const uint2* events;   // noise events {tile pair of the qubit | pauli << 28, shot}
    const int* ev_count;   // per bucket
    const int* ev_base;    // per bucket: first slot in events
    int write_back;        // 1 if some gate changes x|z (H, S, CX)
    const int* ext_q;      // qubits whose columns the next measurement layer needs
    int K;
    uint64_t* Xcol;        // [S][NB][K]
    uint64_t* Zcol;
    const int* gate;       // if set and *gate == 0 the launch does nothing
};

}  // namespace stabdev
