// stab_kernels.hip -- device code of the MI355X tableau simulator (gfx950, wave64).
//
// Storage (per tableau copy s):
//   tab  [2*NR][RS] uint64, row-major.  Row i < NR is destabilizer i, row NR+i stabilizer i
//        (NR = 64*ceil(n/64); rows >= n of each half are zero padding).  A row holds Wc x-words
//        (bit j%64 of word j/64 = x at qubit j) then Wc z-words; RS = 2*Wc.
//   rs   [NB] uint64 sign words of the copy (NB = 2*NR/64; word w holds rows 64w..64w+63).
//   rd   [B][NB] per-shot sign words.  The sign of row i in shot b is rs ^ rd[b].  In the
//        shared mode one x|z tableau serves every shot: gates only ever XOR shot-independent
//        masks into signs, so those go to rs, while noise, random outcomes and resets (the
//        only shot-dependent parts) go to rd.
//
// A "band" is 64 consecutive rows.  The segment kernel stages half a band (32 rows) in LDS,
// turns its 32x32 bit tiles into qubit-major 32-bit words (one bit per row of one qubit
// column), applies a whole run of gate and noise layers there, extracts the columns the next
// measurement layer needs and writes the rows back.  Measurements then work on rows (rowsum,
// Appendix A.2).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "stab_device.h"

#define STAB_KIND_H 1
#define STAB_KIND_S 2
#define STAB_KIND_X 3
#define STAB_KIND_Y 4
#define STAB_KIND_Z 5
#define STAB_KIND_CX 6
#define STAB_KIND_DEP1 10
#define STAB_KIND_DEP2 11
#define STAB_KIND_PAULI1 12

namespace stabdev {

// ------------------------------------------------------------------------------------------
// Philox4x64-10, from Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy as
// 1, 2, 3" (SC'11): ten rounds, each multiplying words 0 and 2 by the two published
// multipliers (full 128-bit products) and mixing the halves with the other words and the
// key; the key advances by the two published Weyl constants between rounds.
// Counter = (c0, c1, 0, 0), key = (k0, k1).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void philox(uint64_t c0, uint64_t c1, uint64_t k0, uint64_t k1,
                                       uint64_t& u0, uint64_t& u1)
{
    uint64_t a = c0, b = c1, c = 0, d = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t pa_lo = 0xD2E7470EE14C6C93ull * a;
        const uint64_t pa_hi = __umul64hi(0xD2E7470EE14C6C93ull, a);
        const uint64_t pc_lo = 0xCA5A826395121157ull * c;
        const uint64_t pc_hi = __umul64hi(0xCA5A826395121157ull, c);
        a = pc_hi ^ b ^ k0;
        b = pc_lo;
        c = pa_hi ^ d ^ k1;
        d = pa_lo;
        k0 += 0x9E3779B97F4A7C15ull;
        k1 += 0xBB67AE8584CAA73Bull;
    }
    u0 = a;
    u1 = b;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m)
{
    const int lo = __shfl_xor((int)(uint32_t)v, m, 64);
    const int hi = __shfl_xor((int)(uint32_t)(v >> 32), m, 64);
    return ((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo;
}

__device__ __forceinline__ int wave_sum(int v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

__device__ __forceinline__ uint64_t wave_xor(uint64_t v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v ^= shfl_xor_u64(v, m);
    return v;
}

__device__ __forceinline__ uint64_t wave_or(uint64_t v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v |= shfl_xor_u64(v, m);
    return v;
}

// Sum over the 64 bit positions of g(x1,z1,x2,z2) from the rowsum algorithm (Appendix A.2):
// the power of i from multiplying the Pauli (x1,z1) into (x2,z2), per bit in {-1, 0, +1}.
__device__ __forceinline__ int gsum(uint64_t x1, uint64_t z1, uint64_t x2, uint64_t z2)
{
    const uint64_t y1 = x1 & z1, xo = x1 & ~z1, zo = ~x1 & z1;
    const uint64_t plus = (y1 & ~x2 & z2) | (xo & x2 & z2) | (zo & x2 & ~z2);
    const uint64_t minus = (y1 & x2 & ~z2) | (xo & ~x2 & z2) | (zo & x2 & z2);
    return __popcll(plus) - __popcll(minus);
}

__device__ __forceinline__ int ctz64(uint64_t v) { return __builtin_ctzll(v); }

// Lane l's 64-bit value, l uniform (scalar result).
__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// v from lane (lane ^ j), j in {1, 2, 4, 8, 16}, without the LDS crossbar: DPP quad permutes
// and row mirrors for j <= 8 (xor 4 = half-mirror then quad xor 3; xor 8 = mirror then
// half-mirror) and the gfx950 permlane16 swap for j = 16.  Every lane must be active.
__device__ __forceinline__ uint32_t lane_xor32(uint32_t v, int j, int lane)
{
    switch (j) {
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
    case 4: {
        const int t = __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_update_dpp(0, t, 0x1B, 0xF, 0xF, true);
    }
    case 8: {
        const int t = __builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_update_dpp(0, t, 0x141, 0xF, 0xF, true);
    }
    default: {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane & 16) ? r[0] : r[1];
    }
    }
}

// Sum over the wave, every lane active: DPP and permlane steps within each 32-lane half, then the
// two halves' totals read out, so the result is uniform.
__device__ __forceinline__ int wave_sum_uniform(int v, int lane)
{
#pragma unroll
    for (int j = 1; j <= 16; j <<= 1) v += (int)lane_xor32((uint32_t)v, j, lane);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 32);
}

__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = min(v, __shfl_xor(v, m, 64));
    return v;
}

__device__ __forceinline__ int wave_excl_scan(int v, int lane)
{
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    return incl - v;
}

// Block barrier that orders LDS accesses only: global loads and stores may stay in flight across it
// (__syncthreads waits for them all, which undoes a prefetch issued before it).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// v is the same in every lane (the compiler cannot see that for values read from LDS): keeping
// it in a scalar register makes loops over it scalar loops.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// ------------------------------------------------------------------------------------------
// init: |0...0> -- destabilizer i = +X_i, stabilizer i = +Z_i, all signs 0.
// ------------------------------------------------------------------------------------------
__global__ void k_init(Geom g, uint64_t* __restrict__ tab, uint64_t* __restrict__ rs,
                       uint64_t* __restrict__ rd)
{
    const size_t rows = (size_t)g.S * 2 * g.NR;
    const size_t total = rows * g.RS;
    for (size_t idx = blk_x(g) * (size_t)blockDim.x + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * blockDim.x) {
        const size_t row = idx / g.RS;
        const int c = (int)(idx - row * g.RS);
        const int rr = (int)(row % (2 * (size_t)g.NR));
        uint64_t v = 0;
        if (rr < g.NR) {
            if (rr < g.n && c == (rr >> 6)) v = 1ull << (rr & 63);
        } else {
            const int i = rr - g.NR;
            if (i < g.n && c == g.Wc + (i >> 6)) v = 1ull << (i & 63);
        }
        tab[idx] = v;
    }
    const size_t nrs = (size_t)g.S * g.NB, nrd = (size_t)g.B * g.NB;
    for (size_t idx = blk_x(g) * (size_t)blockDim.x + threadIdx.x; idx < nrs + nrd;
         idx += (size_t)gridDim.x * blockDim.x) {
        if (idx < nrs) rs[idx] = 0;
        else rd[idx - nrs] = 0;
    }
}

// ------------------------------------------------------------------------------------------
// Noise draws: block (x, y) handles kNoiseUnitsPerBlock consecutive (shot, unit) pairs of noise
// instruction y.  Draws never depend on the tableau, so they are made up front (the whole
// program's in one launch when its event slots fit, else a segment's before it) and the
// segment kernel applies them at their layer.  Event = (tile word index of the qubit
// | pauli << 28, shot).  A block gathers its events in LDS and reserves space with one atomic.
// ------------------------------------------------------------------------------------------
constexpr int kNoiseThreads = 1024;
constexpr int kNoiseUnitsPerBlock = 4 * kNoiseThreads;
constexpr int kNoiseLdsEvents = 2048;
// event slots (8 bytes each) up to which a program's noise is drawn in one launch
constexpr long long kDrawAllEvents = 1ll << 28;

// Instruction y of nd[] (y = blockIdx.y, or reversed with rev).  seg_base (may be NULL): per
// instruction, the first event slot of its segment, when every segment's events are drawn by
// one launch.  The order of a bucket's events depends on block timing; applying them commutes.
__global__ void __launch_bounds__(1024)
k_noise_draw(const NoiseDesc* __restrict__ nd, const int* __restrict__ ntg, int B, uint64_t seed,
             uint64_t first_shot, uint64_t instr_base, uint2* __restrict__ events,
             const long long* __restrict__ seg_base, const int* __restrict__ ev_base, int* __restrict__ ev_count,
             unsigned long long* __restrict__ counters, int rev)
{
    __shared__ uint2 sev[kNoiseLdsEvents];
    __shared__ int s_n, s_base;
    const int bx = rev ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x;
    const int by = rev ? (int)gridDim.y - 1 - (int)blockIdx.y : (int)blockIdx.y;
    const NoiseDesc d = nd[by];
    const long long total = (long long)d.units * B;
    const long long start = (long long)bx * kNoiseUnitsPerBlock;
    if (start >= total) return;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    uint2* gdst = events + (seg_base ? seg_base[by] : 0ll) + ev_base[d.bucket];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const long long idx = start + threadIdx.x + (long long)j * kNoiseThreads;
        if (idx >= total) break;
        const int b = (int)(idx / d.units);
        const int pos = (int)(idx - (long long)b * d.units);
        uint64_t u0, u1;
        philox(instr_base + d.instr, (uint64_t)pos, seed, first_shot + (uint64_t)b, u0, u1);
        uint32_t e[2];
        int ne = 0;
        if (d.kind == STAB_KIND_DEP1) {
            if (u0 < d.t0) e[ne++] = (uint32_t)ntg[d.toff + pos] | ((uint32_t)(1 + (int)__umul64hi(u1, 3ull)) << 28);
        } else if (d.kind == STAB_KIND_DEP2) {
            if (u0 < d.t0) {
                const int k = 1 + (int)__umul64hi(u1, 15ull);
                if (k >> 2) e[ne++] = (uint32_t)ntg[d.toff + 2 * pos] | ((uint32_t)(k >> 2) << 28);
                if (k & 3) e[ne++] = (uint32_t)ntg[d.toff + 2 * pos + 1] | ((uint32_t)(k & 3) << 28);
            }
        } else {  // PAULI1 with cumulative thresholds
            const int P = (u0 < d.t0) ? 1 : (u0 < d.t1) ? 2 : (u0 < d.t2) ? 3 : 0;
            if (P) e[ne++] = (uint32_t)ntg[d.toff + pos] | ((uint32_t)P << 28);
        }
        for (int i = 0; i < ne; ++i) {
            const int slot = atomicAdd(&s_n, 1);
            const uint2 ev = make_uint2(e[i], (uint32_t)b);
            if (slot < kNoiseLdsEvents) sev[slot] = ev;
            else gdst[atomicAdd(&ev_count[d.bucket], 1)] = ev;   // LDS full: direct
        }
    }
    __syncthreads();
    const int n = min(s_n, kNoiseLdsEvents);
    if (threadIdx.x == 0 && s_n) count_add(counters, 7, (unsigned long long)s_n);
    if (n == 0) return;
    if (threadIdx.x == 0) s_base = atomicAdd(&ev_count[d.bucket], n);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) gdst[s_base + i] = sev[i];
}

// ------------------------------------------------------------------------------------------
// Segment kernel helpers.
// ------------------------------------------------------------------------------------------
// The staged tile: the x and z words of qubit q's 32 rows are the pair at (q & 63) * seg_pairs(Wc) +
// (q >> 6) (an odd stride, so consecutive qubits fall on different banks).
__host__ __device__ constexpr int seg_pairs(int Wc) { return Wc | 1; }

// Descriptor of an item of a segment, a gate layer (its gates sorted by kind: CX, H, S, X, Y, Z) or a
// noise layer, as in SegArgs::items with a noise item's count resolved.
__device__ __forceinline__ int4 seg_item(const SegArgs& a, const int4* items, int it)
{
    typedef int v4i __attribute__((ext_vector_type(4)));
    typedef const v4i __attribute__((address_space(4)))* Int4s;
    typedef const int __attribute__((address_space(4)))* Ints;
    if (it >= a.nitems) return make_int4(0, 0, 0, 0);
    if (it < a.nlds) return items[it];
    const v4i v = *((Int4s)a.items + it);
    return make_int4(v.x, v.y, (v.x & 1) ? *((Ints)a.ev_count + v.w) : v.z, v.w);
}

// Registers holding the first PF * blockDim.x entries of an item's list: noise events, or two gates
// each (entry k has gates k and k + half), so that both take the same loads.
template <int PF>
struct ItemBuf {
    uint2 v[PF];
    int x, y, z, w;   // the item
    __device__ bool noise() const { return x & 1; }
    __device__ int gates() const { return z & kGateMask; }
    __device__ int entries() const { return (x & 1) ? z : (gates() + 1) >> 1; }
};

// Wait for a load here, so that no path leaves the loop with it pending (the next items' lists would
// then be waited for with it).
__device__ __forceinline__ void landed(uint2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

constexpr int kSegThreads = 1024;   // of a block of k_segment

// Bytes of a list of `entries` that the descriptor of its first `ahead` covers (the whole list's would
// not fit 32 bits from 2^29 entries on).
__host__ __device__ constexpr int ahead_bytes(int entries, int ahead) { return (entries < ahead ? entries : ahead) * 8; }

// Loads past the list's end are bounded by the buffer descriptor (they return 0): every thread issues
// the same loads whatever the item, so the wait for one item's leaves a later one's in flight.
template <int PF>
__device__ __forceinline__ void fetch_item(const SegArgs& a, int4 d, int tid, int nt, ItemBuf<PF>& b)
{
    b.x = uni(d.x);
    b.y = uni(d.y);
    b.z = uni(d.z);
    b.w = uni(d.w);
    const void* list = b.noise() ? (const void*)(a.events + b.y) : (const void*)(a.gates + b.y);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)list, (short)0, ahead_bytes(b.entries(), PF * kSegThreads), 0x00027000);
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        const auto t = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (tid + u * nt) * 8, 0, 0);
        b.v[u] = make_uint2(t[0], t[1]);
    }
}

// Gates i and i + n of a layer of count gates (x, z, w as in SegArgs::items) on the 32 staged rows; gt:
// the tile pairs of their qubits (0 past the end), w0: i of the wave's first thread.  All four pairs
// are read before any is written (a layer's qubits are distinct).  A wave of CX gates only runs
// those; else every kind runs the same instructions, by masks: with the second qubit equal to the
// first, H and S are a CX's sign rule x0 z1 (x1 ^ z0 ^ 1) = x0 z0 with another update.
__device__ __forceinline__ void apply_gates(uint2* T, uint2 gt, int i, int w0, int n, int count, int x, int z, int w,
                                            uint32_t& racc)
{
    const int c0 = w & kGateMask;
    uint2* t[2][2] = {{T + (gt.x & 0xFFFFu), T + (gt.x >> 16)}, {T + (gt.y & 0xFFFFu), T + (gt.y >> 16)}};
    uint2 q[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        q[e][0] = *t[e][0];
        q[e][1] = *t[e][1];
    }
    const bool on[2] = {i < n, i + n < count};
    if (min(w0 + n + 64, count) <= c0) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint2 a = q[e][0], b = q[e][1];
            if (on[e]) {
                racc ^= a.x & b.y & ~(b.x ^ a.y);
                t[e][1]->x = b.x ^ a.x;
                t[e][0]->y = a.y ^ b.y;
            }
        }
    } else {
        const int c1 = c0 + (w >> kGateBits), c2 = c1 + (z >> kGateBits), c3 = c2 + (x >> 1 & kGateMask),
                  c4 = c3 + (x >> (1 + kGateBits));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            auto below = [&](int c) { return (uint32_t)((i + e * n - c) >> 31); };
            const uint2 a = q[e][0], b = q[e][1];
            const uint32_t u = below(c2), cx = below(c0), hs = u & ~cx, h = below(c1) & hs;
            const uint32_t r = (a.x & b.y & ~(b.x ^ a.y) & u) ^ (a.x & ~below(c3)) ^ (a.y & below(c4) & ~u);
            if (on[e]) {
                racc ^= r;
                t[e][1]->x = b.x ^ (a.x & cx) ^ ((a.x ^ a.y) & h);
                t[e][0]->y = a.y ^ (b.y & cx) ^ (a.x & hs) ^ (a.y & h);
            }
        }
    }
}

// Noise event {tile pair of the qubit | pauli << 28, shot}: flip the signs of the rows the Pauli
// anticommutes with.  LRD: per-shot signs in LDS (a choice at run time would make the atomic a flat
// one, which waits for every load in flight).
template <bool LRD>
__device__ __forceinline__ void apply_event(const uint2* T, uint2 v, int s, int hb, const Geom& g, uint32_t* rdacc,
                                            uint32_t* rd32)
{
    const int sb = (int)v.y - s * g.bpc;
    if (sb < 0 || sb >= g.bpc) return;
    const uint2 q = T[v.x & 0x0FFFFFFFu];
    const int P = (int)(v.x >> 28);
    const uint32_t m = (P == 1) ? q.y : (P == 3) ? q.x : (q.x ^ q.y);
    if (m) {
        if (LRD) atomicXor(&rdacc[sb], m);
        else atomicXor(&rd32[(size_t)(s * g.bpc + sb) * 2 * g.NB + hb], m);
    }
}

// In-register transpose of the 32x32 bit matrix held by each half-wave, one row per lane
// (bit c of lane r's word = element (r, c)); lanes 32..63 transpose their own matrix.
__device__ __forceinline__ uint32_t transpose32(uint32_t v, int lane)
{
    const uint32_t masks[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int st = 0; st < 5; ++st) {
        const int j = 16 >> st;
        const uint32_t m = masks[st];
        const uint32_t o = lane_xor32(v, j, lane);
        if (lane & j) {
            v ^= ((o >> j) ^ v) & m;
        } else {
            v ^= (((v >> j) ^ o) & m) << j;
        }
    }
    return v;
}

// Transpose of 32x32 bit matrices held by lane pairs (lane, lane + 32): lane q * 32 + j has rows
// 16q .. 16q + 15 of pair j's matrix in w, and gets the same rows of its transpose.  One exchange
// between the two lanes, then four stages among a lane's own words: 160 instructions for 32
// matrices, where a row per lane takes 25 for two (transpose32).  Every lane must be active.
__device__ __forceinline__ void transpose32_pairs(uint32_t (&w)[16], int lane)
{
    const uint32_t sel = lane < 32 ? 0x05040100u : 0x07060302u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(w[i], w[i], false, false);
        w[i] = __builtin_amdgcn_perm(r[1], r[0], sel);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t a = w[i], b = w[i + 8];
        w[i] = __builtin_amdgcn_perm(b, a, 0x06020400u);
        w[i + 8] = __builtin_amdgcn_perm(b, a, 0x07030501u);
    }
    const uint32_t masks[3] = {0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int st = 0; st < 3; ++st) {
        const int j = 4 >> st;
        const uint32_t m = masks[st];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i & j) continue;
            const uint32_t a = w[i], b = w[i + j];
            w[i] = (a & m) | ((b << j) & ~m);
            w[i + j] = ((a >> j) & m) | (b & ~m);
        }
    }
}

// Whether any lane has a bit set; an all-zero set of matrices (most of a sparse tableau, such as a
// surface code's) is its own transpose.
__device__ __forceinline__ bool any_bit(const uint32_t (&w)[16])
{
    uint32_t o = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) o |= w[i];
    return __ballot(o != 0u) != 0ull;
}

// ------------------------------------------------------------------------------------------
// Segment kernel: grid (2 * NB half-bands, S copies), 1024 threads.  A block holds 32 rows (half of
// a 64-row band) in LDS as 32-bit qubit-major words, a qubit's x and z bits of the rows side by side
// (seg_pairs).  Two such blocks fit the LDS of one compute unit up to 10176 qubits.  The
// rows are transposed on the way, in registers: a wave's lane pairs load the 32 words of 32
// columns (32 rows of 32 bits each), and write the transposed words; the way back is the same.
// The block owns the 32-bit half of every sign word and column-extract word of its band.
//
// It is bound by the chain from layer to layer, not by bytes (632 blocks of a 10081-qubit tableau
// move 102 MB in 50 us): per layer the list's load, four LDS reads and two writes a gate, and a
// barrier.  So lists are loaded two layers ahead across barriers that order LDS only, gates take 4
// bytes and two of a thread run together, and the descriptors lie in LDS.  Launches of a memory
// round at d = 25 (1249 qubits, 100 shots) 13.5 -> 12.0 us, at d = 71 57 -> 50 us, 40 copies of
// d = 25 95 -> 86 us.
// ------------------------------------------------------------------------------------------
template <bool LRD, int PF>
__global__ void __launch_bounds__(kSegThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_segment(Geom g, uint64_t* __restrict__ tab, uint64_t* __restrict__ rs,
          uint64_t* __restrict__ rd, SegArgs a)
{
    if (a.gate && *a.gate == 0) return;   // an extraction pass with nothing to refresh
    extern __shared__ uint32_t lds32[];
    const int hb = blk_x(g);                     // half-band: band = hb >> 1, half = hb & 1
    const int band = hb >> 1, half = hb & 1;
    const int s = blk_y(g);
    constexpr int nt = kSegThreads;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = uni(tid >> 6), nwaves = nt >> 6;
    const int RS = g.RS, Wc = g.Wc, RP = seg_pairs(Wc);
    uint2* T = (uint2*)lds32;                    // 64 x RP pairs
    uint32_t* red = lds32 + 128 * RP;            // nwaves words
    uint32_t* rdacc = red + 16;                  // bpc words when LRD
    int4* items = (int4*)(lds32 + ((128 * RP + 16 + (LRD ? g.bpc : 0) + 3) & ~3));   // nlds descriptors
    uint64_t* gb = tab + ((size_t)s * 2 * g.NR + (size_t)band * 64 + (size_t)half * 32) * RS;
    uint32_t* rs32 = (uint32_t*)rs;
    uint32_t* rd32 = (uint32_t*)rd;

    for (int it = tid; it < a.nlds; it += nt) {
        int4 v = a.items[it];
        if (v.x & 1) v.z = a.ev_count[v.w];
        items[it] = v;
    }
    // columns j of 32 bits, two lanes each; rows 16 (lane >> 5) .. + 15 and, transposed, the
    // column's bits of the same numbers
    const int ncol = 2 * RS, q16 = (lane >> 5) * 16;
    uint32_t* gr = (uint32_t*)gb + (size_t)q16 * ncol;
    for (int j0 = wave * 32; j0 < ncol; j0 += nwaves * 32) {
        const int j = j0 + (lane & 31);
        uint32_t w[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) w[r] = j < ncol ? gr[r * ncol + j] : 0u;
        if (any_bit(w)) transpose32_pairs(w, lane);
        const int c = j >> 1, comp = c >= Wc;
        uint32_t* t = lds32 + ((32 * (j & 1) + q16) * RP + c - comp * Wc) * 2 + comp;
        if (j < ncol) {
#pragma unroll
            for (int b = 0; b < 16; ++b) t[2 * b * RP] = w[b];
        }
    }
    if (LRD)
        for (int b = tid; b < g.bpc; b += nt) rdacc[b] = 0;
    __syncthreads();

    uint32_t racc = 0;
    // item it's list is loaded two items ahead, into one of three buffers (no register moves: a move
    // would wait for the load), and its descriptor three
    ItemBuf<PF> b0, b1, b2;
    int4 desc = make_int4(0, 0, 0, 0);
    if (a.nitems > 0) {
        fetch_item(a, seg_item(a, items, 0), tid, nt, b0);
        fetch_item(a, seg_item(a, items, 1), tid, nt, b1);
        desc = seg_item(a, items, 2);
    }
    auto step = [&](const ItemBuf<PF>& cur, ItemBuf<PF>& next, int it) {
        fetch_item(a, desc, tid, nt, next);
        desc = seg_item(a, items, it + 3);
        const int w0 = wave * 64, n = cur.entries();
        if (!cur.noise()) {
            const uint2* list = (const uint2*)(a.gates + cur.y);
            const int count = cur.gates();
            auto gates = [&](uint2 gt, int k) {
                apply_gates(T, gt, tid + k, w0 + k, n, count, cur.x, cur.z, cur.w, racc);
            };
#pragma unroll
            for (int u = 0; u < PF; ++u)
                if (w0 + u * nt < n) gates(cur.v[u], u * nt);
            for (int k = PF * nt; w0 + k < n; k += nt) {
                uint2 gt = list[min(tid + k, n - 1)];
                landed(gt);
                gates(gt, k);
            }
        } else {
            const uint2* list = a.events + cur.y;
#pragma unroll
            for (int u = 0; u < PF; ++u)
                if (tid + u * nt < n) apply_event<LRD>(T, cur.v[u], s, 2 * band + half, g, rdacc, rd32);
            // (unsigned: up to 2^31 - 1 events)
            for (uint32_t e0 = tid + PF * nt; e0 < (uint32_t)n; e0 += 4 * nt) {
                uint2 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = list[min(e0 + u * nt, (uint32_t)n - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) landed(v[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (e0 + u * nt < (uint32_t)n) apply_event<LRD>(T, v[u], s, 2 * band + half, g, rdacc, rd32);
            }
        }
        lds_barrier();
    };
    for (int it = 0; it < a.nitems; it += 3) {
        step(b0, b2, it);
        if (it + 1 < a.nitems) step(b1, b0, it + 1);
        if (it + 2 < a.nitems) step(b2, b1, it + 2);
    }

    if (a.K > 0) {
        uint32_t* Xc = (uint32_t*)(a.Xcol + ((size_t)s * g.NB + band) * a.K);
        uint32_t* Zc = (uint32_t*)(a.Zcol + ((size_t)s * g.NB + band) * a.K);
        for (int k = tid; k < a.K; k += nt) {
            const int q = a.ext_q[k];
            const uint2 t = T[(q & 63) * RP + (q >> 6)];
            Xc[2 * k + half] = t.x;
            Zc[2 * k + half] = t.y;
        }
    }
    if (a.write_back) {
        for (int j0 = wave * 32; j0 < ncol; j0 += nwaves * 32) {
            const int j = j0 + (lane & 31);
            const int c = j >> 1, comp = c >= Wc;
            const uint32_t* t = lds32 + ((32 * (j & 1) + q16) * RP + c - comp * Wc) * 2 + comp;
            uint32_t w[16];
#pragma unroll
            for (int b = 0; b < 16; ++b) w[b] = j < ncol ? t[2 * b * RP] : 0u;
            if (any_bit(w)) transpose32_pairs(w, lane);
            if (j < ncol) {
#pragma unroll
                for (int r = 0; r < 16; ++r) gr[r * ncol + j] = w[r];
            }
        }
    }
    // sign contributions: XOR-reduce 32-bit masks
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) racc ^= (uint32_t)__shfl_xor((int)racc, m, 64);
    if (lane == 0) red[wave] = racc;
    __syncthreads();
    if (tid == 0) {
        uint32_t t = 0;
        for (int w = 0; w < nwaves; ++w) t ^= red[w];
        if (t) rs32[((size_t)s * g.NB + band) * 2 + half] ^= t;
    }
    if (LRD) {
        for (int b = tid; b < g.bpc; b += nt) {
            const uint32_t v = rdacc[b];
            if (v) rd32[((size_t)(s * g.bpc + b) * g.NB + band) * 2 + half] ^= v;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Classification and deterministic outcomes of a measurement layer (Sec. 2.4), one wave per
// (copy, target).
//
// pass 0, at layer start: the block's eight consecutive targets have their x columns staged in
// LDS first (a band's eight words are contiguous in Xcol, so the loads are coalesced), then a
// wave takes each target's column one word per 64-row band and lane.  The first stabilizer with x at the qubit is the pivot: the target is
// random, its class is that stabilizer index (k_plan takes it for any that is not negative).  Without one the
// outcome is deterministic: +-Z_a is the product of the stabilizers NR + i over the
// destabilizers i with x at the qubit (class -1).  pass 1, after the random targets on the final
// tableau (only when one ran): the targets k_plan marked deterministic (-2)
// are reduced and marked -3.  A deterministic outcome is unchanged by Z measurements and
// resets on other qubits, so every one of a layer is reduced in parallel (the paper
// serialises every row behind two grid barriers, Alg. 2).
//
// The product.  The destabilizer bits are enumerated in row order (ballot, then scalar loops
// over the few nonzero words), 64 rows at a time with lane c holding the c-th; rows are loaded
// kDetRowBatch at a time (no load conditional, so a batch is in flight at once).  Its phase is
// telescoped: with |u| the number of qubits where u has both x and z, multiplying rows into
// the scratch row S raises i to sum|row| - |S| + 2 sum z_row.x_S (mod 4), and only the parity
// of the last sum matters, so it is XOR-accumulated and popcounted once.  The per-shot part of
// the sign is the parity of each shot's sign bits over the same rows; the bits of a shot group
// of 64 gather in LDS (nrdw words per wave).
// ------------------------------------------------------------------------------------------
// targets (waves) per block: four with one-word rows (small tableaux: more blocks in flight),
// eight otherwise (a band's eight column words are one coalesced 64-byte read)
constexpr int det_targets(int wpl) { return wpl == 1 ? 4 : 8; }
constexpr int kDetRowBatch = 3;                // rows a wave loads at once

// WPL = ceil(Wc / 64): column words (and stabilizer bands) a lane holds of a row.
template <int WPL>
__global__ void __launch_bounds__(64 * det_targets(WPL)) __attribute__((amdgpu_waves_per_eu(4)))
k_det(Geom g, const uint64_t* __restrict__ tab, const uint64_t* __restrict__ rs,
      const uint64_t* __restrict__ rd, const uint64_t* __restrict__ Xcol, int K, int* __restrict__ cls,
      uint8_t* __restrict__ obuf, int* __restrict__ ran, int* __restrict__ err,
      unsigned long long* __restrict__ counters, int pass, int* __restrict__ ran_log)
{
    extern __shared__ uint64_t dsm[];
    constexpr int kDetTargets = det_targets(WPL);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k0 = blk_x(g) * kDetTargets, k = k0 + wave;
    const int s = blk_y(g);
    const int NB = g.NB, nrdw = (g.bpc + 63) >> 6;
    uint64_t* colw = dsm;                                          // [kDetTargets][NB] columns
    uint64_t* parw = dsm + (size_t)kDetTargets * NB + (size_t)wave * nrdw;   // shot parity bits
    // the block's work counters, flushed with one atomic each at the end
    __shared__ unsigned int s_det, s_rows;
    if (threadIdx.x == 0) {
        s_det = 0;
        s_rows = 0;
    }
    if (pass == 0) {
        // k_plan counts its windows here
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *ran = 0;
    } else {
        // (ran_log, when given: how many windows of random targets this layer took, for the host)
        const int r = *ran;
        if (ran_log && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *ran_log = r;
        if (r == 0) return;
    }
    const uint64_t* X = Xcol + (size_t)s * NB * K;
    // eight words per thread at a time: all loads in flight before the LDS stores
    const int tot = NB * kDetTargets;
    for (int i0 = threadIdx.x; i0 < tot; i0 += 8 * (int)blockDim.x) {
        uint64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * (int)blockDim.x;
            const int w = i / kDetTargets, j = i - w * kDetTargets;
            v[u] = (i < tot && k0 + j < K) ? X[(size_t)w * K + k0 + j] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * (int)blockDim.x;
            const int w = i / kDetTargets, j = i - w * kDetTargets;
            if (i < tot) colw[j * NB + w] = v[u];
        }
    }
    __syncthreads();
    // one wave per target; a wave that is done returns from here
    [&]() {
        if (k >= K) return;
        if (pass == 1 && cls[s * K + k] != -2) return;
        const uint64_t* tb = tab + (size_t)s * 2 * g.NR * g.RS;
        const uint64_t* rsc = rs + (size_t)s * NB;
        // the column: destabilizer words cd, stabilizer words cs (band lane + 64 u of each half)
        uint64_t cd[WPL], cs[WPL];
#pragma unroll
        for (int u = 0; u < WPL; ++u) {
            const int w = lane + 64 * u;
            cd[u] = w < g.Wr ? colw[wave * NB + w] : 0ull;
            cs[u] = w < g.Wr && pass == 0 ? colw[wave * NB + g.Wr + w] : 0ull;
        }
        if (pass == 0) {
#pragma unroll
            for (int u = 0; u < WPL; ++u) {
                const uint64_t m = __ballot(cs[u] != 0ull);
                if (m) {
                    const int l = ctz64(m);
                    if (lane == 0) cls[s * K + k] = (l + 64 * u) * 64 + ctz64(readlane_u64(cs[u], l));
                    return;                              // random at layer start
                }
            }
        }
        if (lane == 0) cls[s * K + k] = pass == 0 ? -1 : -3;
        for (int u = lane; u < nrdw; u += 64) parw[u] = 0;
        const uint64_t* base = tb + (size_t)g.NR * g.RS;
        int jc[WPL];
        uint64_t msk[WPL], sx[WPL], sz[WPL], cr[WPL];
#pragma unroll
        for (int t = 0; t < WPL; ++t) {
            const int j = lane + 64 * t;
            jc[t] = j < g.Wc ? j : 0;
            msk[t] = j < g.Wc ? ~0ull : 0ull;
            sx[t] = sz[t] = cr[t] = 0;
        }
        int G = 0, rsum = 0, cnt = 0, nc = 0, myrow = 0;
        // multiply the nc listed rows (lane c holds the c-th) into S, and their shot sign bits
        auto flush = [&]() {
            // nothing below depends on a row's contents except the product itself, so with
            // one-word rows the first batch of rows, the listed rows' shared sign words and the
            // shots' sign words are requested together: one round trip instead of three.  With
            // wider rows the registers that holds cost more occupancy than the round trips save
            // (d=71: 71 -> 90 VGPRs and the pass 18 % slower), so they go one after another.
            uint64_t rx[kDetRowBatch][WPL], rz[kDetRowBatch][WPL];
            auto load = [&](int u0) {
#pragma unroll
                for (int u = 0; u < kDetRowBatch; ++u) {
                    const int i = __shfl(myrow, min(u0 + u, nc - 1), 64);
                    const uint64_t* row = base + (size_t)i * g.RS;
#pragma unroll
                    for (int t = 0; t < WPL; ++t) {
                        rx[u][t] = row[jc[t]];
                        rz[u][t] = row[g.Wc + jc[t]];
                    }
                }
            };
            auto parity = [&]() {
                for (int b0 = 0; b0 < g.bpc; b0 += 64) {
                    const uint64_t* rdb = rd + (size_t)(s * g.bpc + min(b0 + lane, g.bpc - 1)) * g.NB + g.Wr;
                    int par = 0;
                    for (int c = 0; c < nc; c += 8) {
                        int iu[8];
                        uint64_t wv[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) iu[u] = __shfl(myrow, min(c + u, nc - 1), 64);
#pragma unroll
                        for (int u = 0; u < 8; ++u) wv[u] = rdb[iu[u] >> 6];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (c + u < nc) par ^= (int)((wv[u] >> (iu[u] & 63)) & 1ull);
                    }
                    const uint64_t pb = __ballot(par & 1);
                    if (lane == 0) parw[b0 >> 6] ^= pb;
                }
            };
            uint64_t rsw;
            if (WPL == 1) {
                load(0);
                rsw = rsc[g.Wr + ((lane < nc ? myrow : 0) >> 6)];
                parity();
            } else {
                rsw = rsc[g.Wr + ((lane < nc ? myrow : 0) >> 6)];
            }
            rsum += __popcll(__ballot(lane < nc && ((rsw >> (myrow & 63)) & 1ull)));
            for (int u0 = 0; u0 < nc; u0 += kDetRowBatch) {
                if (u0 > 0 || WPL != 1) load(u0);
#pragma unroll
                for (int u = 0; u < kDetRowBatch; ++u) {
                    if (u0 + u >= nc) break;
#pragma unroll
                    for (int t = 0; t < WPL; ++t) {
                        const uint64_t a = rx[u][t] & msk[t], b = rz[u][t] & msk[t];
                        cr[t] ^= b & sx[t];
                        G += __popcll(a & b);
                        sx[t] ^= a;
                        sz[t] ^= b;
                    }
                }
            }
            if (WPL != 1) parity();
            cnt += nc;
            nc = 0;
        };
#pragma unroll
        for (int u = 0; u < WPL; ++u) {
            uint64_t lanes = __ballot(cd[u] != 0ull);
            while (lanes) {
                const int l = ctz64(lanes);
                lanes &= lanes - 1;
                uint64_t v = readlane_u64(cd[u], l);
                const int wb = l + 64 * u;
                while (v) {
                    const int bit = ctz64(v);
                    v &= v - 1;
                    if (lane == nc) myrow = wb * 64 + bit;
                    if (++nc == 64) flush();
                }
            }
        }
        if (nc) flush();
        uint64_t xres = 0;
#pragma unroll
        for (int t = 0; t < WPL; ++t) {
            G += 2 * __popcll(cr[t]) - __popcll(sx[t] & sz[t]);
            xres |= sx[t];
        }
        G = wave_sum(G);
        xres = wave_or(xres);
        const int e = (2 * rsum + G) & 3;
        if (lane == 0 && ((e & 1) || xres)) atomicOr(err, 1);
        const int shared = e >> 1;
        for (int b = lane; b < g.bpc; b += 64)
            obuf[(size_t)(s * g.bpc + b) * K + k] = (uint8_t)(shared ^ (int)((parw[b >> 6] >> (b & 63)) & 1ull));
        if (lane == 0) {
            atomicAdd(&s_det, 1u);
            atomicAdd(&s_rows, (unsigned int)cnt);
        }
    }();
    __syncthreads();
    if (threadIdx.x == 0 && s_det) {
        count_add(counters, pass == 0 ? 2 : 6, (unsigned long long)s_det);
        count_add(counters, 3, (unsigned long long)s_rows);
    }
}

// ------------------------------------------------------------------------------------------
// End of a measurement layer: resets (X on the qubit when the outcome is 1: every row with z
// at the qubit flips sign -- applied once for the whole layer, which is exact because sign
// flips commute with rowsum and with the other measurements of the layer) and the record.
// Block per (sign word w, group of up to kResetShots shots, chunk of kResetChunk targets), a
// wave per shot and its lanes over the chunk's targets.  The waves of a block read the same
// column words at about the same time, so a band's column comes from L2 once per block (the
// other waves hit in L1), not once per shot; the chunks keep enough blocks in flight.
// ------------------------------------------------------------------------------------------
constexpr int kResetShots = 16;
constexpr int kResetChunk = 1024;

__global__ void __launch_bounds__(64 * kResetShots)
k_reset_record(Geom g, uint64_t* __restrict__ rd, const uint64_t* __restrict__ Zcol,
               const uint8_t* __restrict__ obuf, int K, int do_reset, uint8_t* __restrict__ record,
               long long rec_stride, long long rec_off, int do_record)
{
    const int w = blk_x(g);
    const int lane = threadIdx.x & 63;
    const int b = blk_y(g) * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6);
    if (b >= g.B) return;                       // (no block barrier below)
    const int s = b / g.bpc;
    const int kc = (g.rev ? (int)gridDim.z - 1 - (int)blockIdx.z : (int)blockIdx.z) * kResetChunk;
    const int ke = min(K, kc + kResetChunk);
    const uint8_t* ob = obuf + (size_t)b * K;
    const uint64_t* Zc = Zcol + ((size_t)s * g.NB + w) * K;
    uint64_t acc = 0;
    // four targets per lane at a time, every load unconditional so they are all in flight
    for (int k0 = kc + lane; k0 < ke; k0 += 4 * 64) {
        uint8_t o[4];
        uint64_t z[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * 64;
            o[u] = k < ke ? ob[k] : (uint8_t)0;
            z[u] = (do_reset && k < ke) ? Zc[k] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * 64;
            if (o[u]) acc ^= z[u];
            if (do_record && w == 0 && k < ke) record[(size_t)b * rec_stride + rec_off + k] = o[u];
        }
    }
    if (do_reset) {
        acc = wave_xor(acc);
        if (lane == 0 && acc) atomicXor((unsigned long long*)&rd[(size_t)b * g.NB + w], (unsigned long long)acc);
    }
}

// Pack the byte-per-measurement record into bits, LSB first, ceil(M/8) bytes per shot.
__global__ void k_pack(const uint8_t* __restrict__ rec, long long M, int B, uint8_t* __restrict__ out)
{
    const long long nbytes = (M + 7) / 8;
    const long long total = nbytes * B;
    for (long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x; idx < total;
         idx += (long long)gridDim.x * blockDim.x) {
        const long long b = idx / nbytes, j = idx - b * nbytes;
        uint8_t v = 0;
        for (int t = 0; t < 8; ++t) {
            const long long m = j * 8 + t;
            if (m < M && rec[b * M + m]) v |= (uint8_t)(1u << t);
        }
        out[idx] = v;
    }
}

}  // namespace stabdev
