// stab_commute.hip -- pairwise commutation of bit-packed Pauli strings (Sec. 3.2: the
// grouping check).  Two strings commute group-wise iff the parity of
// sum_q (x1_q z2_q + z1_q x2_q) is even, and qubit-wise iff every single-qubit term of that
// sum is 0.  Strings are stored like tableau rows: ceil(n/64) x-words, then as many z-words.
//
// As a contraction: the qubits where A_i and B_j conflict number
//   sum_q [A = X] zB + [A = Z] xB + [A = Y] (xB ^ zB),
// a product of 0/1 matrices with 3n terms; the parity of the count is the group-wise bit, count > 0
// the qubit-wise one.  The matrix cores take it in fp4 with fp32 accumulation, which is exact: the
// terms are 0 and 1 and a count stays below 2^23 (kCommSpan).  An operand needs no conversion: with
// bits w, w + 4, ... of a word masked out in place, a nibble is 0.5, 1 or 2 by w (w = 3 shifted to
// 2), which the operand's block scale makes 1.  The order of the terms is the same for both
// operands, so only rows, columns and the accumulator's layout matter.
//
// A wave owns 64 strings A_i, whose operands it keeps in registers (up to 256 qubits), and walks over
// words of 64 strings B_j; the four waves of a block share the B_j.  B_j are the rows of a product,
// A_i its columns, so a lane has one A_i and packs its own 32 bits of a result word.
//
// At 32768 x 32768 strings of 256 qubits: 0.31 ms against 1.45 ms for the bitwise form (8 integer
// operations per pair and 64 qubits, bound by the VALU), which it replaces at every size (1000 x
// 1000 of 256: 7.5 and 7.3 us, both a launch; 3000 x 3000 of 1000: 26 and 59; 32768 x 32768 of 512:
// 816 and 3128).  The products alone take 0.17 ms at the fp4 peak; packing and masking, 92 VALU
// instructions per 12 products, run beside them in other waves.
//
// Included by stab_api.hip (same translation unit).

namespace stabdev {

constexpr int kCommThreads = 256;
constexpr int kCommRows = 64 * (kCommThreads / 64);                  // A strings per block
constexpr int kCommWords = 4;                                        // x (and z) words of a pass
constexpr int kCommRowWords = 16;                                    // result words of a block's row, at most
constexpr int kCommSpan = 1 << 14;                                   // passes (256 qubits) counted before packing

typedef int comm_op __attribute__((ext_vector_type(8)));             // fp4: the first four words
typedef float comm_acc __attribute__((ext_vector_type(16)));

// A lane's half of a pass's x and z words: the first two or the last two of four.
struct CommBits {
    uint32_t x[kCommWords], z[kCommWords];
};

__device__ __forceinline__ CommBits comm_load(const uint64_t* __restrict__ S, int i, int W, int w0, int half)
{
    const uint64_t* r = S + (size_t)i * 2 * W + w0 + 2 * half;
    uint64_t v[2][2];
    if (w0 + kCommWords <= W) {
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2), aligned(8)));
        const u64x2 x = *(const u64x2*)r, z = *(const u64x2*)(r + W);
        v[0][0] = x[0];
        v[0][1] = x[1];
        v[1][0] = z[0];
        v[1][1] = z[1];
    } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bool in = w0 + 2 * half + t < W;
            v[0][t] = in ? r[t] : 0ull;
            v[1][t] = in ? r[W + t] : 0ull;
        }
    }
    CommBits b;
#pragma unroll
    for (int t = 0; t < kCommWords; ++t) {
        b.x[t] = (uint32_t)(v[0][t >> 1] >> (32 * (t & 1)));
        b.z[t] = (uint32_t)(v[1][t >> 1] >> (32 * (t & 1)));
    }
    return b;
}

// Operand of bits w mod 4.
__device__ __forceinline__ comm_op comm_mask(const uint32_t (&v)[kCommWords], int w)
{
    comm_op o = {};
#pragma unroll
    for (int t = 0; t < kCommWords; ++t)
        o[t] = (int)(w == 3 ? (v[t] >> 1) & 0x44444444u : v[t] & (0x11111111u << w));
    return o;
}

// a: operand with rows B_j; b: with columns A_i; both of bits w mod 4.
__device__ __forceinline__ comm_acc comm_product(const comm_op& a, const comm_op& b, const comm_acc& c, int w)
{
    const int scale = w == 0 ? 128 : w == 1 ? 127 : 126;             // 2^(scale - 127)
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 4, 4, 0, scale, 0, scale);
}

// The accumulators start at 2^23, so that a count is the low bits of its float.
constexpr float kCommZero = 8388608.0f;

// The bits of a lane's 16 counts: row 8 (r / 4) + 4 (lane / 32) + r % 4 is accumulator r.
__device__ __forceinline__ void comm_pack(const comm_acc& c, int half, uint32_t& g, uint32_t& q)
{
    g = q = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        g = __builtin_amdgcn_alignbit(__float_as_uint(c[r]), g, 1);
        if (r % 4 == 3) g >>= 4;
        const int u = 15 - r;
        if (u % 4 == 3) q <<= 4;
        q = __builtin_amdgcn_alignbit(q, __float_as_uint(kCommZero) - __float_as_uint(c[u]), 31);
    }
    g <<= 4 * half;
    q <<= 4 * half;
}

// The three terms of a string on either side.
__device__ __forceinline__ void comm_terms(const CommBits& v, bool a, uint32_t (&f)[3][kCommWords])
{
#pragma unroll
    for (int t = 0; t < kCommWords; ++t) {
        f[0][t] = a ? v.x[t] & ~v.z[t] : v.z[t];
        f[1][t] = a ? v.z[t] & ~v.x[t] : v.x[t];
        f[2][t] = a ? v.x[t] & v.z[t] : v.x[t] ^ v.z[t];
    }
}

// Up to 256 qubits (ONE) the A_i operands stay in registers for all B_j; above, a pass takes 64 x 64
// strings at once, so that each side's are made once for two tiles.  Result words gather in LDS and
// leave as rows of up to 128 bytes, and strings are read 16 bytes a lane: with 8-byte stores to a
// line each and 4-byte loads the 32768 x 32768 case took 0.64 ms.
template <bool ONE>
__global__ void __launch_bounds__(kCommThreads, 2)
k_commute(const uint64_t* __restrict__ A, int na, const uint64_t* __restrict__ B, int nb, int W, int words,
          uint64_t* __restrict__ gc, uint64_t* __restrict__ qwc)
{
    __shared__ uint64_t out[2][kCommThreads][kCommRowWords + 1];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, wave = uni(tid >> 6);
    const int i0 = (int)blockIdx.y * kCommRows + wave * 64;
    if (i0 >= na) return;
    const int nbw = (nb + 63) >> 6;
    const int jw0 = (int)blockIdx.x * words, jw1 = min(nbw, jw0 + words);
    auto a_row = [&](int e) { return min(i0 + 32 * e + (lane & 31), na - 1); };
    auto b_row = [&](int jw, int h) { return min(min(jw, nbw - 1) * 64 + 32 * h + (lane & 31), nb - 1); };
    comm_acc zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = kCommZero;
    // each half-wave has every other four bits of both A tiles: to the words of lane i0 + lane
    auto word = [&](const comm_acc& t0, const comm_acc& t1, uint32_t& g, uint32_t& q) {
        uint32_t g0, g1, q0, q1;
        comm_pack(t0, half, g0, q0);
        comm_pack(t1, half, g1, q1);
        const auto gs = __builtin_amdgcn_permlane32_swap(g0, g1, false, false);
        const auto qs = __builtin_amdgcn_permlane32_swap(q0, q1, false, false);
        g ^= gs[0] | gs[1];
        q |= qs[0] | qs[1];
    };
    comm_op ops[2][3][4];
    CommBits next;
    if (ONE) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            uint32_t f[3][kCommWords];
            comm_terms(comm_load(A, a_row(e), W, 0, half), true, f);
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int w = 0; w < 4; ++w) ops[e][k][w] = comm_mask(f[k], w);
        }
        next = comm_load(B, b_row(jw0, 0), W, 0, half);
    }
    for (int jw = jw0; jw < jw1; ++jw) {
        uint32_t gw[2] = {0, 0}, qw[2] = {0, 0};                     // A_i's 64 bits: B_j 0..31, 32..63
        if (ONE) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                comm_acc acc[2] = {zero, zero};
                uint32_t f[3][kCommWords];
                comm_terms(next, false, f);
                next = comm_load(B, b_row(jw + h, 1 - h), W, 0, half);
#pragma unroll
                for (int w = 0; w < 4; ++w)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const comm_op b = comm_mask(f[k], w);
#pragma unroll
                        for (int e = 0; e < 2; ++e) acc[e] = comm_product(b, ops[e][k][w], acc[e], w);
                    }
                word(acc[0], acc[1], gw[h], qw[h]);
            }
        } else {
            for (int s0 = 0; s0 < W; s0 += kCommSpan * kCommWords) {
                comm_acc acc[2][2] = {{zero, zero}, {zero, zero}};   // [h][e]
                const int s1 = min(W, s0 + kCommSpan * kCommWords);
                CommBits na_[2], nb_[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    na_[e] = comm_load(A, a_row(e), W, s0, half);
                    nb_[e] = comm_load(B, b_row(jw, e), W, s0, half);
                }
                for (int w0 = s0; w0 < s1; w0 += kCommWords) {
                    uint32_t fa[2][3][kCommWords], fb[2][3][kCommWords];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        comm_terms(na_[e], true, fa[e]);
                        comm_terms(nb_[e], false, fb[e]);
                    }
                    const int wn = min(w0 + kCommWords, s1 - 1);     // (the last load is not used)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        na_[e] = comm_load(A, a_row(e), W, wn, half);
                        nb_[e] = comm_load(B, b_row(jw, e), W, wn, half);
                    }
#pragma unroll
                    for (int w = 0; w < 4; ++w)
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            const comm_op a0 = comm_mask(fa[0][k], w), a1 = comm_mask(fa[1][k], w);
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const comm_op b = comm_mask(fb[h][k], w);
                                acc[h][0] = comm_product(b, a0, acc[h][0], w);
                                acc[h][1] = comm_product(b, a1, acc[h][1], w);
                            }
                        }
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) word(acc[h][0], acc[h][1], gw[h], qw[h]);
            }
        }
        const int left = nb - jw * 64;
        const uint64_t in = left >= 64 ? ~0ull : (1ull << left) - 1;
        out[0][tid][jw - jw0] = ((uint64_t)gw[1] << 32 | gw[0]) & in;
        out[1][tid][jw - jw0] = ((uint64_t)qw[1] << 32 | qw[0]) & in;
    }
    // the wave's 64 rows, 16 lanes each four at a time (its own part of the LDS: no barrier)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int c = lane & (kCommRowWords - 1);
    if (c >= jw1 - jw0) return;
    for (int r = lane / kCommRowWords; r < min(64, na - i0); r += 64 / kCommRowWords) {
        const size_t o = (size_t)(i0 + r) * nbw + jw0 + c;
        if (gc) gc[o] = out[0][wave * 64 + r][c];
        if (qwc) qwc[o] = out[1][wave * 64 + r][c];
    }
}

}  // namespace stabdev
