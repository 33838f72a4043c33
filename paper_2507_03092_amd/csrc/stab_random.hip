// stab_random.hip -- the random measurements of a measurement layer (Sec. 2.4), included by
// stab_api.hip after stab_kernels.hip.
//
// Sequential semantics: targets are measured in op order; a random one has pivot p = the first
// stabilizer with x at its qubit; rowsum(i, p) for every other row i with x at the qubit; the
// pivot's destabilizer <- old row p (its own rowsum is overwritten); p <- Z_a with the outcome
// as its sign.  A target an earlier one made deterministic reads the stabilizers selected by
// the destabilizers with x at the qubit.
//
// A layer is taken in windows of up to 256 pending targets, two or three launches each:
//   k_plan   one block per tableau copy eliminates on the window's x bits alone.  Every row has a
//            mask M over the window: at step t its bits from t on are the row's x bits at the
//            targets still to come, its bits before t name the pivots whose rows, as they stood
//            before the window, have been multiplied into it.  Step t: the pivot is the first
//            stabilizer with bit t; every other row with bit t gets M ^= M[p] without bit t, which
//            turns its own bit t from "x at the target" into "multiplied by pivot t".
//   k_snap   copies the pivot rows as they stood before the window, with their signs, and draws
//            the outcomes (k_plan's waves do it when that is little).
//   k_apply  finds the mask every other row ends with and multiplies the row by the snapshots it
//            names.  The elimination acts linearly on a row's bits, so k_plan carries the unit
//            rows along with the tableau's: a row ends with the sum of what the units of its
//            bits end with.  A destabilizer whose partner is pivot t ends with what unit t does,
//            and nothing of its own.
// Every row becomes a product of rows that stood before the window, so all rows are independent
// of each other.  The products are exact: stabilizers commute with each other and with every
// destabilizer but their partner, and a partner is replaced outright, so the factors of each
// product commute and their order does not matter, signs included.
// ------------------------------------------------------------------------------------------

namespace stabdev {

constexpr int kListCap = 16;        // a pivot with more later targets makes its window "dense"
constexpr int kDenseFlag = 1 << 30;
constexpr int kApplyRows = 16;      // rows per block of k_apply: a quarter of a band

constexpr int kWinChunks = 4;       // 64-target chunks of a window
// Rows k_plan holds in LDS with kWinChunks mask words each: all of them up to n = 4096, above
// that only rows with x at some target of the window; a window with more of those is cut to its
// first 64 targets, one word a row.
constexpr int kPlanRows = 4096;

// Targets of a window that is not the layer's last, at least.
__host__ __device__ inline int least_window(const Geom& g) { return g.NR > kPlanRows ? 64 : 64 * kWinChunks; }

// Scratch of the random measurements (per copy s; Tc = min(64 kWinChunks, the program's largest layer)).
struct RandBufs {
    int4* win;        // [S] {pending targets of the layer, the window's first, how many, 0}; the count
                      // carries kDenseFlag if a pivot has x at more than kListCap later targets
    int* piv;         // [S][Tc] stabilizer index of the target's pivot, -1: deterministic by then
    int* cw;          // [S][Tc] i-exponent of the snapshot: |x & z| + 2 * shared sign (mod 4)
    int* dirty;       // [S][NB] quarters of the band changed in this layer (NULL: a layer takes one window at most)
    uint64_t* pm;     // [S][Tc][kWinChunks] of target t: in its own chunk's word, what unit t ends
                      // that chunk with (pivots of the chunk); in the others, its pivot's mask at
                      // the start of the chunk
    uint64_t* hit;    // [S][Tc] the chunk's steps that hit unit t, its own among them
    uint64_t* snap;   // [S][Tc][RS] the pivot row before the window
    uint64_t* lrd;    // [S][Tc][nrdw] its per-shot signs, bit b = shot b of the copy
    int Tc;
};

// In-register transpose of a 64x64 bit matrix held one row per lane, without the LDS crossbar:
// the off-diagonal 32x32 blocks change places in one permlane32 swap, then every 32x32 block is
// transposed by DPP steps.  Every lane must be active.
__device__ __forceinline__ uint64_t transpose64_dpp(uint64_t v, int lane)
{
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)(v >> 32), false, false);
    const uint32_t lo = transpose32(r[0], lane), hi = transpose32(r[1], lane);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

__device__ __forceinline__ uint64_t uni64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// ------------------------------------------------------------------------------------------
// k_plan: grid S.  Window 0 lists the layer's pending targets (random at its start, in op
// order); a window goes on where the one before it stopped.  The rows' masks lie in LDS in row
// order, and the window is taken 64 targets (one mask word) at a time: only rows with a bit in
// the chunk can be hit in it, and only that word decides who is, so the chunk's rows are listed,
// their words eliminated by one wave from registers (up to kOneWave rows, no barrier; more rows
// take the whole block, a barrier a step), and the other words follow from the outcome, all rows
// at once: row ^= the masks, as they stood before the chunk, of the pivots its word now names.
// Bound by the steps' dependent scalar chain (one wave), not by memory.
// ------------------------------------------------------------------------------------------
constexpr int kOneWave = 1024;

// Of one chunk's elimination.
struct ChunkLds {
    int key[2][16], pidx[64], hits;                     // pidx: the pivots, as indices in the row list (-1: none)
    uint64_t slot[2][16], pw[64];                       // pw: their words of the chunk at their steps
    uint64_t unit[64], uhit[64];                        // what the units end with; the steps that hit them
};

struct PlanLds {
    int k[64 * kWinChunks], piv[64 * kWinChunks], cnt[16], dense, nrun;
    ChunkLds c;
    uint64_t pm[64 * kWinChunks][kWinChunks], hit[64 * kWinChunks];
};

// Of the waves' counts cnt[0..nw), nw <= 16: the sum over the waves before this one, and the sum.
__device__ __forceinline__ int2 wave_counts(const int* cnt, int nw, int wave, int lane)
{
    const int v = (lane & 15) < nw ? cnt[lane & 15] : 0;
    int before = (lane & 15) < wave ? v : 0, total = v;
#pragma unroll
    for (int d = 1; d <= 8; d <<= 1) {
        before += (int)lane_xor32((uint32_t)before, d, lane);
        total += (int)lane_xor32((uint32_t)total, d, lane);
    }
    return make_int2(uni(before), uni(total));
}

// The window's start: the pending list (window 0) and the first target; returns how many pending
// targets are left from it on, 0 at the end of the layer.
__device__ __forceinline__ int plan_begin(const Geom& g, PlanLds& L, int K, const int* cls, int* pd, const RandBufs& R,
                                          int win, int* ran, int s, int& start)
{
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = uni(tid >> 6), nw = nt >> 6;
    int np;
    start = 0;
    if (win == 0) {
        int base = 0;
        for (int k0 = 0; k0 < K; k0 += nt) {
            const int k = k0 + tid;
            const bool f = k < K && cls[(size_t)s * K + k] >= 0;
            const uint64_t m = __ballot(f);
            if (lane == 0) L.cnt[wave] = __popcll(m);
            __syncthreads();
            const int2 pc = wave_counts(L.cnt, nw, wave, lane);
            const int at = base + pc.x + __popcll(m & ((1ull << lane) - 1ull));
            if (f) {
                pd[at] = k;
                if (at < R.Tc) L.k[at] = k;
            }
            base += pc.y;
            __syncthreads();
        }
        np = base;
        if (R.dirty)
            for (int b = tid; b < g.NB; b += nt) R.dirty[(size_t)s * g.NB + b] = 0;
    } else {
        const int4 v = R.win[s];
        np = v.x;
        start = v.y + (v.z & ~kDenseFlag);
        for (int t = tid; t < min(R.Tc, np - start); t += nt) L.k[t] = pd[start + t];
    }
    __syncthreads();
    if (tid == 0) {
        R.win[s] = make_int4(np, start, 0, 0);         // (z: plan_end, if there is a target left)
        if (np > start) atomicMax(ran, win + 1);
        L.dense = 0;
        L.nrun = 0;
        L.c.hits = 0;
    }
    __syncthreads();
    return np - start;
}

// The elimination of one chunk on its mask words by one wave; row i of the list is lane i % 64's
// w[i / 64].
template <int R>
__device__ __forceinline__ void chunk_steps_wave(ChunkLds& L, uint64_t* Mc, const uint16_t* act, int na, int nt)
{
    const int lane = threadIdx.x & 63;
    uint32_t w[R][2];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const uint64_t v = u * 64 + lane < na ? Mc[act[u * 64 + lane]] : 0ull;
        w[u][0] = (uint32_t)v;
        w[u][1] = (uint32_t)(v >> 32);
    }
    int hits = 0, mypiv = -1;                     // (hits: per lane)
    uint32_t mypw[2] = {0u, 0u}, hist[2] = {0u, 0u};
    uint32_t un[2] = {lane < nt && lane < 32 ? 1u << lane : 0u, lane < nt && lane >= 32 ? 1u << (lane - 32) : 0u};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int te = min(32, nt - 32 * h);
#pragma unroll R <= 4 ? 4 : 1
        for (int j = 0; j < te; ++j) {
            int mk[R];                            // -1: hit
            uint64_t bm[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                mk[u] = __builtin_amdgcn_sbfe((int)w[u][h], j, 1);
                bm[u] = __ballot(mk[u] != 0);
            }
            const int mu = __builtin_amdgcn_sbfe((int)un[h], j, 1);
            // the first row: up to four masks at a time, selects instead of branches within them
            constexpr int Q = R < 4 ? R : 4;
            int pi = -1;
            uint32_t p0 = 0, p1 = 0;
#pragma unroll
            for (int v = 0; v < R; v += Q) {
                uint64_t some = 0;
#pragma unroll
                for (int u = v; u < v + Q; ++u) some |= bm[u];
                if (R == Q || (pi < 0 && some)) {
                    uint64_t b = bm[v];
                    uint32_t q0 = w[v][0], q1 = w[v][1];
                    int at = 64 * v;
#pragma unroll
                    for (int u = v + 1; u < v + Q; ++u) {
                        const bool none = b == 0ull;
                        b = none ? bm[u] : b;
                        q0 = none ? w[u][0] : q0;
                        q1 = none ? w[u][1] : q1;
                        at = none ? 64 * u : at;
                    }
                    const int l = ctz64(b | 1ull << 63);
                    p0 = (uint32_t)__builtin_amdgcn_readlane((int)q0, l);
                    p1 = (uint32_t)__builtin_amdgcn_readlane((int)q1, l);
                    // (without a row nothing changes)
                    pi = b ? at + l : -1;
                    p0 = b ? p0 : 0u;
                    p1 = b ? p1 : 0u;
                }
            }
            const bool me = lane == 32 * h + j;
            mypiv = me ? pi : mypiv;
            mypw[0] = me ? p0 : mypw[0];
            mypw[1] = me ? p1 : mypw[1];
            const uint32_t bit = pi < 0 ? 0u : 1u << j;
            if (h) p1 ^= bit;
            else p0 ^= bit;
#pragma unroll
            for (int u = 0; u < R; ++u) {
                hits -= mk[u];
                // (the pivot itself is left with its own bit alone: it is never hit again)
                w[u][0] ^= (uint32_t)mk[u] & p0;
                w[u][1] ^= (uint32_t)mk[u] & p1;
            }
            un[0] ^= (uint32_t)mu & p0;
            un[1] ^= (uint32_t)mu & p1;
            hist[h] |= (uint32_t)mu & bit;
        }
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (u * 64 + lane < na) Mc[act[u * 64 + lane]] = (uint64_t)w[u][0] | ((uint64_t)w[u][1] << 32);
    L.pidx[lane] = mypiv;
    L.pw[lane] = (uint64_t)mypw[0] | ((uint64_t)mypw[1] << 32);
    L.unit[lane] = (uint64_t)un[0] | ((uint64_t)un[1] << 32);
    L.uhit[lane] = (uint64_t)hist[0] | ((uint64_t)hist[1] << 32);
    hits = wave_sum(hits);
    if (lane == 0) L.hits += hits;
}

// The same by a block of 64 NW threads, row i of the list being thread i % (64 NW)'s w[i / (64 NW)].
// Each wave offers its first row with the bit in a slot of its own and takes the lowest offer;
// the slots alternate between two sets, so a wave that runs ahead writes the set nobody reads.
template <int R, int NW>
__device__ __forceinline__ void chunk_steps_block(ChunkLds& L, uint64_t* Mc, const uint16_t* act, int na, int nt)
{
    constexpr int NT = 64 * NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    uint64_t w[R];
#pragma unroll
    for (int u = 0; u < R; ++u) w[u] = u * NT + tid < na ? Mc[act[u * NT + tid]] : 0ull;
    uint64_t un = lane < nt ? 1ull << lane : 0ull, hist = 0ull;   // (wave 0's are kept)
    int hits = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int te = min(32, nt - 32 * h);
        for (int j = 0; j < te; ++j) {
            const uint32_t bit = 1u << j;
            const int buf = j & 1;
            bool hb[R];
            uint64_t bm[R];
            int first = INT_MAX;
#pragma unroll
            for (int u = R - 1; u >= 0; --u) {
                hb[u] = ((uint32_t)(w[u] >> (32 * h)) & bit) != 0u;
                bm[u] = __ballot(hb[u]);
                if (bm[u]) first = u * NT + wave * 64 + ctz64(bm[u]);
            }
            if (lane == 0) L.key[buf][wave] = first;
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (first == u * NT + tid) L.slot[buf][wave] = w[u];
            __syncthreads();
            int pi = (lane & 15) < NW ? L.key[buf][lane & 15] : INT_MAX;
#pragma unroll
            for (int d = 1; d <= 8; d <<= 1) pi = min(pi, (int)lane_xor32((uint32_t)pi, d, lane));
            pi = uni(pi);
            const uint64_t pw = pi == INT_MAX ? 0ull : L.slot[buf][(pi >> 6) & (NW - 1)];
            if (tid == 0) {
                L.pidx[32 * h + j] = pi == INT_MAX ? -1 : pi;
                L.pw[32 * h + j] = pw;
            }
            if (pi == INT_MAX) continue;
            const uint64_t px = pw ^ ((uint64_t)bit << (32 * h));
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (!bm[u]) continue;
                hits += __popcll(bm[u]);
                if (hb[u]) w[u] ^= px;
            }
            if ((un >> (32 * h + j)) & 1ull) {
                un ^= px;
                hist |= 1ull << (32 * h + j);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
        if (u * NT + tid < na) Mc[act[u * NT + tid]] = w[u];
    if (wave == 0) {
        L.unit[lane] = un;
        L.uhit[lane] = hist;
    }
    if (lane == 0) atomicAdd(&L.hits, hits);
}

// What the snapshots are taken of, and the outcome draws' key.
struct Snap {
    const uint64_t* tab;
    const uint64_t* rs;
    const uint64_t* rd;
    uint8_t* obuf;
    uint64_t seed, first_shot, instr;
    int pos_base;
    int fused;      // k_plan takes the snapshots
};

// How many pending targets the window leaves (the first copy's count, the same in all), with the
// launch's number, to a word of pinned host memory: the host reads it while the window is planned.
template <bool POST>
__device__ __forceinline__ void post_left(uint64_t* post, uint32_t seq, int s, int left)
{
    if (POST && s == 0 && threadIdx.x == 0)
        __hip_atomic_store(post, (uint64_t)seq << 32 | (uint32_t)left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The snapshot of target t (index k in its layer, pivot p) by a group of 64 nw threads, wave w of
// it: row and i-exponent by the first wave, per-shot signs and outcome draws by all.
__device__ __forceinline__ void snap_target(const Geom& g, const Snap& S, const RandBufs& R, int s, int t, int k, int p,
                                            int K, int w, int nw)
{
    const int lane = threadIdx.x & 63, nrdw = (g.bpc + 63) >> 6;
    const int pw = g.Wr + (p >> 6), pb = p & 63;
    if (w == 0) {
        const uint64_t* row = S.tab + ((size_t)s * 2 * g.NR + g.NR + p) * g.RS;
        uint64_t* dst = R.snap + ((size_t)s * R.Tc + t) * g.RS;
        const uint64_t sw = S.rs[(size_t)s * g.NB + pw];
        int wt = 0;
        for (int j = lane; j < g.Wc; j += 64) {
            const uint64_t x = row[j], z = row[g.Wc + j];
            dst[j] = x;
            dst[g.Wc + j] = z;
            wt += __popcll(x & z);
        }
        wt = wave_sum(wt);
        if (lane == 0) R.cw[(size_t)s * R.Tc + t] = (wt + 2 * (int)((sw >> pb) & 1ull)) & 3;
    }
    for (int u = w; u < nrdw; u += nw) {
        const int b = 64 * u + lane;
        const int gb = s * g.bpc + min(b, g.bpc - 1);
        const uint64_t v = S.rd[(size_t)gb * g.NB + pw];
        uint64_t u0, u1;
        philox(S.instr, (uint64_t)(S.pos_base + k), S.seed, S.first_shot + (uint64_t)gb, u0, u1);
        const uint64_t m = __ballot(b < g.bpc && ((v >> pb) & 1ull));
        if (b < g.bpc) S.obuf[(size_t)gb * K + k] = (uint8_t)(u0 >> 63);
        if (lane == 0) R.lrd[((size_t)s * R.Tc + t) * nrdw + u] = m;
    }
}

__device__ __forceinline__ void plan_end(PlanLds& L, int K, int* cls, const RandBufs& R, int s, int nwt,
                                         unsigned long long* counters)
{
    constexpr int TW = kWinChunks;
    const int tid = threadIdx.x, nt = blockDim.x;
    // (stores last: nothing waits for them)
    for (int i = tid; i < nwt * TW; i += nt) R.pm[(size_t)s * R.Tc * TW + i] = (&L.pm[0][0])[i];
    for (int t = tid; t < nwt; t += nt) {
        R.piv[(size_t)s * R.Tc + t] = L.piv[t];
        R.hit[(size_t)s * R.Tc + t] = L.hit[t];
        if (L.piv[t] < 0) cls[(size_t)s * K + L.k[t]] = -2;   // deterministic by now: reduced after the layer
    }
    if (tid == 0) {
        R.win[s].z = nwt | (L.dense ? kDenseFlag : 0);
        count_add(counters, 0, 1ull);
        if (L.dense) count_add(counters, 1, 1ull);
        count_add(counters, 4, (unsigned long long)L.nrun);
        count_add(counters, 5, (unsigned long long)(L.c.hits - L.nrun));
    }
}

// Dynamic LDS: the row list's masks, its rows and the chunk's list.
__host__ __device__ inline int plan_lds_bytes(int NR)
{
    return NR <= kPlanRows ? NR * (kWinChunks * 8 + 4) : kPlanRows * (kWinChunks * 8 + 4);
}
static_assert(kPlanRows * (kWinChunks * 8 + 4) >= kMaxBands * 64 * 12, "a cut window's one-word rows must fit");

template <bool POST>
__global__ void __launch_bounds__(1024)
k_plan(Geom g, const uint64_t* __restrict__ Xcol, int K, int* __restrict__ cls, int* __restrict__ pend, RandBufs R,
       int win, int* __restrict__ ran, Snap S, unsigned long long* __restrict__ counters, uint64_t* post, uint32_t seq)
{
    constexpr int TW = kWinChunks;
    extern __shared__ uint64_t M[];                       // [tw][cap] masks
    __shared__ PlanLds L;
    const int s = blk_x(g);
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = uni(tid >> 6), nw = nthr >> 6;
    int start;
    const int left = plan_begin(g, L, K, cls, pend + (size_t)s * K, R, win, ran, s, start);
    if (left <= 0) {
        post_left<POST>(post, seq, s, 0);
        return;
    }
    int nwt = min(R.Tc, left), tw = TW, cap = min(g.NR, kPlanRows), n = 0;
    const uint64_t* Xs = Xcol + (size_t)s * g.NB * K + (size_t)g.Wr * K;
    uint16_t *rid, *act;
    // the window's x columns, 64 rows x 64 targets at a time, turned into a mask per row; rows
    // without a bit are dropped, the others listed in row order (a wave takes bp bands in a row)
    while (true) {
        rid = (uint16_t*)(M + (size_t)cap * tw);
        act = rid + cap;
        int kc[TW];
#pragma unroll
        for (int c = 0; c < TW; ++c) kc[c] = 64 * c + lane < nwt ? L.k[64 * c + lane] : -1;
        const int bp = min(4, (g.Wr + nw - 1) / nw);
        n = 0;
        for (int b0 = 0; b0 < g.Wr; b0 += nw * bp) {
            uint64_t v[4][TW], nz[4];
            int mine = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int band = b0 + wave * bp + i;
                const bool in = i < bp && band < g.Wr;
#pragma unroll
                for (int c = 0; c < TW; ++c) v[i][c] = (in && kc[c] >= 0) ? Xs[(uint32_t)(band * K + kc[c])] : 0ull;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint64_t o = 0;
#pragma unroll
                for (int c = 0; c < TW; ++c) {
                    if (__ballot(v[i][c] != 0ull)) v[i][c] = transpose64_dpp(v[i][c], lane);
                    o |= v[i][c];
                }
                nz[i] = __ballot(o != 0ull);
                mine += __popcll(nz[i]);
            }
            if (lane == 0) L.cnt[wave] = mine;
            __syncthreads();
            const int2 pc = wave_counts(L.cnt, nw, wave, lane);
            int at = n + pc.x;
            n += pc.y;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int pos = at + __popcll(nz[i] & ((1ull << lane) - 1ull));
                if (((nz[i] >> lane) & 1ull) && pos < cap) {
                    rid[pos] = (uint16_t)((b0 + wave * bp + i) * 64 + lane);
#pragma unroll
                    for (int c = 0; c < TW; ++c)
                        if (c < tw) M[c * cap + pos] = v[i][c];
                }
                at += __popcll(nz[i]);
            }
            __syncthreads();
        }
        if (n <= cap) break;
        nwt = min(nwt, 64);
        tw = 1;
        cap = g.NR;
    }
    post_left<POST>(post, seq, s, left - nwt);
    const int nch = (nwt + 63) >> 6;
    const int per = (n + nthr - 1) / nthr;                 // 64-row runs of the list a wave takes
    for (int c = 0; c < nch; ++c) {
        const int nt = min(64, nwt - 64 * c);
        // rows with a bit in the chunk, in row order
        int mine = 0;
        for (int q = 0; q < per; ++q) {
            const int i = (wave * per + q) * 64 + lane;
            mine += __popcll(__ballot(i < n && M[c * cap + i] != 0ull));
        }
        if (lane == 0) L.cnt[wave] = mine;
        if (tid < 64) {
            L.c.pidx[tid] = -1;
            L.c.unit[tid] = L.c.uhit[tid] = 0ull;
        }
        __syncthreads();
        const int2 pc = wave_counts(L.cnt, nw, wave, lane);
        int at = pc.x;
        const int na = pc.y;
        for (int q = 0; q < per; ++q) {
            const int i = (wave * per + q) * 64 + lane;
            const bool f = i < n && M[c * cap + i] != 0ull;
            const uint64_t m = __ballot(f);
            if (f) act[at + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)i;
            at += __popcll(m);
        }
        __syncthreads();
        if (na <= kOneWave) {
            if (wave == 0 && na > 0) {
                uint64_t* Mc = M + (size_t)c * cap;
                if (na <= 64) chunk_steps_wave<1>(L.c, Mc, act, na, nt);
                else if (na <= 128) chunk_steps_wave<2>(L.c, Mc, act, na, nt);
                else if (na <= 256) chunk_steps_wave<4>(L.c, Mc, act, na, nt);
                else chunk_steps_wave<kOneWave / 64>(L.c, Mc, act, na, nt);
            }
        } else if (na <= 4096) {
            chunk_steps_block<4, 16>(L.c, M + (size_t)c * cap, act, na, nt);
        } else {
            chunk_steps_block<kMaxBands / 16, 16>(L.c, M + (size_t)c * cap, act, na, nt);
        }
        __syncthreads();
        for (int t = tid; t < nt; t += nthr) {
            const int pi = L.c.pidx[t];
            const uint64_t runm = __ballot(pi >= 0);       // (t = lane: 64 threads, one wave, take it)
            const int row = pi >= 0 ? act[pi] : 0;
            int later = pi >= 0 ? __popcll(L.c.pw[t] & (t < 63 ? ~0ull << (t + 1) : 0ull)) : 0;
#pragma unroll
            for (int w = 0; w < TW; ++w) {
                uint64_t v = pi >= 0 && w != c && w < nch ? M[w * cap + row] : 0ull;
                if (w > c) later += __popcll(v);
                if (w == c) v = L.c.unit[t] & runm;
                L.pm[64 * c + t][w] = v;
            }
            L.hit[64 * c + t] = L.c.uhit[t];
            L.piv[64 * c + t] = pi >= 0 ? (int)rid[row] : -1;
            if (later > kListCap) L.dense = 1;
            if (t == 0) L.nrun += __popcll(runm);
        }
        __syncthreads();
        // the other words of the chunk's rows (a pivot names itself alone and becomes 0)
        if (nch > 1) {
            for (int e = tid; e < na; e += nthr) {
                const int i = act[e];
                uint64_t f = M[c * cap + i], v[TW];
#pragma unroll
                for (int w = 0; w < TW; ++w) v[w] = 0ull;
                while (f) {
                    const uint64_t* q = L.pm[64 * c + ctz64(f)];
                    f &= f - 1;
#pragma unroll
                    for (int w = 0; w < TW; ++w) v[w] ^= q[w];
                }
#pragma unroll
                for (int w = 0; w < TW; ++w)
                    if (w != c && w < nch) M[w * cap + i] ^= v[w];
            }
            __syncthreads();
        }
    }
    if (S.fused)
        for (int t = wave; t < nwt; t += nw) {
            const int p = uni(L.piv[t]);
            if (p >= 0) snap_target(g, S, R, s, t, uni(L.k[t]), p, K, 0, 1);
        }
    plan_end(L, K, cls, R, s, nwt, counters);
}

// ------------------------------------------------------------------------------------------
// k_snap: grid (Tc, S), a block per target of the window; not launched when k_plan's waves took the
// snapshots (Snap::fused).
// ------------------------------------------------------------------------------------------
constexpr int kSnapThreads = 256;

__global__ void __launch_bounds__(kSnapThreads)
k_snap(Geom g, int K, const int* __restrict__ pend, Snap S, RandBufs R)
{
    const int t = blk_x(g), s = blk_y(g);
    const int4 wn = R.win[s];
    if (t >= (wn.z & ~kDenseFlag)) return;
    const int p = uni(R.piv[(size_t)s * R.Tc + t]);
    if (p < 0) return;
    snap_target(g, S, R, s, t, uni(pend[(size_t)s * K + wn.y + t]), p, K, uni(threadIdx.x >> 6), kSnapThreads / 64);
}

// ------------------------------------------------------------------------------------------
// k_apply: grid (8 Wr quarter bands, S): 16 rows a block, which fills the chip for small tableaux
// and spreads the bands most targets hit.
// One wave turns the rows' x bits into masks, four lanes a row.  Rows are then updated by groups of lanes, the smallest power of two that covers
// a row's x words, four snapshots in flight; the per-shot signs by a wave per 64 shots.  The phase
// is telescoped: multiplying P_1..P_m into D raises i to sum |P| + |D| - |product| +
// 2 sum z_P.x_D (mod 4), |u| the number of qubits where u has both x and z, and only the parity
// of the last sum matters.  Last, a quarter band some window of this layer changed writes its part
// of the x columns of the next window's targets.
// ------------------------------------------------------------------------------------------
constexpr int apply_threads(int wpl) { return wpl == 1 ? 256 : 512; }

template <int WPL>
__global__ void __launch_bounds__(apply_threads(WPL))
k_apply(Geom g, uint64_t* __restrict__ tab, uint64_t* __restrict__ rs, uint64_t* __restrict__ rd,
        uint64_t* __restrict__ Xcol, int K, const int* __restrict__ tq, const int* __restrict__ pend, RandBufs R,
        const uint8_t* __restrict__ obuf, int* __restrict__ err, unsigned long long* __restrict__ counters)
{
    constexpr int TW = kWinChunks, T = 64 * TW, kThreads = apply_threads(WPL), kWaves = kThreads / 64;
    static_assert(kWaves >= TW && kApplyRows * TW == 64, "a wave per chunk; a lane per row and chunk");
    const int quarter = blk_x(g) & 3, band = blk_x(g) >> 2, s = blk_y(g);
    const int4 wn = R.win[s];
    const int cnt = wn.z, nwt = cnt & ~kDenseFlag;
    if (nwt == 0) return;
    __shared__ int s_k[T], s_piv[T], s_list[kApplyRows], s_pt[kApplyRows];
    __shared__ uint64_t s_pm[T][TW], s_hit[T], s_M[TW][kApplyRows], s_l[kWaves][T];
    __shared__ unsigned long long s_nz[TW], s_sp[TW], s_run[TW];
    __shared__ unsigned int s_ph, s_act, s_rep, s_pvm;
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int Wc = g.Wc, RS = g.RS, NB = g.NB, nrdw = (g.bpc + 63) >> 6;
    const bool destab = band < g.Wr;
    const int hq = (destab ? band : band - g.Wr) * 4 + quarter;     // the quarter within its half
    const int* pd = pend + (size_t)s * K + wn.y;
    uint16_t* X = (uint16_t*)(Xcol + ((size_t)s * NB + band) * K) + quarter;   // (X[4 k]: 16 rows at target k)
    uint64_t* tb = tab + ((size_t)s * 2 * g.NR + (size_t)band * 64 + quarter * kApplyRows) * RS;

    if (tid < kApplyRows) s_pt[tid] = -1;
    __syncthreads();
    // the window's targets and pivots, and the rows' x bits at them
    if (wave < TW) {
        const int t = 64 * wave + lane;
        const int k = t < nwt ? pd[t] : -1;
        const int p = t < nwt ? R.piv[(size_t)s * R.Tc + t] : -1;
        // (a target that did not run selects stabilizers by its bits, it hits nothing)
        uint64_t v = p >= 0 ? (uint64_t)X[4 * (size_t)k] : 0ull;
        s_k[t] = k;
        s_piv[t] = p;
        const uint64_t run = __ballot(p >= 0), nz = __ballot(v != 0ull);
        const uint64_t sp = __ballot(p >= 0 && (p / kApplyRows) == hq);
        if ((sp >> lane) & 1ull) s_pt[p & (kApplyRows - 1)] = t;
        if (nz) v = transpose64_dpp(v, lane);
        if (lane < kApplyRows) s_M[wave][lane] = v;
        if (lane == 0) {
            s_run[wave] = run;
            s_nz[wave] = nz;
            s_sp[wave] = sp;
        }
    }
    if (tid == 0) {
        s_ph = 0u;
        s_bad = 0;
    }
    __syncthreads();
    bool any = false;
#pragma unroll
    for (int c = 0; c < TW; ++c) any |= (s_nz[c] | s_sp[c]) != 0ull;
    if (any) {
        const uint64_t* gp = R.pm + (size_t)s * R.Tc * TW;
        for (int i = tid; i < nwt * TW; i += kThreads) (&s_pm[0][0])[i] = gp[i];
        const uint64_t* gh = R.hit + (size_t)s * R.Tc;
        for (int i = tid; i < nwt; i += kThreads) s_hit[i] = gh[i];
        __syncthreads();
        if (wave == 0) {
            // lane = row + 16 q: the four lanes of a row take 16 bits of a word each and hold the
            // row's whole mask
            const int nch = (nwt + 63) >> 6, r = lane & (kApplyRows - 1), q = lane / kApplyRows;
            const int own = s_pt[r];                       // the target whose pivot is the row (or its partner)
            const int pt = destab ? -1 : own;
            uint64_t M[TW];
#pragma unroll
            for (int c = 0; c < TW; ++c) M[c] = pt < 0 ? s_M[c][r] : 0ull;
            int rep = 0, nh = 0;
#pragma unroll
            for (int c = 0; c < TW; ++c) {
                if (c >= nch) break;
                uint64_t f = M[c] & (0xffffull << (16 * q)), F = 0ull, H = 0ull;
                if (__ballot(f != 0ull)) {
                    while (f) {
                        const int t = 64 * c + ctz64(f);
                        f &= f - 1;
                        F ^= s_pm[t][c];
                        H ^= s_hit[t];
                    }
                    F ^= shfl_xor_u64(F, 16);
                    H ^= shfl_xor_u64(H, 16);
                    F ^= shfl_xor_u64(F, 32);
                    H ^= shfl_xor_u64(H, 32);
                }
                if (destab && own >= 0 && (own >> 6) >= c) {
                    // a partner: nothing of its own, up to its pivot's step nothing at all
                    F = H = 0ull;
                    if ((own >> 6) == c) {
                        rep = 1;
                        F = s_pm[own][c];
                        H = s_hit[own] & ~(1ull << (own & 63));
#pragma unroll
                        for (int i = 0; i < TW; ++i) M[i] = 0ull;
                    }
                }
                M[c] = F;
                nh += __popcll(H);
                if (nch > 1) {
                    f = F & (0xffffull << (16 * q));
                    if (__ballot(f != 0ull)) {
                        uint64_t a[TW];
#pragma unroll
                        for (int i = 0; i < TW; ++i) a[i] = 0ull;
                        while (f) {
                            const uint64_t* v = s_pm[64 * c + ctz64(f)];
                            f &= f - 1;
#pragma unroll
                            for (int i = 0; i < TW; ++i) a[i] ^= v[i];
                        }
#pragma unroll
                        for (int i = 0; i < TW; ++i) {
                            if (i == c) continue;
                            a[i] ^= shfl_xor_u64(a[i], 16);
                            a[i] ^= shfl_xor_u64(a[i], 32);
                            // (bits at targets that do not run hit nothing)
                            M[i] ^= a[i] & s_run[i];
                        }
                    }
                }
            }
            uint64_t eo = 0;
#pragma unroll
            for (int c = 0; c < TW; ++c) {
                if (lane < kApplyRows) s_M[c][lane] = M[c];
                eo |= M[c];
            }
            const bool first = lane < kApplyRows;
            const uint64_t rm = __ballot(first && rep), pm = __ballot(first && pt >= 0),
                           am = __ballot(first && eo != 0ull) | rm, all = am | pm;
            if ((all >> lane) & 1ull) s_list[__popcll(all & ((1ull << lane) - 1ull))] = lane;
            const int nwalk = __popcll(__ballot(first && (nh > 0 || rep)));
            nh = wave_sum(first ? nh : 0);
            if (lane == 0) {
                s_act = (unsigned int)am;
                s_rep = (unsigned int)rm;
                s_pvm = (unsigned int)pm;
                if (destab && nwalk) {
                    count_add(counters, 8, (unsigned long long)nh);
                    count_add(counters, 9, (unsigned long long)nwalk);
                    if (cnt & kDenseFlag) {
                        count_add(counters, 10, (unsigned long long)nwalk);
                        count_add(counters, 11, (unsigned long long)(nh + __popcll(rm)));
                    }
                }
            }
        }
        __syncthreads();
        const unsigned int rm = s_rep, pm = s_pvm, repl = rm | pm, all = s_act | pm;
        const int nrows = __popc(all);
        // ---- rows ----
        int lpr = 64;
        if (WPL == 1)
            while (lpr > 1 && (lpr >> 1) >= Wc) lpr >>= 1;
        const int groups = 64 / lpr, grp = lane / lpr, sub = lane & (lpr - 1);
        const uint64_t* snap = R.snap + (size_t)s * R.Tc * RS;
        const int* cw = R.cw + (size_t)s * R.Tc;
        for (int i0 = wave * groups; i0 < nrows; i0 += kWaves * groups) {
            const int i = i0 + grp;
            const bool ok = i < nrows;
            const int r = s_list[ok ? i : 0];
            const bool own = !((repl >> r) & 1u);           // the row keeps its own factor
            const bool isp = (pm >> r) & 1u;
            uint64_t* row = tb + (size_t)r * RS;
            uint64_t x[WPL], z[WPL], cr[WPL];
            int G = 0, Gs = 0;
#pragma unroll
            for (int q = 0; q < WPL; ++q) {
                const int cwd = sub + 64 * q;
                const bool in = ok && own && cwd < Wc;
                x[q] = in ? row[cwd] : 0ull;
                z[q] = in ? row[Wc + cwd] : 0ull;
                cr[q] = 0ull;
            }
#pragma unroll
            for (int q = 0; q < WPL; ++q) G += __popcll(x[q] & z[q]);
#pragma unroll
            for (int c = 0; c < TW; ++c) {
                uint64_t m = ok ? s_M[c][r] : 0ull;
                while (m) {
                    uint64_t px[4][WPL], pz[4][WPL];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const bool on = m != 0ull;
                        const int t = 64 * c + (on ? ctz64(m) : 0);
                        m &= m - 1;
                        if (on) Gs += cw[t];
                        const uint64_t* pr = snap + (size_t)t * RS;
#pragma unroll
                        for (int q = 0; q < WPL; ++q) {
                            const int cwd = sub + 64 * q;
                            const bool in = on && cwd < Wc;
                            px[v][q] = in ? pr[cwd] : 0ull;
                            pz[v][q] = in ? pr[Wc + cwd] : 0ull;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int q = 0; q < WPL; ++q) {
                            cr[q] ^= pz[v][q] & x[q];
                            x[q] ^= px[v][q];
                            z[q] ^= pz[v][q];
                        }
                }
            }
#pragma unroll
            for (int q = 0; q < WPL; ++q) G += 2 * __popcll(cr[q]) - __popcll(x[q] & z[q]);
            for (int d = lpr >> 1; d >= 1; d >>= 1) G += __shfl_xor(G, d, 64);
            G = (G + Gs) & 3;
            if (ok) {
                const int a = isp ? tq[s_k[s_pt[r]]] : -1;
#pragma unroll
                for (int q = 0; q < WPL; ++q) {
                    const int cwd = sub + 64 * q;
                    if (cwd < Wc) {
                        row[cwd] = x[q];
                        row[Wc + cwd] = isp ? (cwd == (a >> 6) ? 1ull << (a & 63) : 0ull) : z[q];
                    }
                }
                if (sub == 0 && !isp) {
                    if (G & 1) s_bad = 1;
                    if (G & 2) atomicXor(&s_ph, 1u << r);
                }
            }
        }
        // ---- per-shot signs: lane = row + 16 * chunk ----
        if (all) {
            for (int u = wave; u < nrdw; u += kWaves) {
                const uint64_t* lr = R.lrd + (size_t)s * R.Tc * nrdw + u;
                for (int t = lane; t < nwt; t += 64) s_l[wave][t] = s_piv[t] >= 0 ? lr[(size_t)t * nrdw] : 0ull;
                __builtin_amdgcn_wave_barrier();
                const int c = lane / kApplyRows;
                uint64_t F = 0, m = s_M[c][lane & (kApplyRows - 1)];
                while (m) {
                    F ^= s_l[wave][64 * c + ctz64(m)];
                    m &= m - 1;
                }
                F ^= shfl_xor_u64(F, 16);
                F ^= shfl_xor_u64(F, 32);
                const uint32_t flip = (uint32_t)transpose64_dpp(lane < kApplyRows ? F : 0ull, lane);
                const int b = 64 * u + lane;
                const bool in = b < g.bpc;
                const int gb = s * g.bpc + min(b, g.bpc - 1);
                uint16_t* w = (uint16_t*)(rd + (size_t)gb * NB + band) + quarter;
                const uint32_t old = in ? *w : 0u;
                uint32_t nv = (old & ~repl) ^ flip;
                uint32_t q = (uint32_t)uni((int)pm);
                while (q) {
                    const int r = __builtin_ctz(q);
                    q &= q - 1;
                    if (obuf[(size_t)gb * K + s_k[s_pt[r]]]) nv ^= 1u << r;
                }
                if (in && nv != old) *w = (uint16_t)nv;
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
        if (tid == 0 && all) {
            uint16_t* w = (uint16_t*)(rs + (size_t)s * NB + band) + quarter;
            *w = (uint16_t)((*w & ~repl) ^ s_ph);
            if (s_bad) atomicOr(err, destab ? 8 : 4);
        }
        any = all != 0u;
    }
    // ---- the next window's x columns: lane = row + 16 * target ----
    const int nx = min(R.Tc, wn.x - wn.y - nwt);
    if (nx <= 0) return;
    int* dirty = R.dirty + (size_t)s * NB + band;
    if (!(any || ((*dirty >> quarter) & 1))) return;
    const int* pn = pd + nwt;
    for (int t0 = 16 * wave; t0 < nx; t0 += 16 * kWaves) {
        uint64_t v[4];
        int kk[4], aa[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            kk[u] = pn[min(t0 + 4 * u + lane / kApplyRows, nx - 1)];
            aa[u] = tq[kk[u]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = tb[(size_t)(lane & (kApplyRows - 1)) * RS + (aa[u] >> 6)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t m = __ballot((v[u] >> (aa[u] & 63)) & 1ull);
            if ((lane & (kApplyRows - 1)) == 0 && t0 + 4 * u + lane / kApplyRows < nx)
                X[4 * (size_t)kk[u]] = (uint16_t)(m >> lane);
        }
    }
    if (any && tid == 0) atomicOr(dirty, 1 << quarter);
}

}  // namespace stabdev
