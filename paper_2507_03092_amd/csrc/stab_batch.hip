// stab_batch.hip -- uneven multi-circuit batching: many independent circuits of different
// sizes, each with its own tableau and its own op stream, run by ONE persistent launch.
//
// One block per circuit executes that circuit's whole program: runs of gate and noise layers
// as band passes (64 rows staged in LDS and turned into qubit-major words, every layer of
// the run applied there, written back once), and measurement instructions with the results of
// Sec. 2.4 target by target (pivot = first stabilizer row with x at the qubit, rowsum from it
// (Appendix A.2) for a random outcome, the product of the selected stabilizer rows for a
// deterministic one), random targets of an instruction in windows whose rows are read and written
// once (batch_window).  Blocks are dispatched largest circuit first so the long ones start early.
//
// Randomness: Philox4x64-10 with key (seed, circuit index), counter (instruction index in the
// circuit's stream, target position), the index counting every instruction the circuit has
// executed since the batch was created or reset: circuit c draws exactly what a one-shot
// context with first_shot = c draws for the same sequence of streams.
//
// Included by stab_api.hip (same translation unit: it shares the device helpers above).

namespace stabdev {

// Largest circuit of a batch: a lane owns at most two x words and two z words of a row.
constexpr int kBatchMaxWc = 128;
// The kernel comes in two widths, BW = 8 waves (two blocks share a compute unit) and 16 (one block
// has it alone): batch_waves().
constexpr int kBatchWavesMax = 16;

struct BatchCirc {
    int n, Wc, RS, NR;          // NR = 64 * Wc rows per half; RS = 2 * Wc words per row
    long long tab_off;          // first word of the tableau [2*NR][RS]
    long long rs_off;           // first word of the sign vector [2*Wc]
    int step_begin, step_count; // program steps
    long long rec_bit_off;      // bit offset of the circuit's first record in the output
    long long col_off;          // first word of the column scratch [2][NB][col_k] (if col_k > 0)
    int col_k;                  // targets the scratch holds per band (0: no scratch)
};

struct BatchMeas {
    uint64_t instr;  // instruction index in the circuit's stream
    uint64_t t0, t1; // T1T2 thresholds: reset iff u0 < t0, else Z iff u0 < t1
    int kind;        // M, MR, R or T1T2
    int tq;          // first target in the measurement target array
    int K;           // targets
    int rec;         // record index (within the circuit) of the first target; -1 if none
    int fast;        // distinct qubits: its columns can be extracted in the band pass before it
};

// Program step: (0, first gate, gates, modifies x|z) gate layer on disjoint qubits;
// (1, noise descriptor, 0, 0) noise layer; (2, measurement descriptor, 0, 0).
struct BatchArgs {
    const BatchCirc* circ;
    const int* order;           // block -> circuit
    const int4* steps;
    const uint2* gates;
    const NoiseDesc* noise;
    const int* noise_tg;
    const BatchMeas* meas;
    const int* meas_tg;
    uint64_t* tab;
    uint64_t* rs;
    uint32_t* rec;              // packed record bits, zeroed before the launch
    uint64_t* cols;             // base of the circuits' column scratch
    const uint64_t* ibase;      // per circuit: instructions it executed before this launch
    const ulonglong2* keys;     // per circuit RNG key, or NULL for (seed, circuit index)
    int meas_quota;             // stop a circuit after this many measurement steps (0: run all)
    int tile;                   // launch configuration (kTileWholeWave and rows in flight)
    int lds_words;              // LDS of a block
    uint64_t seed;
    int* err;
    unsigned long long* counters;
};

// The kernel's parts are functions of their own (not inlined): together their registers made the
// whole kernel spill.  They take the arguments by the kernel argument segment's address, which
// keeps them in scalar registers, and LDS by its address.
typedef const __attribute__((address_space(4))) BatchArgs* ArgsPtr;
typedef __attribute__((address_space(3))) void* LdsPtr;

#define kNoSel ((LdsPtr)(uint32_t)-1)

// A part of the kernel.  not_tail_called: with a call that the compiler marks as a tail call the callee
// saves the registers it uses (44 of a thread's 128 for a band pass: 90 KB a block to memory and back
// a call), any other call leaves that to the caller, which holds next to nothing.  A launch of 300
// circuits of 64 qubits, ten gate layers each, 37.4 -> 32.5 us; 300 shots of a T1/T2 memory of 49 qubits
// 1.02 -> 0.93 ms.
#define BATCH_CALL __noinline__ __attribute__((not_tail_called))

__device__ __forceinline__ BatchArgs uniform_args(ArgsPtr p)
{
    return *(const BatchArgs*)(ArgsPtr)uni64((uint64_t)(uintptr_t)p);
}

__device__ __forceinline__ BatchCirc uniform_circ(const BatchCirc* c)
{
    BatchCirc C = *c;
    C.n = uni(C.n);
    C.Wc = uni(C.Wc);
    C.RS = uni(C.RS);
    C.NR = uni(C.NR);
    C.tab_off = (long long)uni64((uint64_t)C.tab_off);
    C.rs_off = (long long)uni64((uint64_t)C.rs_off);
    C.rec_bit_off = (long long)uni64((uint64_t)C.rec_bit_off);
    C.col_off = (long long)uni64((uint64_t)C.col_off);
    C.step_begin = uni(C.step_begin);
    C.step_count = uni(C.step_count);
    C.col_k = uni(C.col_k);
    return C;
}

__device__ __forceinline__ BatchMeas uniform_meas(const BatchMeas* m)
{
    BatchMeas M = *m;
    M.instr = uni64(M.instr);
    M.t0 = uni64(M.t0);
    M.t1 = uni64(M.t1);
    M.kind = uni(M.kind);
    M.tq = uni(M.tq);
    M.K = uni(M.K);
    M.rec = uni(M.rec);
    M.fast = uni(M.fast);
    return M;
}

// Random-at-start targets of an instruction taken at a time (batch_window): 64, or 32 where the
// products of their pivot rows would not fit in LDS.
__host__ __device__ constexpr int batch_win(int Wc) { return Wc <= 64 ? 64 : 32; }

// LDS of a measurement instruction, in words (uint64): kept parts, then a region shared by the
// window's row masks and list, its pivot products (three per pair of targets and a row of zeros),
// the slow form's buffers and, up to 4096 qubits, the band tile of an extraction pass.
struct BatchLds {
    int outb, rndb, evb, rlist, sel, own, chunk, tabs, wave, region, total;
};

// Noise steps and events of a run of gate and noise layers that are listed behind the band tile.
constexpr int kBatchNoiseSteps = 30, kBatchNoiseEvents = 512;
constexpr int kBatchSteps = 64;                  // steps of a run kept beside them
// bands of a pass in LDS at once, at most
constexpr int kBatchBands = 4;
__host__ __device__ constexpr int batch_tile_words(int RS, int bands = 1)
{
    return bands * 64 * (RS + 1) + RS + 2 + 4 * kBatchSteps / 2 + (kBatchNoiseSteps + 2 + kBatchNoiseEvents) / 2;
}

constexpr int kBatchChunkWords = (sizeof(ChunkLds) + 7) / 8;
// unit, hit and column tables (256 words each), exponent table (256 bytes), column rows (64 words),
// the window's targets, pivots and exponents (3 x 64 ints), 32 ints of scratch
constexpr int kBatchTabWords = 3 * 256 + 32 + 64 + 96 + 16;
constexpr int kBatchWaveWords = 64 + 16 + 8;     // per wave: masks, rows and exponents of a band's changed rows

__host__ __device__ inline BatchLds batch_lds(int Wc, int BW)
{
    const int RS = 2 * Wc, NB = 2 * Wc;
    BatchLds L;
    int o = NB;                                   // sign words first
    L.outb = o; o += Wc;
    L.rndb = o; o += Wc;
    L.evb = o; o += Wc;
    L.rlist = o; o += 16 * Wc;                    // (uint16, 64 Wc)
    L.sel = o; o += Wc <= 64 ? 16 * Wc : 0;       // (T1T2 events take the fast form up to 4096 qubits)
    L.own = o; o += 8 * Wc;                       // (int8, a row pair each)
    L.chunk = o; o += kBatchChunkWords;
    L.tabs = o; o += kBatchTabWords;
    L.wave = o; o += BW * kBatchWaveWords;
    o = (o + 1) & ~1;
    L.region = o;
    const int plan = 64 * Wc + 16 * Wc;           // masks, list (uint16)
    const int prod = (batch_win(Wc) / 2 * 3 + 1) * RS;
    const int slow = NB + RS + 2 * BW * RS + 16 + NB * 64 * 2 / 8;
    const int tile = Wc <= 64 ? batch_tile_words(RS) : 0;
    int r = plan > prod ? plan : prod;
    r = r > slow ? r : slow;
    r = r > tile ? r : tile;
    L.total = o + r;
    return L;
}

// LDS words the batch kernel needs for circuits with up to Wc column words (one with 64 needs more
// than one with a few more, whose windows are smaller).
__host__ __device__ inline int batch_lds_words(int Wc, int BW)
{
    const int seg = batch_tile_words(2 * Wc), meas = batch_lds(Wc, BW).total;
    const int m64 = Wc > 64 ? batch_lds(64, BW).total : 0;
    const int m = meas > m64 ? meas : m64;
    return seg > m ? seg : m;
}

constexpr int kMK = 7, kMRK = 8, kRK = 9, kT1T2K = 13;   // kinds (include/stab.h enum)
// A measurement instruction with at least this many targets gets an extraction-only band
// pass when no gate pass precedes it.
constexpr int kBatchExtractMin = 8;
// An instruction on a single target of a circuit of at most so many words takes the slow form, whose
// steps are fewer (200 circuits of 64 qubits, one target an instruction, 109 us fast and 97 slow; two
// targets, if they are not random, 109 and 125).
constexpr int kBatchSlowWc = 4;

__device__ __forceinline__ ulonglong2 batch_key(const BatchArgs& A, int ci)
{
    if (A.keys) return A.keys[ci];
    ulonglong2 k;
    k.x = A.seed;
    k.y = (uint64_t)ci;
    return k;
}

// -------------------------------------------------------------------------------- gates ---
__device__ __forceinline__ void batch_gate(uint64_t* T, int RSP, int Wc, uint2 gt, uint64_t& racc)
{
    const int kind = (int)(gt.x & 15u);
    const int q0 = (int)(gt.x >> 4);
    const int i0 = (q0 & 63) * RSP + (q0 >> 6);
    const uint64_t x0 = T[i0], z0 = T[i0 + Wc];
    switch (kind) {
    case STAB_KIND_H:
        racc ^= x0 & z0;
        T[i0] = z0;
        T[i0 + Wc] = x0;
        break;
    case STAB_KIND_S:
        racc ^= x0 & z0;
        T[i0 + Wc] = z0 ^ x0;
        break;
    case STAB_KIND_X: racc ^= z0; break;
    case STAB_KIND_Y: racc ^= x0 ^ z0; break;
    case STAB_KIND_Z: racc ^= x0; break;
    case STAB_KIND_CX: {
        const int q1 = (int)gt.y;
        const int i1 = (q1 & 63) * RSP + (q1 >> 6);
        const uint64_t x1 = T[i1], z1 = T[i1 + Wc];
        racc ^= x0 & z1 & ~(x1 ^ z0);
        T[i1] = x1 ^ x0;
        T[i0 + Wc] = z0 ^ z1;
    } break;
    default: break;
    }
}

// Noise unit u of descriptor d for circuit ci: f(qubit, Pauli) for each error it draws.
template <class F>
__device__ __forceinline__ void batch_noise(const NoiseDesc& d, const int* __restrict__ ntg, int u, ulonglong2 key,
                                            uint64_t ibase, F f)
{
    uint64_t u0, u1;
    philox(ibase + d.instr, (uint64_t)u, key.x, key.y, u0, u1);
    if (d.kind == STAB_KIND_DEP1) {
        if (u0 < d.t0) f(ntg[d.toff + u], 1 + (int)__umul64hi(u1, 3ull));
    } else if (d.kind == STAB_KIND_DEP2) {
        if (u0 < d.t0) {
            const int k = 1 + (int)__umul64hi(u1, 15ull);
            if (k >> 2) f(ntg[d.toff + 2 * u], k >> 2);
            if (k & 3) f(ntg[d.toff + 2 * u + 1], k & 3);
        }
    } else {
        const int p = (u0 < d.t0) ? 1 : (u0 < d.t1) ? 2 : (u0 < d.t2) ? 3 : 0;
        if (p) f(ntg[d.toff + u], p);
    }
}

// A list filled step by step by a whole block: append(i) adds step i's entries at slots counted up in
// *count, and off[i + 1] becomes the end of step i's.  The end is read between two barriers: without
// the second, a thread already in step i + 1 could count entries of its own into step i's.
template <class Append, class Barrier>
__host__ __device__ __forceinline__ void list_by_step(int nsteps, int tid, int* off, const int* count, Append append,
                                                      Barrier barrier)
{
    for (int i = 0; i < nsteps; ++i) {
        append(i);
        barrier();
        if (tid == 0) off[i + 1] = *count;
        barrier();
    }
}

// One run of gate/noise steps [st, en) over every band of the circuit.
// With ncol > 0, the band pass also writes the x and z columns of targets tq[sel[k]] (tq[k] with sel
// = kNoSel; tq: their start in the target array), k < ncol, 64 rows per word, to the circuit's
// column scratch, [band][k].
//
// The run's noise is drawn once, into a list of events behind the tile (a run with more steps or
// errors than it holds draws again for every band).  Up to kBatchBands bands are taken at once, as
// many as fit: a pass is seven barrier-separated steps of a few LDS round trips each, so it is bound
// by latency (64 % of wave time waits, VALU 37 % busy), and four bands share its steps: 1024 circuits
// of 64 to 2048 qubits 22.1 -> 19.9 ms, 100 shots of a 1249-qubit circuit 48.9 -> 47.9 ms.  Their rows
// are loaded while the bands before them are worked on, and zero 64x64 tiles, their own transposes,
// are left alone.
template <int BW>
__device__ BATCH_CALL void batch_segment(ArgsPtr ap, int ci_, int st_, int en_, LdsPtr lds_, int tq_, LdsPtr sel_,
                                         int ncol_)
{
    constexpr int nt = (64 * BW), PF = 4;      // 16-byte pairs a thread loads ahead
    const BatchArgs A = uniform_args(ap);
    const int ci = uni(ci_), st = uni(st_), en = uni(en_), ncol = uni(ncol_);
    const BatchCirc C = uniform_circ(A.circ + ci);
    extern __shared__ uint64_t lds_all[];
    uint64_t* lds = (uint64_t*)lds_;
    const int* tq = A.meas_tg + uni(tq_);
    const uint16_t* sel = (const uint16_t*)sel_;
    const bool has_sel = uni((int)(uint32_t)(uintptr_t)sel_) != -1;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int RS = C.RS, RSP = C.RS + 1, Wc = C.Wc, NB = 2 * C.Wc;
    uint64_t* T = lds;
    const int room = A.lds_words - (int)(((uint32_t)(uintptr_t)lds_ - (uint32_t)(uintptr_t)(LdsPtr)lds_all) / 8);
    int nbd = 1;                                   // bands at once
    while (nbd < kBatchBands && nbd < NB && batch_tile_words(RS, nbd + 1) <= room) ++nbd;
    nbd = uni(nbd);
    uint64_t* sacc = lds + nbd * 64 * RSP;         // sign flips per band
    // (an index, not an aligned address: that would make its accesses flat ones, which wait for every
    // load in flight: 45.7 -> 44.5 ms for 100 shots of the 1249-qubit circuit)
    int4* steps = (int4*)(lds + ((nbd * 64 * RSP + NB + 1) & ~1));
    int* off = (int*)(steps + kBatchSteps);        // noise step i's events: [off[i], off[i + 1])
    uint32_t* evs = (uint32_t*)off + kBatchNoiseSteps + 2;
    uint64_t* tab = A.tab + C.tab_off;
    uint64_t* rs = A.rs + C.rs_off;
    const ulonglong2 key = batch_key(A, ci);
    const uint64_t ibase = A.ibase[ci];
    int wb = 0, nn = 0, g0 = -1;                   // g0: the first gate layer
    for (int k = st; k < en; ++k) {
        const int4 s = A.steps[k];
        wb |= s.x == 0 ? s.w : 0;
        nn += s.x != 0;
        if (s.x == 0 && g0 < 0) g0 = k;
    }
    wb = uni(wb);
    nn = uni(nn);
    g0 = uni(g0);
    for (int w = tid; w < NB; w += nt) sacc[w] = 0ull;
    for (int k = tid; k < min(en - st, kBatchSteps); k += nt) steps[k] = A.steps[st + k];
    auto step_at = [&](int k) {
        const int4 s = k - st < kBatchSteps ? steps[k - st] : A.steps[k];
        return make_int4(uni(s.x), uni(s.y), uni(s.z), 0);
    };
    // the first gate layer's gates and the extracted columns' tile words stay in registers for
    // all bands, a later layer's gates are loaded while the one before is applied
    constexpr int GP = 2, XP = 3;
    uint2 gfirst[GP], gnext[GP];
    int xq[XP];
    auto gate_fetch = [&](int k, uint2* g) {
        const int4 s = A.steps[k];
#pragma unroll
        for (int u = 0; u < GP; ++u)
            if (tid + u * nt < s.z) g[u] = A.gates[s.y + tid + u * nt];
    };
    if (g0 >= 0) gate_fetch(g0, gfirst);
#pragma unroll
    for (int u = 0; u < XP; ++u) {
        const int k = tid + u * nt;
        const int q = k < ncol ? tq[has_sel ? (int)sel[k] : k] : 0;
        xq[u] = (q & 63) * RSP + (q >> 6);
    }
    __syncthreads();
    bool listed = nn > 0 && nn <= kBatchNoiseSteps;
    if (listed) {
        int* nev = off + kBatchNoiseSteps + 1;
        if (tid == 0) off[0] = *nev = 0;
        __syncthreads();
        int k = st;
        list_by_step(
            nn, tid, off, nev,
            [&](int) {
                while (A.steps[k].x == 0) ++k;
                const NoiseDesc d = A.noise[A.steps[k++].y];
                for (int u = tid; u < d.units; u += nt)
                    batch_noise(d, A.noise_tg, u, key, ibase, [&](int q, int P) {
                        const int e = atomicAdd(nev, 1);
                        if (e < kBatchNoiseEvents) evs[e] = (uint32_t)((q & 63) * RSP + (q >> 6)) | (uint32_t)P << 28;
                    });
            },
            [] { __syncthreads(); });
        listed = uni(off[nn]) <= kBatchNoiseEvents;
    }
    const int TS = 64 * RSP;                       // words between the bands' tiles
    auto flips = [&](const uint64_t* Tb, int iq, int P) {
        const uint64_t xq = Tb[iq], zq = Tb[iq + Wc];
        return P == 1 ? zq : P == 3 ? xq : (xq ^ zq);
    };
    const int npairs = 32 * RS;
    ulonglong2 pf[PF];
    auto fetch = [&](int band, int np) {
        const ulonglong2* gb2 = (const ulonglong2*)(tab + (size_t)band * 64 * RS);
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int p = u * nt + tid;
            if (p < np) pf[u] = gb2[p];
        }
    };
    // (row r of the pass's bands, pair of words from column c on: the rows of a tile follow each other)
    auto slot = [&](int p) {
        const int i = 2 * p;
        const int r = i / RS;
        return r * RSP + (i - r * RS);
    };
    int at[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u) at[u] = slot(u * nt + tid);
    auto transpose = [&](int nb) {
        for (int id = wave; id < nb * RS; id += 2 * BW) {
            const int id2 = id + BW;
            const int b0 = id / RS, b1 = id2 / RS;
            uint64_t* p0 = T + b0 * TS + lane * RSP + (id - b0 * RS);
            uint64_t* p1 = T + b1 * TS + lane * RSP + (id2 - b1 * RS);
            const uint64_t a = *p0, b = id2 < nb * RS ? *p1 : 0ull;
            if (__ballot(a != 0ull)) *p0 = transpose64_dpp(a, lane);
            if (__ballot(b != 0ull)) *p1 = transpose64_dpp(b, lane);
        }
    };
    fetch(0, min(nbd, NB) * npairs);
    for (int band = 0; band < NB; band += nbd) {
        const int nb = min(nbd, NB - band), np = nb * npairs;
        uint64_t* gb = tab + (size_t)band * 64 * RS;
#pragma unroll
        for (int u = 0; u < PF; ++u)
            if (u * nt + tid < np) {
                T[at[u]] = pf[u].x;
                T[at[u] + 1] = pf[u].y;
            }
        for (int p0 = PF * nt; p0 < np; p0 += 4 * nt) {
            ulonglong2 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * nt + tid;
                if (p < np) v[u] = ((const ulonglong2*)gb)[p];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * nt + tid;
                if (p < np) {
                    const int a = slot(p);
                    T[a] = v[u].x;
                    T[a + 1] = v[u].y;
                }
            }
        }
        lds_barrier();
        if (band + nbd < NB) fetch(band + nbd, min(nbd, NB - band - nbd) * npairs);
        transpose(nb);
        lds_barrier();
        uint64_t racc[kBatchBands];
#pragma unroll
        for (int b = 0; b < kBatchBands; ++b) racc[b] = 0ull;
        for (int k = st, i = 0; k < en; ++k) {
            const int4 s = step_at(k);
            const bool gate_next = k + 1 < en && step_at(k + 1).x == 0;
            if (s.x == 0) {
                // (a layer right before another hands its successor's gates over; after a noise
                // layer they are loaded here)
                uint2 g[GP];
#pragma unroll
                for (int u = 0; u < GP; ++u) g[u] = k == g0 ? gfirst[u] : gnext[u];
                if (k != g0 && !(k > st && step_at(k - 1).x == 0)) gate_fetch(k, g);
                if (gate_next) gate_fetch(k + 1, gnext);
#pragma unroll
                for (int b = 0; b < kBatchBands; ++b) {
                    if (b >= nb) break;
#pragma unroll
                    for (int u = 0; u < GP; ++u)
                        if (tid + u * nt < s.z) batch_gate(T + b * TS, RSP, Wc, g[u], racc[b]);
                    for (int gi = tid + GP * nt; gi < s.z; gi += nt)
                        batch_gate(T + b * TS, RSP, Wc, A.gates[s.y + gi], racc[b]);
                }
                lds_barrier();
            } else {
                if (listed) {
                    const int e0 = off[i], e1 = off[i + 1];
                    for (int e = e0 + tid; e < e1; e += nt) {
                        const uint32_t v = evs[e];
#pragma unroll
                        for (int b = 0; b < kBatchBands; ++b)
                            if (b < nb) racc[b] ^= flips(T + b * TS, (int)(v & 0x0FFFFFFFu), (int)(v >> 28));
                    }
                } else {
                    const NoiseDesc d = A.noise[s.y];
                    for (int u = tid; u < d.units; u += nt)
                        batch_noise(d, A.noise_tg, u, key, ibase, [&](int q, int P) {
#pragma unroll
                            for (int b = 0; b < kBatchBands; ++b)
                                if (b < nb) racc[b] ^= flips(T + b * TS, (q & 63) * RSP + (q >> 6), P);
                        });
                }
                ++i;
                if (gate_next) lds_barrier();         // (noise only reads the tile)
            }
        }
        if (ncol > 0) {
            for (int b = 0; b < nb; ++b) {
                const uint64_t* Tb = T + b * TS;
                uint64_t* Xs = A.cols + C.col_off + (size_t)(band + b) * C.col_k;
                uint64_t* Zs = Xs + (size_t)NB * C.col_k;
#pragma unroll
                for (int u = 0; u < XP; ++u)
                    if (tid + u * nt < ncol) {
                        Xs[tid + u * nt] = Tb[xq[u]];
                        Zs[tid + u * nt] = Tb[xq[u] + Wc];
                    }
                for (int k = tid + XP * nt; k < ncol; k += nt) {
                    const int q = tq[has_sel ? (int)sel[k] : k];
                    const int iq = (q & 63) * RSP + (q >> 6);
                    Xs[k] = Tb[iq];
                    Zs[k] = Tb[iq + Wc];
                }
            }
        }
        if (wb) {
            lds_barrier();      // the transpose back rewrites the tile
            transpose(nb);
            lds_barrier();
            ulonglong2* gw2 = (ulonglong2*)gb;
            for (int p = tid, u = 0; p < np; p += nt, ++u) {
                const int a = slot(p);
                ulonglong2 v;
                v.x = T[a];
                v.y = T[a + 1];
                gw2[p] = v;
            }
        }
#pragma unroll
        for (int b = 0; b < kBatchBands; ++b)
            if (b < nb && __ballot(racc[b] != 0ull)) {
                const uint64_t v = wave_xor(racc[b]);
                if (lane == 0) atomicXor((unsigned long long*)&sacc[band + b], (unsigned long long)v);
            }
        lds_barrier();          // the next bands reuse the tile
    }
    __syncthreads();
    for (int w = tid; w < NB; w += nt)
        if (sacc[w]) rs[w] ^= sacc[w];
    __syncthreads();
    if (tid == 0) count_add(A.counters, 7, (unsigned long long)NB * 64 * RS * 8 * (wb ? 2 : 1));
}

// -------------------------------------------------------------------------- measurement ---
// Bit `bit` of word `word` of every row, as 64-row words (one per band), into out[0..NB).
// With xor_into set the words are XORed into out (used to flip signs) instead of stored.
template <int BW>
__device__ __forceinline__ void batch_column(const uint64_t* __restrict__ tab, int RS, int NB,
                                             int word, int bit, uint64_t* out, bool xor_into)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c0 = wave; c0 < NB; c0 += 4 * BW) {
        uint64_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * BW;
            v[u] = (c < NB) ? tab[(size_t)(64 * c + lane) * RS + word] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * BW;
            const uint64_t m = __ballot((v[u] >> bit) & 1ull);
            if (c < NB && lane == 0) {
                if (xor_into) out[c] ^= m;
                else out[c] = m;
            }
        }
    }
}

// Rows whose bit is set in words [w0, w1) of bits, minus `skip` rows, listed in row order into
// list (uint16) -- block-wide; returns the count (valid in every thread after the call).
template <int BW>
__device__ int batch_list(const uint64_t* bits, int w0, int w1, int skip0, int skip1,
                          uint16_t* list, int* s_tot)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int* wtot = s_tot + 1;
    int total = 0;
    for (int base = w0; base < w1; base += (64 * BW)) {
        const int w = base + tid;
        uint64_t m = 0;
        if (w < w1) {
            m = bits[w];
            if ((skip0 >> 6) == w) m &= ~(1ull << (skip0 & 63));
            if ((skip1 >> 6) == w) m &= ~(1ull << (skip1 & 63));
        }
        const int c = __popcll(m);
        const int ex = wave_excl_scan(c, lane);
        if (lane == 63) wtot[wave] = ex + c;
        __syncthreads();
        int off = total;
        for (int v = 0; v < wave; ++v) off += wtot[v];
        int t = 0;
        for (int v = 0; v < BW; ++v) t += wtot[v];
        off += ex;
        while (m) {
            list[off++] = (uint16_t)(64 * w + ctz64(m));
            m &= m - 1;
        }
        total += t;
        __syncthreads();
    }
    return total;
}

// Launch configuration of the batch kernel (BatchArgs::tile): bits 0-7 rows each lane group
// keeps in flight in a rowsum (2, 4 or 8, at most 4 with two x words per lane; 0 = 8 for one
// x word per lane, 2 for two); bit 8
// set: every row takes the whole wave (64 lanes per row), clear: a row takes the smallest
// power of two of lanes that covers its x words, so a wave updates 64 / lanes rows per load.
constexpr int kTileWholeWave = 1 << 8;
// bit 9 set: 16 waves a block, one block per compute unit; clear: 8 waves, two blocks.
constexpr int kTileOneBlock = 1 << 9;

// rowsum(row, p) for every listed row: x|z ^= pivot, sign from the g-sum (Appendix A.2).
// A row is owned by a group of lpr lanes (lane sub of the group holds x words sub,
// sub + lpr, ..., NW of them, and the matching z words); a wave holds 64 / lpr groups and
// each group keeps R rows in flight so their loads overlap.  The g-sums are reduced within
// the group, eight bits per row, four rows per int.
template <int NW, int R, int BW>
__device__ void batch_rowsum_tile(const BatchCirc& C, uint64_t* __restrict__ tab, const uint64_t* prow,
                                  int rp, const uint16_t* list, int nlist, uint64_t* sg, int* err, int lpr)
{
    static_assert(R <= 8, "two packed ints hold eight rows");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int Wc = C.Wc, RS = C.RS;
    const int sub = lane & (lpr - 1), grp = lane / lpr, groups = 64 / lpr;
    uint64_t px[NW], pz[NW];
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        const int j = sub + lpr * t;
        px[t] = (j < Wc) ? prow[j] : 0;
        pz[t] = (j < Wc) ? prow[Wc + j] : 0;
    }
    const int step = R * groups;
    for (int base = wave * step; base < nlist; base += BW * step) {
        uint64_t x[R][NW], z[R][NW];
        int row[R];
        bool ok[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int li = base + r * groups + grp;
            ok[r] = li < nlist;
            row[r] = ok[r] ? (int)list[li] : 0;
#pragma unroll
            for (int t = 0; t < NW; ++t) {
                const int j = sub + lpr * t;
                x[r][t] = z[r][t] = 0;
                if (ok[r] && j < Wc) {
                    x[r][t] = tab[(size_t)row[r] * RS + j];
                    z[r][t] = tab[(size_t)row[r] * RS + Wc + j];
                }
            }
        }
        int pk[2] = {0, 0};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int G = 0;
#pragma unroll
            for (int t = 0; t < NW; ++t) G += gsum(px[t], pz[t], x[r][t], z[r][t]);
            pk[r >> 2] += (G & 3) << (8 * (r & 3));
        }
        // at most 64 lanes add at most 3 each: the 8-bit fields do not carry
        for (int m = lpr >> 1; m >= 1; m >>= 1) {
            pk[0] += __shfl_xor(pk[0], m, 64);
            if (R > 4) pk[1] += __shfl_xor(pk[1], m, 64);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (ok[r]) {
#pragma unroll
                for (int t = 0; t < NW; ++t) {
                    const int j = sub + lpr * t;
                    if (j < Wc) {
                        tab[(size_t)row[r] * RS + j] = x[r][t] ^ px[t];
                        tab[(size_t)row[r] * RS + Wc + j] = z[r][t] ^ pz[t];
                    }
                }
                if (sub == 0) {
                    const int G = (pk[r >> 2] >> (8 * (r & 3))) & 3;
                    const int ri = (int)((sg[row[r] >> 6] >> (row[r] & 63)) & 1ull);
                    const int e = (2 * ri + 2 * rp + G) & 3;
                    if (e & 1) atomicOr(err, 1);
                    if ((e >> 1) != ri) atomicXor((unsigned long long*)&sg[row[r] >> 6], 1ull << (row[r] & 63));
                }
            }
        }
    }
}

template <int NW, int BW>
__device__ void batch_rowsum(const BatchCirc& C, uint64_t* __restrict__ tab, const uint64_t* prow, int rp,
                             const uint16_t* list, int nlist, uint64_t* sg, int* err, int tile)
{
    int lpr = 64;
    if (!(tile & kTileWholeWave))
        while (lpr > 1 && (lpr >> 1) >= C.Wc) lpr >>= 1;
    const int R = tile & 0xff;
    // two x words per lane: at most 4 rows in flight (register budget)
    if ((R == 8 || R == 0) && NW == 1) batch_rowsum_tile<NW, 8, BW>(C, tab, prow, rp, list, nlist, sg, err, lpr);
    else if (R == 2 || (R == 0 && NW == 2)) batch_rowsum_tile<NW, 2, BW>(C, tab, prow, rp, list, nlist, sg, err, lpr);
    else batch_rowsum_tile<NW, 4, BW>(C, tab, prow, rp, list, nlist, sg, err, lpr);
}

// Sign of the product of the listed stabilizer rows (destabilizer indices i -> row NR + i):
// for Paulis P_k = (-1)^r_k i^|x_k & z_k| X^x_k Z^z_k the product carries
// i^(sum_k (2 r_k + |x_k & z_k|) + 2 sum_{i<k} z_i . x_k); the rows commute, so waves reduce
// contiguous chunks and the cross terms between chunks are added from their (X, Z) parities.
// The result must be +-Z (X = 0 and an even exponent), else *err is set.  Block-wide.
template <int NW, int BW>
__device__ int batch_det(const BatchCirc& C, const uint64_t* __restrict__ tab, const uint16_t* list,
                         int nlist, const uint64_t* sg, uint64_t* part, int* s_res, int* err)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int Wc = C.Wc, RS = C.RS, NR = C.NR;
    const int per = (nlist + BW - 1) / BW;
    const int b0 = min(nlist, wave * per), b1 = min(nlist, b0 + per);
    uint64_t X[NW], Z[NW];
#pragma unroll
    for (int t = 0; t < NW; ++t) X[t] = Z[t] = 0;
    int e = 0, cross = 0;
    for (int c0 = b0; c0 < b1; c0 += 4) {
        uint64_t x[4][NW], z[4][NW];
        int ii[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            ii[r] = (c0 + r < b1) ? (int)list[c0 + r] : -1;
#pragma unroll
            for (int t = 0; t < NW; ++t) {
                const int j = lane + 64 * t;
                x[r][t] = z[r][t] = 0;
                if (ii[r] >= 0 && j < Wc) {
                    x[r][t] = tab[(size_t)(NR + ii[r]) * RS + j];
                    z[r][t] = tab[(size_t)(NR + ii[r]) * RS + Wc + j];
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int t = 0; t < NW; ++t) {
                e += __popcll(x[r][t] & z[r][t]);
                cross += __popcll(Z[t] & x[r][t]);
                X[t] ^= x[r][t];
                Z[t] ^= z[r][t];
            }
            if (ii[r] >= 0 && lane == 0) e += 2 * (int)((sg[(NR + ii[r]) >> 6] >> ((NR + ii[r]) & 63)) & 1ull);
        }
    }
    // chunk parities for the cross terms between waves
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        const int j = lane + 64 * t;
        if (j < Wc) {
            part[(2 * wave) * Wc + j] = X[t];
            part[(2 * wave + 1) * Wc + j] = Z[t];
        }
    }
    int v = wave_sum((e & 3) + 2 * (cross & 1));
    if (lane == 0) s_res[1 + wave] = v;
    __syncthreads();
    if (wave == 0) {
        int cr = 0;
        uint64_t xall = 0;
#pragma unroll
        for (int t = 0; t < NW; ++t) {
            const int j = lane + 64 * t;
            if (j < Wc) {
                uint64_t zp = 0, xa = 0;
                for (int w = 0; w < BW; ++w) {
                    const uint64_t xw = part[(2 * w) * Wc + j];
                    cr += __popcll(zp & xw);
                    zp ^= part[(2 * w + 1) * Wc + j];
                    xa ^= xw;
                }
                xall |= xa;
            }
        }
        cr = wave_sum(cr & 1);
        xall = wave_or(xall);
        if (lane == 0) {
            int tot = 2 * cr;
            for (int w = 0; w < BW; ++w) tot += s_res[1 + w];
            tot &= 3;
            if ((tot & 1) || xall) atomicOr(err, 1);
            s_res[0] = tot >> 1;
        }
    }
    __syncthreads();
    return s_res[0];
}

// LDS of a measurement instruction (batch_lds).
struct MeasLds {
    uint64_t* sg;      // NB sign words
    uint64_t* outb;    // outcome bits of the instruction's targets
    uint64_t* rndb;    // random-at-start bits
    uint64_t* evb;     // T1T2: the resets' random outcomes
    uint16_t* rlist;   // the random-at-start targets in op order
    uint16_t* sel;     // T1T2: positions of the events, resets first
    int8_t* own;       // row pair -> the window's target whose pivot it is, -1
    ChunkLds* chunk;
    uint64_t *u4, *h4, *x4;    // by nibble of a mask: units, hits, columns of later targets
    uint8_t* g4;       // exponents of the products
    uint64_t* xr;      // x bits of the pivots at 64 later targets
    int *tk, *tp, *tc; // the window's targets: index in the instruction, pivot row, exponent
    uint64_t* we;      // this wave's changed rows: masks,
    uint16_t* wr;      //   rows,
    uint8_t* wg;       //   exponents
    uint64_t* region;
    // slow form (in the region)
    uint64_t* colx;    // NB words: x bit of the target, per row
    uint64_t* prow;    // RS words: pivot row
    uint64_t* part;    // 2 * BW * RS words
    int* s_int;        // 32 ints: pivot, list and det scratch, T1T2 event masks
    uint16_t* list;    // 2 * NR row indices
};

template <int BW>
__device__ __forceinline__ MeasLds meas_lds(const BatchCirc& C, uint64_t* lds)
{
    const int NB = 2 * C.Wc, RS = C.RS;
    const BatchLds B = batch_lds(C.Wc, BW);
    MeasLds L;
    L.sg = lds;
    L.outb = lds + B.outb;
    L.rndb = lds + B.rndb;
    L.evb = lds + B.evb;
    L.rlist = (uint16_t*)(lds + B.rlist);
    L.sel = (uint16_t*)(lds + B.sel);
    L.own = (int8_t*)(lds + B.own);
    L.chunk = (ChunkLds*)(lds + B.chunk);
    L.u4 = lds + B.tabs;
    L.h4 = L.u4 + 256;
    L.x4 = L.h4 + 256;
    L.g4 = (uint8_t*)(L.x4 + 256);
    L.xr = L.x4 + 256 + 32;
    L.tk = (int*)(L.xr + 64);
    L.tp = L.tk + 64;
    L.tc = L.tp + 64;
    L.s_int = L.tc + 64;
    uint64_t* w = lds + B.wave + (threadIdx.x >> 6) * kBatchWaveWords;
    L.we = w;
    L.wr = (uint16_t*)(w + 64);
    L.wg = (uint8_t*)(w + 64 + 16);
    L.region = lds + B.region;
    L.colx = L.region;
    L.prow = L.colx + NB;
    L.part = L.prow + RS;
    L.list = (uint16_t*)(L.part + 2 * BW * RS);
    return L;
}

struct MeasWork {
    int nrand = 0, ndet = 0;
    long long nrows = 0, bytes = 0;
};

// Z measurement of qubit a on the live tableau (block-wide): the x column gathered a word per row,
// pivot search, then rowsum and row moves (random, outcome rand_bit) or the deterministic
// product.
template <int NW, int BW>
__device__ int batch_measure_one(const BatchArgs& A, const BatchCirc& C, int a, int rand_bit, const MeasLds& L,
                                 MeasWork& W)
{
    const int tid = threadIdx.x;
    const int Wc = C.Wc, RS = C.RS, NR = C.NR, NB = 2 * C.Wc;
    uint64_t* tab = A.tab + C.tab_off;
    const long long row_b = (long long)RS * 8;
    const long long col_b = (long long)2 * NR * 8;
    batch_column<BW>(tab, RS, NB, a >> 6, a & 63, L.colx, false);
    __syncthreads();
    // pivot: first stabilizer row with x at a (rows NR + n .. 2NR - 1 are zero padding)
    if (tid < 64) {
        int first = 0x7fffffff;
        for (int w = Wc + tid; w < NB; w += 64)
            if (L.colx[w]) first = min(first, 64 * w + ctz64(L.colx[w]));
        first = wave_min(first);
        if (tid == 0) L.s_int[0] = first;
    }
    __syncthreads();
    const int p = L.s_int[0];
    int outcome;
    if (p != 0x7fffffff) {
        outcome = rand_bit;
        for (int j = tid; j < RS; j += (64 * BW)) L.prow[j] = tab[(size_t)p * RS + j];
        const int rp = (int)((L.sg[p >> 6] >> (p & 63)) & 1ull);
        const int nl = batch_list<BW>(L.colx, 0, NB, p, p - NR, L.list, L.s_int + 1);
        __syncthreads();    // prow staged
        batch_rowsum<NW, BW>(C, tab, L.prow, rp, L.list, nl, L.sg, A.err, A.tile);
        __syncthreads();
        // destabilizer p - NR <- old stabilizer p; stabilizer p <- (-1)^outcome Z_a
        const int d = p - NR;
        for (int j = tid; j < RS; j += (64 * BW)) {
            tab[(size_t)d * RS + j] = L.prow[j];
            tab[(size_t)p * RS + j] = (j == Wc + (a >> 6)) ? (1ull << (a & 63)) : 0ull;
        }
        if (tid == 0) {
            uint64_t wd = L.sg[d >> 6];
            wd = (wd & ~(1ull << (d & 63))) | ((uint64_t)rp << (d & 63));
            L.sg[d >> 6] = wd;
            uint64_t wp = L.sg[p >> 6];
            wp = (wp & ~(1ull << (p & 63))) | ((uint64_t)outcome << (p & 63));
            L.sg[p >> 6] = wp;
        }
        ++W.nrand;
        W.nrows += nl;
        // column, pivot row, rowsum read+write, two row writes
        W.bytes += col_b + row_b + 2 * nl * row_b + 2 * row_b;
    } else {
        const int nl = batch_list<BW>(L.colx, 0, Wc, -1, -1, L.list, L.s_int + 1);
        outcome = batch_det<NW, BW>(C, tab, L.list, nl, L.sg, L.part, L.s_int + 10, A.err);
        ++W.ndet;
        W.nrows += nl;
        W.bytes += col_b + nl * row_b;
    }
    __syncthreads();
    return outcome;
}

// One wave: the outcome of target k of an instruction whose columns are in the scratch, if it
// is deterministic (no stabilizer has x at the qubit); -1 if it is random.  The product of
// the stabilizers selected by the destabilizers with x at the qubit, as in batch_det.
template <int NW>
__device__ int batch_det_from_cols(const BatchArgs& A, const BatchCirc& C, const uint64_t* Xs, int k,
                                   const uint64_t* sg, int& nrows)
{
    const int lane = threadIdx.x & 63;
    const int Wc = C.Wc, RS = C.RS, NR = C.NR, CK = C.col_k;
    const uint64_t* tab = A.tab + C.tab_off;
    // the column, a word of either half per lane (and 64 words on)
    uint64_t cd[NW];
    bool st = false;
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        const int w = lane + 64 * t;
        cd[t] = w < Wc ? Xs[(size_t)w * CK + k] : 0ull;
        st |= w < Wc && Xs[(size_t)(Wc + w) * CK + k] != 0ull;
    }
    if (__ballot(st)) return -1;
    uint64_t X[NW], Z[NW];
#pragma unroll
    for (int t = 0; t < NW; ++t) X[t] = Z[t] = 0;
    int e = 0, cross = 0, rows = 0, nc = 0, mine = 0;
    // the listed rows (lane c holds the c-th), four at a time in flight
    auto flush = [&]() {
        const uint64_t sw = sg[(NR + (lane < nc ? mine : 0)) >> 6];
        e += lane < nc ? 2 * (int)((sw >> (mine & 63)) & 1ull) : 0;
        for (int c = 0; c < nc; c += 4) {
            uint64_t x[4][NW], z[4][NW];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = __builtin_amdgcn_readlane(mine, min(c + u, nc - 1));
                const uint64_t* row = tab + (size_t)(NR + i) * RS;
#pragma unroll
                for (int t = 0; t < NW; ++t) {
                    const int j = lane + 64 * t;
                    const bool in = c + u < nc && j < Wc;
                    x[u][t] = in ? row[j] : 0ull;
                    z[u][t] = in ? row[Wc + j] : 0ull;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < NW; ++t) {
                    e += __popcll(x[u][t] & z[u][t]);
                    cross += __popcll(Z[t] & x[u][t]);
                    X[t] ^= x[u][t];
                    Z[t] ^= z[u][t];
                }
        }
        rows += nc;
        nc = 0;
    };
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        uint64_t lanes = __ballot(cd[t] != 0ull);
        while (lanes) {
            const int l = ctz64(lanes);
            lanes &= lanes - 1;
            uint64_t v = readlane_u64(cd[t], l);
            while (v) {
                const int i = 64 * (l + 64 * t) + ctz64(v);
                v &= v - 1;
                if (lane == nc) mine = i;
                if (++nc == 64) flush();
            }
        }
    }
    if (nc) flush();
    uint64_t xr = 0;
#pragma unroll
    for (int t = 0; t < NW; ++t) xr |= X[t];
    // (without the LDS crossbar: with few rows the reductions are half of it.  300 circuits of 64 qubits,
    // all measured ten times, none random: 312 -> 296 us)
    const int tot = wave_sum_uniform((e & 3) + 2 * (cross & 1), lane) & 3;
    const bool bad = (tot & 1) || __ballot(xr != 0ull);
    if (lane == 0 && bad) atomicOr(A.err, 1);
    nrows += rows;
    return tot >> 1;
}

// The outcomes of n targets whose columns are in the scratch, a wave a target: the instruction's own
// (a random one is marked in L.rndb) or, with listed set, those of L.rlist (whole block).  A part of its
// own, so that its loop has registers to itself.
template <int NW, int BW>
__device__ BATCH_CALL void batch_dets(ArgsPtr ap, int ci_, LdsPtr lds_, int n_, int listed_)
{
    const BatchArgs A = uniform_args(ap);
    const int n = uni(n_), listed = uni(listed_);
    const BatchCirc C = uniform_circ(A.circ + uni(ci_));
    const MeasLds L = meas_lds<BW>(C, (uint64_t*)lds_);
    const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    const uint64_t* Xs = A.cols + C.col_off;
    int nrows = 0, ndet = 0;
    for (int i = wave; i < n; i += BW) {
        const int k = listed ? uni((int)L.rlist[i]) : i;
        const int o = batch_det_from_cols<NW>(A, C, Xs, k, L.sg, nrows);
        if (lane == 0) {
            if (o < 0) atomicOr((unsigned long long*)&L.rndb[k >> 6], 1ull << (k & 63));
            else if (o) atomicOr((unsigned long long*)&L.outb[k >> 6], 1ull << (k & 63));
        }
        if (o >= 0) ++ndet;
    }
    if (lane == 0 && ndet) {
        count_add(A.counters, 2, (unsigned long long)ndet);
        count_add(A.counters, 5, (unsigned long long)nrows);
        count_add(A.counters, 6, (unsigned long long)((long long)ndet * 2 * C.Wc * 8 + (long long)nrows * C.RS * 8));
    }
    __syncthreads();
}

// x and z columns of the listed targets k = list[0 .. n) (qubit tq[sel[k]], or tq[k]) from the live
// rows into the scratch: a word of every row a column, four targets of a band at a time per wave.
// For few targets: a full pass over the bands costs as much as about 60 of them.
constexpr int kBatchGatherMax = 60;

template <int BW>
__device__ void batch_gather(const BatchArgs& A, const BatchCirc& C, const int* tq, const uint16_t* sel,
                             const uint16_t* list, int n)
{
    const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    const int NB = 2 * C.Wc, CK = C.col_k, quads = (n + 3) / 4;
    const uint64_t* tab = A.tab + C.tab_off;
    uint64_t* Xs = A.cols + C.col_off;
    uint64_t* Zs = Xs + (size_t)NB * CK;
    for (int id = wave; id < NB * quads; id += BW) {
        const int band = id / quads, i0 = 4 * (id - band * quads);
        const uint64_t* row = tab + (size_t)(64 * band + lane) * C.RS;
        uint64_t x[4], z[4];
        int k[4], a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u, n - 1);
            k[u] = uni(list ? (int)list[i] : i);
            a[u] = uni(tq[sel ? (int)sel[k[u]] : k[u]]);
            x[u] = row[a[u] >> 6];
            z[u] = row[C.Wc + (a[u] >> 6)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t mx = __ballot((x[u] >> (a[u] & 63)) & 1ull), mz = __ballot((z[u] >> (a[u] & 63)) & 1ull);
            if (lane == 0 && i0 + u < n) {
                Xs[(size_t)band * CK + k[u]] = mx;
                Zs[(size_t)band * CK + k[u]] = mz;
            }
        }
    }
    __syncthreads();
}

// The events of a T1T2 instruction on distinct qubits: L.sel lists the positions of its resets, in
// op order, then of its Zs; L.evb holds the resets' random outcomes.  Draws do not depend on the
// tableau, so they are made before the band pass that extracts the events' columns.  Returns
// {resets, events}.
template <int BW>
__device__ int2 batch_events(const BatchArgs& A, const BatchCirc& C, int ci, const BatchMeas& md, const MeasLds& L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const ulonglong2 key = batch_key(A, ci);
    int* cnt = L.s_int;
    for (int w = tid; w < C.Wc; w += (64 * BW)) L.evb[w] = 0;
    int nres = 0, nz = 0;
    for (int t0 = 0; t0 < md.K; t0 += (64 * BW)) {
        const int t = t0 + tid;
        bool r = false, z = false, o = false;
        if (t < md.K) {
            uint64_t u0, u1;
            philox(A.ibase[ci] + md.instr, (uint64_t)t, key.x, key.y, u0, u1);
            r = u0 < md.t0;
            z = !r && u0 < md.t1;
            o = (u1 >> 63) != 0;
        }
        const uint64_t mr = __ballot(r), mz = __ballot(z);
        __syncthreads();                        // (evb cleared; cnt free)
        if (lane == 0) {
            cnt[wave] = __popcll(mr);
            cnt[16 + wave] = __popcll(mz);
        }
        __syncthreads();
        const int2 cr = wave_counts(cnt, BW, wave, lane), cz = wave_counts(cnt + 16, BW, wave, lane);
        const uint64_t below = (1ull << lane) - 1ull;
        if (r) {
            const int j = nres + cr.x + __popcll(mr & below);
            L.sel[j] = (uint16_t)t;
            if (o) atomicOr((unsigned long long*)&L.evb[j >> 6], 1ull << (j & 63));
        }
        // (Zs wait in rlist)
        if (z) L.rlist[nz + cz.x + __popcll(mz & below)] = (uint16_t)t;
        nres += cr.y;
        nz += cz.y;
    }
    __syncthreads();
    for (int i = tid; i < nz; i += (64 * BW)) L.sel[nres + i] = L.rlist[i];
    __syncthreads();
    return make_int2(nres, nres + nz);
}

// The elimination's two forms.
template <int R, bool BLOCK, int BW>
__device__ BATCH_CALL void batch_steps(LdsPtr chunk, LdsPtr M, LdsPtr act, int na, int nt)
{
    if (BLOCK) chunk_steps_block<R, BW>(*(ChunkLds*)chunk, (uint64_t*)M, (const uint16_t*)act, na, nt);
    else chunk_steps_wave<R>(*(ChunkLds*)chunk, (uint64_t*)M, (const uint16_t*)act, na, nt);
}

// By the nibbles of a mask: the XOR of a table's entries.
__device__ __forceinline__ uint64_t nibble_xor(const uint64_t* tab, uint64_t m)
{
    uint64_t v = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) v ^= tab[16 * i + (int)((m >> (4 * i)) & 15)];
    return v;
}

// Up to batch_win(Wc) of the instruction's random-at-start targets, rl[i0 ..] of nr (whole block):
// the elimination of stab_random.hip on one 64-bit mask per row, from the column scratch, then one
// pass over the rows.  A row is read and written once for the window instead of once per target
// that hits it, multiplied by up to batch_win / 2 products of pivot pairs from LDS; that traffic
// is what bound the target-by-target form (4.2 TB/s of row reads and writes).  1024 circuits of 64 to
// 2048 qubits: 97 -> 22 ms a launch; of a block's 8.4 ms now, 3.8 are rows, 0.5 the elimination
// and products and 3.9 band passes.  The scratch columns of the later targets are updated by the same linear
// map.  Returns nd plus the targets of the window that the others made deterministic, which are
// appended to rl[0 .. nd).
template <int NW, int BW>
__device__ BATCH_CALL int batch_window(ArgsPtr ap, int ci_, int mi_, LdsPtr lds_, int i0_, int nr_, int nd_)
{
    const BatchArgs A = uniform_args(ap);
    const int ci = uni(ci_), i0 = uni(i0_), nr = uni(nr_);
    int nd = uni(nd_);
    const BatchCirc C = uniform_circ(A.circ + ci);
    const BatchMeas md = uniform_meas(A.meas + uni(mi_));
    const MeasLds L = meas_lds<BW>(C, (uint64_t*)lds_);
    const uint16_t* sel = md.kind == kT1T2K ? L.sel : nullptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int Wc = C.Wc, RS = C.RS, NR = C.NR, NB = 2 * C.Wc, CK = C.col_k;
    const int nt = min(batch_win(Wc), nr - i0);
    uint64_t* tab = A.tab + C.tab_off;
    uint64_t* Xs = A.cols + C.col_off;
    uint64_t* M = L.region;
    uint16_t* act = (uint16_t*)(M + NR);
    ChunkLds& K = *L.chunk;
    int* cnt = L.s_int;
    const ulonglong2 key = batch_key(A, ci);
    const int* tq = A.meas_tg + md.tq;
    for (int r = tid; r < NR / 8; r += (64 * BW)) ((uint64_t*)L.own)[r] = ~0ull;
    if (tid < 64) {
        L.tk[tid] = tid < nt ? (int)L.rlist[i0 + tid] : -1;
        K.pidx[tid] = -1;
        K.unit[tid] = K.uhit[tid] = 0ull;
        if (tid == 0) K.hits = 0;
    }
    __syncthreads();
    // stabilizer rows with x at a target, listed in row order (a wave takes consecutive bands)
    const int kt = L.tk[lane];
    const int bpw = (Wc + BW - 1) / BW;
    int mine = 0;
    for (int b = wave * bpw; b < min(Wc, (wave + 1) * bpw); ++b) {
        uint64_t v = kt >= 0 ? Xs[(size_t)(Wc + b) * CK + kt] : 0ull;
        if (__ballot(v != 0ull)) v = transpose64_dpp(v, lane);
        M[64 * b + lane] = v;
        mine += __popcll(__ballot(v != 0ull));
    }
    if (lane == 0) cnt[wave] = mine;
    __syncthreads();
    const int2 pc = wave_counts(cnt, BW, wave, lane);
    const int na = pc.y;
    int at = pc.x;
    for (int b = wave * bpw; b < min(Wc, (wave + 1) * bpw); ++b) {
        const bool f = M[64 * b + lane] != 0ull;
        const uint64_t m = __ballot(f);
        if (f) act[at + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(64 * b + lane);
        at += __popcll(m);
    }
    __syncthreads();
    const LdsPtr lk = (LdsPtr)&K, lm = (LdsPtr)M, la = (LdsPtr)act;
    if (na <= kOneWave) {
        if (wave == 0 && na > 0) {
            if (na <= 64) batch_steps<1, false, BW>(lk, lm, la, na, nt);
            else if (na <= 256) batch_steps<4, false, BW>(lk, lm, la, na, nt);
            else batch_steps<kOneWave / 64, false, BW>(lk, lm, la, na, nt);
        }
    } else if (na <= 4 * (64 * BW)) {
        batch_steps<4, true, BW>(lk, lm, la, na, nt);
    } else {
        batch_steps<16, true, BW>(lk, lm, la, na, nt);
    }
    __syncthreads();
    // the window's targets: pivots, outcomes; the others' rows follow from the units
    uint64_t run = 0;
    if (wave == 0) {
        const int pi = lane < nt ? K.pidx[lane] : -1;
        const int p = pi >= 0 ? (int)act[pi] : -1;
        run = __ballot(p >= 0);
        L.tp[lane] = p;
        if (p >= 0) {
            L.own[p] = (int8_t)lane;
            bool o;
            if (sel) {
                o = (L.evb[kt >> 6] >> (kt & 63)) & 1ull;
            } else {
                uint64_t u0, u1;
                philox(A.ibase[ci] + md.instr, (uint64_t)kt, key.x, key.y, u0, u1);
                o = (u0 >> 63) != 0;
            }
            if (o) atomicOr((unsigned long long*)&L.outb[kt >> 6], 1ull << (kt & 63));
        }
        K.unit[lane] = p >= 0 ? K.unit[lane] & run : 0ull;
        K.uhit[lane] = p >= 0 ? K.uhit[lane] : 0ull;
        const uint64_t det = __ballot(lane < nt && p < 0);
        if ((det >> lane) & 1ull) L.rlist[nd + __popcll(det & ((1ull << lane) - 1ull))] = (uint16_t)kt;
        if (lane == 0) *(uint64_t*)(L.s_int + 8) = run;
    }
    __syncthreads();
    run = uni64(*(const uint64_t*)(L.s_int + 8));
    const int nrun = __popcll(run);
    nd += nt - nrun;
    for (int e = tid; e < 256; e += (64 * BW)) {
        uint64_t u = 0, h = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if ((e >> i) & 1) {
                u ^= K.unit[4 * (e >> 4) + i];
                h ^= K.uhit[4 * (e >> 4) + i];
            }
        L.u4[e] = u;
        L.h4[e] = h;
    }
    // products of the pivots, pair by pair ((x, z) word pairs; rows 3 q + {0, 1, 2}), a row of zeros,
    // and their exponents: |P| + 2 sign each, and 2 z_2.x_1 when both are taken
    ulonglong2* prod = (ulonglong2*)L.region;
    const int npair = (nt + 1) / 2, zero = 3 * npair;
    for (int j = tid; j < Wc; j += (64 * BW)) prod[(size_t)zero * Wc + j] = make_ulonglong2(0ull, 0ull);
    for (int q = wave; q < npair; q += BW) {
        const int p0 = uni(L.tp[2 * q]), p1 = uni(L.tp[2 * q + 1]);
        const uint64_t* r0 = tab + (size_t)(NR + max(p0, 0)) * RS;
        const uint64_t* r1 = tab + (size_t)(NR + max(p1, 0)) * RS;
        int w0 = 0, w1 = 0, cr = 0;
        for (int j = lane; j < Wc; j += 64) {
            ulonglong2 a, b;
            a.x = p0 >= 0 ? r0[j] : 0ull;
            a.y = p0 >= 0 ? r0[Wc + j] : 0ull;
            b.x = p1 >= 0 ? r1[j] : 0ull;
            b.y = p1 >= 0 ? r1[Wc + j] : 0ull;
            prod[(size_t)(3 * q) * Wc + j] = a;
            prod[(size_t)(3 * q + 1) * Wc + j] = b;
            prod[(size_t)(3 * q + 2) * Wc + j] = make_ulonglong2(a.x ^ b.x, a.y ^ b.y);
            w0 += __popcll(a.x & a.y);
            w1 += __popcll(b.x & b.y);
            cr += __popcll(b.y & a.x);
        }
        const int v = wave_sum_uniform((w0 & 3) | (w1 & 3) << 8 | (cr & 1) << 16, lane);
        if (lane == 0) {
            // (sums of at most 64 x 3 per byte)
            const int s0 = p0 >= 0 ? (int)((L.sg[Wc + (p0 >> 6)] >> (p0 & 63)) & 1ull) : 0;
            const int s1 = p1 >= 0 ? (int)((L.sg[Wc + (p1 >> 6)] >> (p1 & 63)) & 1ull) : 0;
            L.tc[2 * q] = ((v & 255) + 2 * s0) & 3;
            L.tc[2 * q + 1] = (((v >> 8) & 255) + 2 * s1) & 3;
            L.tc[2 * q] |= ((v >> 16) & 1) << 2;           // bit 2: z_2.x_1 of the pair
        }
    }
    __syncthreads();
    for (int e = tid; e < 256; e += (64 * BW)) {
        int gsum = 0;
        const int t0 = 4 * (e >> 4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (((e >> i) & 1) && t0 + i < 2 * npair) gsum += L.tc[t0 + i] & 3;
#pragma unroll
        for (int i = 0; i < 4; i += 2)
            if (((e >> i) & 3) == 3 && t0 + i < 2 * npair) gsum += 2 * (L.tc[t0 + i] >> 2);
        L.g4[e] = (uint8_t)(gsum & 3);
    }
    __syncthreads();

    // masks of a band's 64 rows (lane = row): rep = partners, piv = pivots of the window
    auto band_masks = [&](int band, uint64_t& rep, uint64_t& piv, uint64_t& H) {
        uint64_t w = (kt >= 0 && ((run >> lane) & 1ull)) ? Xs[(size_t)band * CK + kt] : 0ull;
        uint64_t F = 0;
        H = 0;
        if (__ballot(w != 0ull)) {
            w = transpose64_dpp(w, lane);
            F = nibble_xor(L.u4, w);
            H = nibble_xor(L.h4, w);
        }
        const bool destab = band < Wc;
        const int t = L.own[64 * (destab ? band : band - Wc) + lane];
        const uint64_t own = __ballot(t >= 0);
        rep = destab ? own : 0ull;
        piv = destab ? 0ull : own;
        if (t >= 0) {
            F = destab ? K.unit[t] : 0ull;
            // rowsums counted: those before the replacement, then the old pivot row's
            if (destab) H = (H & ((1ull << t) - 1ull)) | (K.uhit[t] & ~((2ull << t) - 1ull));
        }
        return F;
    };

    // ---- the later targets' columns, 64 at a time ----
    for (int l0 = i0 + nt; l0 < nr; l0 += 64) {
        const int kl = l0 + lane < nr ? (int)L.rlist[l0 + lane] : -1;
        const int a = kl >= 0 ? tq[sel ? (int)sel[kl] : kl] : 0;
        for (int t = wave; t < 64; t += BW) {
            bool b = false;
            if (t < 2 * npair) b = kl >= 0 && ((prod[(size_t)(3 * (t >> 1) + (t & 1)) * Wc + (a >> 6)].x >> (a & 63)) & 1ull);
            const uint64_t m = __ballot(b);
            if (lane == 0) L.xr[t] = m;
        }
        __syncthreads();
        for (int e = tid; e < 256; e += (64 * BW)) {
            uint64_t v = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((e >> i) & 1) v ^= L.xr[4 * (e >> 4) + i];
            L.x4[e] = v;
        }
        __syncthreads();
        for (int band = wave; band < NB; band += BW) {
            uint64_t rep, piv, H;
            const uint64_t old = kl >= 0 ? Xs[(size_t)band * CK + kl] : 0ull;
            const uint64_t F = band_masks(band, rep, piv, H);
            uint64_t d = __ballot(F != 0ull) ? nibble_xor(L.x4, F) : 0ull;
            if (__ballot(d != 0ull)) d = transpose64_dpp(d, lane);
            const uint64_t nv = (old & ~(rep | piv)) ^ d;
            if (kl >= 0 && nv != old) Xs[(size_t)band * CK + kl] = nv;
        }
        __syncthreads();
    }

    // ---- the rows ----
    int lpr = 64;
    if (NW == 1)
        while (lpr > 1 && (lpr >> 1) >= Wc) lpr >>= 1;
    const int groups = 64 / lpr, grp = lane / lpr, sub = lane & (lpr - 1);
    constexpr int R = NW == 1 ? 4 : 2;
    long long changed = 0, hits = 0;
    for (int band = wave; band < NB; band += BW) {
        uint64_t rep, piv, H;
        const uint64_t F = band_masks(band, rep, piv, H);
        const uint64_t all = __ballot(F != 0ull) | rep | piv;
        const int n = __popcll(all);
        if (band < Wc) hits += __popcll(H);                 // (lane = row; the stabilizers' are K.hits)
        if (n == 0) continue;
        changed += n;
        if ((all >> lane) & 1ull) {
            const int i = __popcll(all & ((1ull << lane) - 1ull));
            int gs = 0;
#pragma unroll
            for (int q = 0; q < 16; ++q) gs += L.g4[16 * q + (int)((F >> (4 * q)) & 15)];
            L.we[i] = F;
            L.wr[i] = (uint16_t)(lane | (int)((rep >> lane) & 1ull) << 6 | (int)((piv >> lane) & 1ull) << 7);
            L.wg[i] = (uint8_t)(gs & 3);
        }
        __builtin_amdgcn_wave_barrier();
        uint64_t flip = 0;                                  // rows whose sign flips, by the groups' first lanes
        for (int n0 = 0; n0 < n; n0 += R * groups) {
            uint64_t x[R][NW], z[R][NW], cr[R][NW], E[R];
            int rw[R], G[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = n0 + r * groups + grp;
                const bool ok = i < n;
                rw[r] = ok ? (int)L.wr[i] : -1;
                E[r] = ok ? L.we[i] : 0ull;
                G[r] = ok && sub == 0 ? (int)L.wg[i] : 0;
                const uint64_t* row = tab + (size_t)(64 * band + (rw[r] & 63)) * RS;
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    const int j = sub + 64 * q;
                    const bool in = ok && rw[r] < 64 && j < Wc;
                    x[r][q] = in ? row[j] : 0ull;
                    z[r][q] = in ? row[Wc + j] : 0ull;
                    cr[r][q] = 0ull;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int q = 0; q < NW; ++q) G[r] += __popcll(x[r][q] & z[r][q]);
            for (int q = 0; q < npair; ++q) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int v = (int)((E[r] >> (2 * q)) & 3);
                    const ulonglong2* pr = prod + (size_t)(v ? 3 * q + v - 1 : zero) * Wc;
#pragma unroll
                    for (int u = 0; u < NW; ++u) {
                        // (lanes past Wc take the last word and are masked below)
                        const ulonglong2 w = pr[min(sub + 64 * u, Wc - 1)];
                        cr[r][u] ^= w.y & x[r][u];
                        x[r][u] ^= w.x;
                        z[r][u] ^= w.y;
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (int q = 0; q < NW; ++q)
                    if (sub + 64 * q < Wc) G[r] += 2 * __popcll(cr[r][q]) - __popcll(x[r][q] & z[r][q]);
                for (int d = lpr >> 1; d >= 1; d >>= 1) G[r] += __shfl_xor(G[r], d, 64);
                if (rw[r] < 0) continue;
                const int row_i = 64 * band + (rw[r] & 63);
                uint64_t* row = tab + (size_t)row_i * RS;
                const bool isp = rw[r] & 128;
                int a = -1;
                if (isp) {
                    const int k = L.tk[(int)L.own[row_i - NR]];
                    a = tq[sel ? (int)sel[k] : k];
                }
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    const int j = sub + 64 * q;
                    if (j < Wc) {
                        row[j] = isp ? 0ull : x[r][q];
                        row[Wc + j] = isp ? (j == (a >> 6) ? 1ull << (a & 63) : 0ull) : z[r][q];
                    }
                }
                if (sub == 0 && !isp) {
                    if (G[r] & 1) atomicOr(A.err, 1);
                    if (G[r] & 2) flip |= 1ull << (rw[r] & 63);
                }
            }
        }
        flip = wave_xor(flip);
        // pivots take their outcomes, partners start from +
        uint64_t outm = 0;
        if (piv) {
            const int t = ((piv >> lane) & 1ull) ? (int)L.own[64 * (band - Wc) + lane] : -1;
            const int k = t >= 0 ? L.tk[t] : 0;
            outm = __ballot(t >= 0 && ((L.outb[k >> 6] >> (k & 63)) & 1ull));
        }
        if (lane == 0) L.sg[band] = ((L.sg[band] & ~(rep | piv)) ^ flip) | outm;
        __builtin_amdgcn_wave_barrier();
    }
    hits = wave_sum((int)hits);
    if (lane == 0) {
        // row traffic of the window's one pass
        if (changed) count_add(A.counters, 6, (unsigned long long)(2 * changed * RS * 8));
        if (hits) count_add(A.counters, 5, (unsigned long long)hits);
    }
    __syncthreads();
    if (tid == 0) {
        count_add(A.counters, 4, (unsigned long long)nrun);
        count_add(A.counters, 5, (unsigned long long)(K.hits - nrun));
        // columns of the window's targets (read) and of the later ones (read and written), pivot rows
        count_add(A.counters, 6, (unsigned long long)((long long)NB * 8 * (nt + 2 * (nr - i0 - nt)) + (long long)nrun * RS * 8));
    }
    __syncthreads();
    return nd;
}

// The only random-at-start target k of the instruction, on the live tableau (whole block): a window
// for one is the longer chain of short steps (300 circuits of 64 qubits, a random target a time, 166 ->
// 152 us; 200 of 1249 qubits 1.62 -> 1.60 ms).
template <int NW, int BW>
__device__ BATCH_CALL void batch_single(ArgsPtr ap, int ci_, int mi_, LdsPtr lds_, int k_)
{
    BatchArgs A = uniform_args(ap);
    A.tile = 0;      // (one form of the rowsum: less code)
    const int ci = uni(ci_), k = uni(k_);
    const BatchCirc C = uniform_circ(A.circ + ci);
    const BatchMeas md = uniform_meas(A.meas + uni(mi_));
    const MeasLds L = meas_lds<BW>(C, (uint64_t*)lds_);
    const bool stoch = md.kind == kT1T2K;
    const ulonglong2 key = batch_key(A, ci);
    uint64_t u0, u1;
    philox(A.ibase[ci] + md.instr, (uint64_t)k, key.x, key.y, u0, u1);
    const int o = stoch ? (int)((L.evb[k >> 6] >> (k & 63)) & 1ull) : (int)(u0 >> 63);
    const int a = A.meas_tg[md.tq + (stoch ? (int)L.sel[k] : k)];
    MeasWork W;
    batch_measure_one<NW, BW>(A, C, a, o, L, W);
    if (threadIdx.x == 0) {
        if (o) L.outb[k >> 6] |= 1ull << (k & 63);
        count_add(A.counters, 4, (unsigned long long)W.nrand);
        count_add(A.counters, 5, (unsigned long long)W.nrows);
        count_add(A.counters, 6, (unsigned long long)W.bytes);
    }
    __syncthreads();
}

// One M / MR / R / T1T2 instruction of circuit ci.
//
// Slow form (any instruction): target by target on the live tableau.  In a T1T2 instruction a Philox
// draw per target picks reset (u0 < t0: a measurement whose random outcome is u1 >> 63, then X if
// it is 1), Z (u0 < t1: sign flip of every row with x at the qubit) or nothing; one wave draws 64
// targets at a time (draws do not depend on the tableau).
//
// Fast form (M/MR/R on distinct qubits whose columns the band pass extracted): every target
// deterministic at the start of the instruction is reduced at once, one wave per target (a
// deterministic outcome does not change when other qubits are measured or reset); the
// random-at-start ones then run a window at a time (batch_window); resets come last (an X on a
// measured qubit flips signs only, which commutes with the other measurements).  A T1T2 instruction
// on distinct qubits runs here with its events as the targets (batch_events): target by target they
// cost a block-wide column gather, pivot search and rowsum each, 62 of the 117 ms of 100 shots of a
// 1249-qubit circuit, which take 46 ms in all with the events in windows.
template <int NW, int BW>
__device__ BATCH_CALL void batch_measure_fast(ArgsPtr ap, int ci_, int mi_, LdsPtr lds_, int nres_, int nev_)
{
    const BatchArgs A = uniform_args(ap);
    const int ci = uni(ci_), mi = uni(mi_);
    const int2 events = make_int2(uni(nres_), uni(nev_));
    const BatchCirc C = uniform_circ(A.circ + ci);
    const BatchMeas md = uniform_meas(A.meas + mi);
    const MeasLds L = meas_lds<BW>(C, (uint64_t*)lds_);
    const int tid = threadIdx.x;
    const int Wc = C.Wc, NB = 2 * C.Wc;
    uint64_t* rs = A.rs + C.rs_off;
    for (int w = tid; w < NB; w += (64 * BW)) L.sg[w] = rs[w];
    __syncthreads();
    {
        const uint64_t* Xs = A.cols + C.col_off;
        const uint64_t* Zs = Xs + (size_t)NB * C.col_k;
        // the targets: the instruction's, or a T1T2 instruction's resets
        const bool stoch = md.kind == kT1T2K;
        const uint16_t* sel = stoch ? L.sel : nullptr;
        const int* tq = A.meas_tg + md.tq;
        const int nk = stoch ? events.x : md.K, KW = (nk + 63) >> 6;
        for (int w = tid; w < KW; w += (64 * BW)) L.outb[w] = L.rndb[w] = 0;
        // Zs first (they commute with resets of other qubits): sign flips of rows with x at them
        for (int w = tid; w < NB && events.y > events.x; w += (64 * BW)) {
            uint64_t v = L.sg[w];
            for (int k = events.x; k < events.y; ++k) v ^= Xs[(size_t)w * C.col_k + k];
            L.sg[w] = v;
        }
        __syncthreads();
        if (nk > 0) batch_dets<NW, BW>(ap, ci, lds_, nk, 0);
        // random at the start of the instruction: a window at a time; those the others turned
        // deterministic (gathered at the front of rl) come after them all
        uint16_t* rl = L.rlist;
        const int nr = batch_list<BW>(L.rndb, 0, KW, -1, -1, rl, L.s_int + 1);
        const bool ran = nr > 0;
        int nd = 0;
        if (nr == 1) batch_single<NW, BW>(ap, ci, mi, lds_, rl[0]);
        else for (int i = 0; i < nr; i += batch_win(Wc)) nd = uni(batch_window<NW, BW>(ap, ci, mi, lds_, i, nr, nd));
        // those and the resets with outcome 1 need columns of the live tableau again: gathered when
        // they are few, else (the tile fits beside what is kept up to 4096 qubits) by a band pass
        if (ran) {
            uint16_t* need = rl + nd;
            int nn = nd;
            if (md.kind != kMK) {
                __syncthreads();
                nn += batch_list<BW>(L.outb, 0, KW, -1, -1, need, L.s_int + 1);
            }
            if (nn > kBatchGatherMax && Wc <= 64) batch_segment<BW>(ap, ci, 0, 0, (LdsPtr)L.region, md.tq, stoch ? (LdsPtr)L.sel : kNoSel, nk);
            else if (nn > 0) batch_gather<BW>(A, C, tq, sel, rl, nn);
            if (nd > 0) batch_dets<NW, BW>(ap, ci, lds_, nd, 1);
        }
        if (md.rec >= 0)
            for (int k = tid; k < md.K; k += (64 * BW))
                if ((L.outb[k >> 6] >> (k & 63)) & 1ull) {
                    const long long rb = C.rec_bit_off + md.rec + k;
                    atomicOr(&A.rec[rb >> 5], 1u << (rb & 31));
                }
        if (md.kind != kMK) {
            // (a deterministic outcome 1 found just above has its column in the scratch too: it was
            // among the gathered)
            for (int w = tid; w < NB; w += (64 * BW)) {
                uint64_t x = 0;
                for (int kw = 0; kw < KW; ++kw) {
                    uint64_t m = L.outb[kw];
                    while (m) {
                        const int k = 64 * kw + ctz64(m);
                        m &= m - 1;
                        x ^= Zs[(size_t)w * C.col_k + k];
                    }
                }
                L.sg[w] ^= x;
            }
            __syncthreads();
        }
    }
    __syncthreads();
    for (int w = tid; w < NB; w += (64 * BW)) rs[w] = L.sg[w];
    __syncthreads();
}

// The slow form (see above).
template <int NW, int BW>
__device__ BATCH_CALL void batch_measure_slow(ArgsPtr ap, int ci_, int mi_, LdsPtr lds_)
{
    const BatchArgs A = uniform_args(ap);
    const int ci = uni(ci_);
    const BatchCirc C = uniform_circ(A.circ + ci);
    const BatchMeas md = uniform_meas(A.meas + uni(mi_));
    const MeasLds L = meas_lds<BW>(C, (uint64_t*)lds_);
    const int tid = threadIdx.x;
    const int Wc = C.Wc, RS = C.RS, NR = C.NR, NB = 2 * C.Wc;
    uint64_t* tab = A.tab + C.tab_off;
    uint64_t* rs = A.rs + C.rs_off;
    const ulonglong2 key = batch_key(A, ci);
    const long long col_b = (long long)2 * NR * 8;
    MeasWork W;
    for (int w = tid; w < NB; w += (64 * BW)) L.sg[w] = rs[w];
    __syncthreads();
    {
        const bool stoch = md.kind == kT1T2K;
        uint64_t* s_ev = (uint64_t*)(L.s_int + 24);        // a T1T2 chunk: reset, Z, outcome masks
        for (int c0 = 0; c0 < md.K; c0 += 64) {
            const int cn = min(64, md.K - c0);
            const uint64_t live = cn == 64 ? ~0ull : ((1ull << cn) - 1ull);
            uint64_t ev_meas = live, ev_z = 0, ev_bits = 0;  // M / MR / R: every target, in order
            if (stoch) {
                if (tid < 64) {
                    int act = 0, rb = 0;
                    if (tid < cn) {
                        uint64_t u0, u1;
                        philox(A.ibase[ci] + md.instr, (uint64_t)(c0 + tid), key.x, key.y, u0, u1);
                        act = u0 < md.t0 ? 1 : (u0 < md.t1 ? 2 : 0);
                        rb = (int)(u1 >> 63);
                    }
                    const uint64_t m1 = __ballot(act == 1), m2 = __ballot(act == 2), mb = __ballot(rb);
                    if (tid == 0) {
                        s_ev[0] = m1;
                        s_ev[1] = m2;
                        s_ev[2] = mb;
                    }
                }
                __syncthreads();
                ev_meas = s_ev[0];
                ev_z = s_ev[1];
                ev_bits = s_ev[2];
                __syncthreads();
            }
            uint64_t evm = (ev_meas | ev_z) & live;
            while (evm) {
                const int bit = ctz64(evm);
                evm &= evm - 1;
                const int t = c0 + bit;
                const int a = A.meas_tg[md.tq + t];
                if ((ev_z >> bit) & 1ull) {
                    // Z on the qubit: flip the sign of every row with x at it
                    batch_column<BW>(tab, RS, NB, a >> 6, a & 63, L.sg, true);
                    __syncthreads();
                    W.bytes += col_b;
                    continue;
                }
                int rand_bit;
                if (stoch) {
                    rand_bit = (int)((ev_bits >> bit) & 1ull);
                } else {
                    uint64_t u0, u1;
                    philox(A.ibase[ci] + md.instr, (uint64_t)t, key.x, key.y, u0, u1);
                    rand_bit = (int)(u0 >> 63);
                }
                const int outcome = batch_measure_one<NW, BW>(A, C, a, rand_bit, L, W);
                if (md.rec >= 0 && tid == 0 && outcome) {
                    const long long rb = C.rec_bit_off + md.rec + t;
                    atomicOr(&A.rec[rb >> 5], 1u << (rb & 31));
                }
                if (md.kind != kMK && outcome) {
                    // reset: apply X_a, i.e. flip the sign of every row with z at a
                    batch_column<BW>(tab, RS, NB, Wc + (a >> 6), a & 63, L.sg, true);
                    __syncthreads();
                    W.bytes += col_b;
                }
            }
        }
    }
    __syncthreads();
    for (int w = tid; w < NB; w += (64 * BW)) rs[w] = L.sg[w];
    if (tid == 0 && (W.ndet || W.nrand || W.nrows)) {
        count_add(A.counters, 4, (unsigned long long)W.nrand);
        count_add(A.counters, 2, (unsigned long long)W.ndet);
        count_add(A.counters, 5, (unsigned long long)W.nrows);
        count_add(A.counters, 6, (unsigned long long)W.bytes);
    }
    __syncthreads();
}

// NW = x words per lane of a row: 1 when every circuit has at most 4096 qubits, else 2.  Registers are
// capped at 128 (four waves per SIMD): two blocks of 8 waves share a compute unit, or one of 16.
template <int NW, int BW>
__global__ void __launch_bounds__(64 * BW) __attribute__((amdgpu_waves_per_eu(4))) k_batch(BatchArgs A)
{
    extern __shared__ uint64_t lds[];
    const ArgsPtr ap = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();   // A is the only argument
    const LdsPtr lp = (LdsPtr)lds;
    const int ci = A.order[blockIdx.x];
    const BatchCirc C = uniform_circ(A.circ + ci);
    const int end = C.step_begin + C.step_count;
    const MeasLds L = meas_lds<BW>(C, lds);
    // the band passes' tile lies beside a T1T2 instruction's event list where it fits
    const LdsPtr tile = C.Wc <= 64 ? (LdsPtr)L.region : lp, lsel = (LdsPtr)L.sel;
    int done = 0, ext_step = -1;
    int2 ev = make_int2(0, 0);
    // whether a measurement instruction can take its columns from the scratch, and how many: a T1T2
    // instruction's events (drawn here) or all its targets
    auto columns = [&](const BatchMeas& m) {
        if (!A.cols || !m.fast || C.col_k == 0) return -1;
        if (m.kind != kT1T2K) return m.K <= C.col_k && (m.K > 1 || C.Wc > kBatchSlowWc) ? m.K : -1;
        if (C.Wc > 64) return -1;
        ev = batch_events<BW>(A, C, ci, m, L);
        return ev.y <= C.col_k ? ev.y : -1;
    };
    for (int st = C.step_begin; st < end && (A.meas_quota == 0 || done < A.meas_quota);) {
        const int4 s0 = A.steps[st];
        if (s0.x == 2) {
            const int mi = uni(s0.y);
            if (ext_step != st) {
                // no band pass ran since the last measurement: gathering the columns, or a pass
                // that only reads the rows, is far cheaper than measuring target by target
                const BatchMeas md = uniform_meas(A.meas + mi);
                const bool stoch = md.kind == kT1T2K;
                const int nc = md.K >= kBatchExtractMin ? columns(md) : -1;
                if (nc >= 0) {
                    if (nc > kBatchGatherMax || (!stoch && C.Wc > 64))
                        batch_segment<BW>(ap, ci, st, st, tile, md.tq, stoch ? lsel : kNoSel, nc);
                    else if (nc > 0)
                        batch_gather<BW>(A, C, A.meas_tg + md.tq, stoch ? L.sel : nullptr, nullptr, nc);
                    ext_step = st;
                }
            }
            // (a T1T2 instruction of a small circuit has no event most times: 100 shots of a memory of 17
            // qubits 421 -> 393 us)
            if (ext_step != st) batch_measure_slow<NW, BW>(ap, ci, mi, lp);
            else if (ev.y > 0 || uni(A.meas[mi].kind) != kT1T2K) batch_measure_fast<NW, BW>(ap, ci, mi, lp, ev.x, ev.y);
            ev = make_int2(0, 0);
            ext_step = -1;
            ++st;
            ++done;
            continue;
        }
        int en = st + 1;
        while (en < end && A.steps[en].x != 2) ++en;
        // the next measurement's columns come out of this band pass when it allows that
        int nc = -1, tq = 0;
        bool stoch = false;
        if (en < end) {
            const BatchMeas m = uniform_meas(A.meas + uni(A.steps[en].y));
            nc = columns(m);
            tq = m.tq;
            stoch = m.kind == kT1T2K;
        }
        batch_segment<BW>(ap, ci, st, en, tile, tq, stoch ? lsel : kNoSel, max(nc, 0));
        if (nc >= 0) ext_step = en;
        st = en;
    }
}

// |0...0> for every circuit: block per circuit.
__global__ void k_batch_init(const BatchCirc* __restrict__ circ, uint64_t* __restrict__ tab,
                             uint64_t* __restrict__ rs)
{
    const BatchCirc C = circ[blockIdx.x];
    uint64_t* t = tab + C.tab_off;
    const long long words = (long long)2 * C.NR * C.RS;
    for (long long idx = threadIdx.x; idx < words; idx += blockDim.x) {
        const int row = (int)(idx / C.RS);
        const int c = (int)(idx - (long long)row * C.RS);
        uint64_t v = 0;
        if (row < C.NR) {
            if (row < C.n && c == (row >> 6)) v = 1ull << (row & 63);
        } else {
            const int i = row - C.NR;
            if (i < C.n && c == C.Wc + (i >> 6)) v = 1ull << (i & 63);
        }
        t[idx] = v;
    }
    for (int w = threadIdx.x; w < 2 * C.Wc; w += blockDim.x) rs[C.rs_off + w] = 0;
}

__global__ void k_zero32(uint32_t* __restrict__ p, long long n)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = 0;
}

}  // namespace stabdev
