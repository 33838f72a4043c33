// Checks of the library's host side and of its device code's host-callable parts, compiled for the
// host alone and run without a GPU by test_host_rules_cpu.py: `host_rules <check>` prints what is
// wrong and returns 1, or returns 0.
#include "stab_api.hip"

#include <cstring>
#include <pthread.h>
#include <thread>
#include <unistd.h>

static int bad = 0;

#define EXPECT(cond, ...)                \
    do {                                 \
        if (!(cond)) {                   \
            std::printf(__VA_ARGS__);    \
            std::printf("\n");           \
            ++bad;                       \
        }                                \
    } while (0)

// The list of a run's noise events: a thread that is late after each barrier still reads every
// step's end before the others append to the next.
static void check_list_by_step()
{
    constexpr int T = 4, N = 8;
    int off[N + 1] = {}, count = 0;
    pthread_barrier_t bar;
    pthread_barrier_init(&bar, nullptr, T);
    std::vector<std::thread> th;
    for (int t = 0; t < T; ++t)
        th.emplace_back([&, t] {
            list_by_step(
                N, t, off, &count, [&](int i) { __atomic_fetch_add(&count, t == 0 ? 0 : i + t, __ATOMIC_SEQ_CST); },
                [&] {
                    pthread_barrier_wait(&bar);
                    if (t == 0) usleep(3000);
                });
        });
    for (auto& x : th) x.join();
    pthread_barrier_destroy(&bar);
    int want = 0;
    for (int i = 0; i < N; ++i) {
        for (int t = 1; t < T; ++t) want += i + t;
        EXPECT(off[i + 1] == want, "step %d ends at %d, not %d", i, off[i + 1], want);
    }
}

// A layer that may take more than one window has the array of changed quarter bands: more targets
// than a window holds, or rows k_plan may have to cut a window for.
static void check_windows_of_a_layer()
{
    for (int n : {1, 64, 300, 4096, 4097, 4160, 10240})
        for (int K : {1, 63, 64, 65, 130, 256, 257, 4096}) {
            if (K > n) continue;
            const Geom g = make_geom(n, 3, STAB_MODE_SHARED);
            const int least = g.NR > kPlanRows ? 64 : 64 * kWinChunks;   // targets of the smallest window but the last
            const RandLayout L = rand_layout(g, K);
            EXPECT(L.multi == (K > least), "n %d, %d targets: multi %d", n, K, (int)L.multi);
            EXPECT((rand_bufs(L, (void*)256).dirty != nullptr) == (K > least), "n %d, %d targets: dirty", n, K);
            EXPECT(L.pm - L.dirty >= (K > least ? (size_t)g.S * g.NB * 4 : 0), "n %d, %d targets: size", n, K);
        }
}

// The part of a noise list that a segment loads ahead, up to the most events a segment may have.
static void check_list_ahead()
{
    for (int ahead : {1024, 2048})
        for (int n : {0, 1, 1023, 1024, 1025, 2048, 1 << 20, (1 << 28) - 1, 1 << 28, 1 << 29, (1 << 29) + 5, 1 << 30, INT_MAX}) {
            const int got = ahead_bytes(n, ahead), want = 8 * std::min(n, ahead);
            EXPECT(got == want, "%d entries, %d ahead: %d bytes, not %d", n, ahead, got, want);
        }
}

// A captured layer holds three launches a window: as many windows as it takes, known or at most one.
static void check_captures()
{
    for (int n : {300, 4096, 4097, 10081})
        for (int K : {1, 64, 65, 256, 257, 5040}) {
            if (K > n) continue;
            const Geom g = make_geom(n, 10, STAB_MODE_SHARED);
            EXPECT(captures(g, K, true), "n %d, %d targets: windows known", n, K);
            EXPECT(captures(g, K, false) == !rand_layout(g, K).multi, "n %d, %d targets: windows unknown", n, K);
        }
}

// Waves of the batch kernel: small circuits never take 16, a launch configuration decides itself.
static void check_batch_waves()
{
    for (int nc : {1, 100, 256, 257, 1024})
        for (int wc : {1, 5, 6, 20, 128}) {
            const int want = nc <= 256 && wc > 5 ? 16 : 8;
            EXPECT(batch_waves(nc, wc, 0, 256) == want, "%d circuits of %d words: %d waves", nc, wc, batch_waves(nc, wc, 0, 256));
            EXPECT(batch_waves(nc, wc, 8, 256) == 8 && batch_waves(nc, wc, 0x208, 256) == 16, "configured: %d, %d", nc, wc);
        }
}

// The scratch limit of stab_sample_noalloc: a gate counts 8 bytes, and what is carved stays within
// the slack of what is counted.
static void check_noalloc_limit()
{
    auto counted = [](int n, int shots, int mode, int layers, int K, size_t* carved) {
        std::vector<stab_instr> ins;
        std::vector<int32_t> tg;
        auto add = [&](uint32_t kind, int m) {
            stab_instr i{};
            i.kind = kind;
            i.ntargets = (uint32_t)m;
            ins.push_back(i);
            for (int q = 0; q < m; ++q) tg.push_back(q);
        };
        for (int l = 0; l < layers; ++l) add(l & 1 ? STAB_S : STAB_H, n);
        add(STAB_M, K);
        const Geom g = make_geom(n, shots, mode);
        stab_program P;
        ProgramBlob B;
        if (compile_host(g, ins.data(), (int)ins.size(), tg.data(), (int64_t)tg.size(), P, B)) return (size_t)0;
        size_t sizes[kExecBufs], sum = 256 + align256(kNumCounters * kCounterStripes * 8) + align256(B.bytes.size());
        exec_sizes(g, P, false, sizes);
        for (size_t b : sizes) sum += std::max<size_t>(align256(b), 256);
        if (carved) *carved = sum;
        return noalloc_bytes(g, P, B);
    };
    for (int n : {32, 64, 4096}) {
        const size_t a = counted(n, 1, STAB_MODE_SHARED, 32, 1, nullptr), b = counted(n, 1, STAB_MODE_SHARED, 64, 1, nullptr);
        EXPECT(b - a == 32 * (size_t)(16 + 8 * n), "n %d: 32 layers count %zu bytes", n, b - a);
    }
    for (int n : {1, 2, 63, 64, 300, 1249, 4096, 4097, 10240})
        for (int shots : {1, 2, 100, 1000, 20000, 65535})
            for (int mode : {STAB_MODE_SHARED, STAB_MODE_FULL})
                for (int K : {1, 2, 64, 65, 256, 257, 1000, 4000}) {
                    if (K > n) continue;
                    size_t carved = 0;
                    const size_t c = counted(n, shots, mode, 3, K, &carved);
                    if (c == 0 || c > STAB_NOALLOC_SCRATCH_BYTES) continue;
                    EXPECT(carved <= STAB_NOALLOC_SCRATCH_BYTES + kScratchSlack, "n %d, %d shots, mode %d, %d targets: %zu carved, %zu counted",
                           n, shots, mode, K, carved, c);
                }
}

int main(int argc, char** argv)
{
    const struct {
        const char* name;
        void (*run)();
    } checks[] = {{"list_by_step", check_list_by_step}, {"windows_of_a_layer", check_windows_of_a_layer},
                  {"list_ahead", check_list_ahead},
                  {"captures", check_captures},
                  {"batch_waves", check_batch_waves},
                  {"noalloc_limit", check_noalloc_limit}};
    for (const auto& c : checks)
        if (argc == 2 && !std::strcmp(argv[1], c.name)) {
            c.run();
            return bad ? 1 : 0;
        }
    std::printf("unknown check\n");
    return 2;
}
