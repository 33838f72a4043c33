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

int main(int argc, char** argv)
{
    const struct {
        const char* name;
        void (*run)();
    } checks[] = {{"list_by_step", check_list_by_step}, {"windows_of_a_layer", check_windows_of_a_layer},
                  {"list_ahead", check_list_ahead},
                  {"captures", check_captures},
                  {"batch_waves", check_batch_waves}};
    for (const auto& c : checks)
        if (argc == 2 && !std::strcmp(argv[1], c.name)) {
            c.run();
            return bad ? 1 : 0;
        }
    std::printf("unknown check\n");
    return 2;
}
