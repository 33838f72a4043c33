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

int main(int argc, char** argv)
{
    const struct {
        const char* name;
        void (*run)();
    } checks[] = {{"list_by_step", check_list_by_step}};
    for (const auto& c : checks)
        if (argc == 2 && !std::strcmp(argv[1], c.name)) {
            c.run();
            return bad ? 1 : 0;
        }
    std::printf("unknown check\n");
    return 2;
}
