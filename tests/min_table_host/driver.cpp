// One workgroup's use of MinTable (drsf_dev.h) on host threads: clear, add,
// flush, with one wave at its adds before another has begun to clear.  Every
// target must end with the lowest value added to it.
#include <stdio.h>
#include <time.h>

#include <algorithm>
#include <thread>
#include <vector>

#include "drsf_dev.h"

thread_local StubDim threadIdx;
StubDim blockDim{drsf::BLOCK};
pthread_barrier_t stub_barrier;

static uint64_t value(int thread, int i) { return drsf::hmix((uint64_t)thread * 1000 + i) >> 20; }

// late: the wave that comes to the table last; targets: pieces in play
static int run(int late, int targets, int per_thread) {
    std::vector<uint64_t> arr(targets, drsf::KEY_INF), want(targets, drsf::KEY_INF);
    drsf::MinTable tab;  // holds what the memory held: places taken by targets of an earlier use
    for (int s = 0; s < drsf::MIN_SLOTS; s++) {
        tab.id[s] = s % targets;
        tab.val[s] = drsf::KEY_INF;
    }
    tab.used = drsf::MIN_SLOTS;
    pthread_barrier_init(&stub_barrier, nullptr, drsf::BLOCK);
    std::vector<std::thread> group;
    for (int t = 0; t < drsf::BLOCK; t++)
        group.emplace_back([&, t] {
            threadIdx.x = (unsigned)t;
            if (t / drsf::WAVE == late) {
                const timespec wait{0, 50 * 1000 * 1000};
                nanosleep(&wait, nullptr);
            }
            tab.clear();
            for (int i = 0; i < per_thread; i++) {
                tab.add((t * 7 + i * 13) % targets, value(t, i), arr.data());
                if (i % 4 == 3) tab.flush_half(arr.data());
            }
            tab.flush(arr.data());
        });
    for (auto &t : group) t.join();
    pthread_barrier_destroy(&stub_barrier);
    for (int t = 0; t < drsf::BLOCK; t++)
        for (int i = 0; i < per_thread; i++) {
            uint64_t &w = want[(t * 7 + i * 13) % targets];
            w = std::min(w, value(t, i));
        }
    int wrong = 0;
    for (int p = 0; p < targets; p++) wrong += arr[p] != want[p];
    printf("late wave %d, %d targets, %d values a thread: %d wrong\n", late, targets, per_thread, wrong);
    return wrong;
}

int main() {
    int wrong = 0;
    for (int late = 0; late < drsf::BLOCK / drsf::WAVE; late++)
        for (int targets : {1, 300, 5000})  // one hot piece; a part of the table; more than it holds
            for (int per_thread : {1, 2, 13}) wrong += run(late, targets, per_thread);
    return wrong != 0;
}
