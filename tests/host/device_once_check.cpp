// DeviceOnce (csrc/lss_device_once.h) with pretended GPUs: each gets its own run, a failure is retried, and threads that
// come first together all return only after the work is done.
#include "lss_device_once.h"

#include <cstdio>
#include <thread>
#include <vector>

enum Status { OK = 0, FAILED = 1 };

int main()
{
    lss::DeviceOnce once;
    int runs[80] = {};
    for (int round = 0; round < 3; ++round)
        for (int dev : {0, 1, 7, 63, 70}) once.run(dev, [&] { ++runs[dev]; return OK; });
    if (runs[0] != 1 || runs[1] != 1 || runs[7] != 1 || runs[63] != 1) { std::puts("not once per GPU"); return 1; }
    if (runs[70] != 3) { std::puts("a GPU past the mask must run it every time"); return 1; }

    lss::DeviceOnce retry;
    int tries = 0;
    const auto second_works = [&] { return ++tries < 2 ? FAILED : OK; };
    if (retry.run(3, second_works) != FAILED || retry.run(3, second_works) != OK || retry.run(3, second_works) != OK || tries != 2) {
        std::puts("a failure must be reported and tried again");
        return 1;
    }

    lss::DeviceOnce shared;
    std::atomic<int> set[4] = {};
    std::atomic<int> early{0};
    std::vector<std::thread> threads;
    for (int i = 0; i < 8; ++i)
        threads.emplace_back([&, i] {
            for (int dev = 0; dev < 4; ++dev) {
                shared.run((dev + i) % 4, [&] { set[(dev + i) % 4] = 1; return OK; });
                if (!set[(dev + i) % 4]) ++early;
            }
        });
    for (std::thread &t : threads) t.join();
    if (early != 0) { std::puts("returned before the work was done"); return 1; }
    std::puts("clean");
    return 0;
}
