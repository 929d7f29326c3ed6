// per_device (csrc/per_device.hpp) with two devices and none: each is asked once,
// its own answer returned, whichever came first.
#include "per_device.hpp"

#include <cstdio>
#include <thread>
#include <vector>

static thread_local int current = 0;   // what hipGetDevice answers; -1: an error
static int asked[2];

extern "C" hipError_t hipGetDevice(int* dev) {
    if (current < 0) return hipErrorNoDevice;
    *dev = current;
    return hipSuccess;
}

static int limit() {
    return amg355::per_device([](int dev) {
        asked[dev] += 1;
        return 100 + dev;
    });
}

int main() {
    int bad = 0;
    for (int round = 0; round < 3; ++round)
        for (int dev : {1, 0, -1}) {
            current = dev;
            bad += limit() != (dev < 0 ? 0 : 100 + dev);
        }
    std::vector<std::thread> threads;
    std::vector<int> wrong(8, 0);
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&wrong, t] {
            current = t % 2;
            for (int k = 0; k < 1000; ++k) wrong[t] += limit() != 100 + t % 2;
        });
    for (auto& t : threads) t.join();
    for (int w : wrong) bad += w;
    bad += asked[0] != 1 || asked[1] != 1;
    std::printf("%s\n", bad ? "per_device: wrong" : "per_device: ok");
    return bad != 0;
}
