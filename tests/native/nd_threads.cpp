// Test-only program: the nested-dissection plan of a box grid where no thread
// can be had (stacks larger than the address space left), and then with threads:
// the same order.  Prints "same" and returns 0.
#include <pthread.h>
#include <sys/resource.h>

#include <cstdio>
#include <exception>
#include <thread>
#include <vector>

#include "msp_nd.h"

int main()
{
    const int m = 20, n = m * m * m;
    std::vector<int> rp(1, 0), ci;
    for (int k = 0; k < m; ++k)
        for (int j = 0; j < m; ++j)
            for (int i = 0; i < m; ++i) {
                const int c = i + m * (j + m * k);
                if (k) ci.push_back(c - m * m);
                if (j) ci.push_back(c - m);
                if (i) ci.push_back(c - 1);
                ci.push_back(c);
                if (i + 1 < m) ci.push_back(c + 1);
                if (j + 1 < m) ci.push_back(c + m);
                if (k + 1 < m) ci.push_back(c + m * m);
                rp.push_back((int)ci.size());
            }
    pthread_attr_t a;
    size_t usual = 0;
    pthread_attr_init(&a);
    pthread_getattr_default_np(&a);
    pthread_attr_getstacksize(&a, &usual);
    pthread_attr_setstacksize(&a, (size_t)64 << 30);
    pthread_setattr_default_np(&a);
    rlimit lim{};
    getrlimit(RLIMIT_AS, &lim);
    rlimit tight = lim;
    tight.rlim_cur = (rlim_t)16 << 30;
    setrlimit(RLIMIT_AS, &tight);
    bool refused = false;
    try {
        std::thread([] {}).join();
    } catch (const std::exception &) {
        refused = true;
    }
    if (!refused) return std::puts("threads could be had"), 2;
    msp::NdPlan alone, with;
    try {
        if (!msp::nd_plan(n, rp.data(), ci.data(), alone)) return std::puts("declined"), 3;
    } catch (const std::exception &e) {
        return std::printf("threw: %s\n", e.what()), 4;
    }
    setrlimit(RLIMIT_AS, &lim);
    pthread_attr_setstacksize(&a, usual);
    pthread_setattr_default_np(&a);
    if (!msp::nd_plan(n, rp.data(), ci.data(), with)) return std::puts("declined"), 3;
    if (alone.perm != with.perm || alone.wtot != with.wtot) return std::puts("differ"), 5;
    std::puts("same");
    return 0;
}
