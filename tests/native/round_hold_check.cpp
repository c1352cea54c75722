// Host unit checks of RoundHold (paper_2110_01481_amd/csrc/group_budget.h): the hold of a
// batched engine's rounds, extended while nobody waits and given up to a waiter otherwise.
// Built and run by tests/test_group_budget_host.py; prints "ok" when every check passes.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>

#include "group_budget.h"

using abg::GroupBudget;
using abg::RoundHold;

#define CHECK(c)                                              \
    do {                                                      \
        if (!(c)) {                                           \
            std::printf("failed line %d: %s\n", __LINE__, #c); \
            std::exit(1);                                     \
        }                                                     \
    } while (0)

int main()
{
    const long long U = GroupBudget::kUnits;
    {   // alone: later rounds extend the hold, the last one to end gives it back
        GroupBudget b;
        RoundHold h;
        h.take(b);
        h.take(b);
        h.take(b);
        CHECK(b.in_use() == U && !b.contended());
        h.give();
        h.give();
        CHECK(b.in_use() == U);
        h.give();
        CHECK(b.in_use() == 0);
        h.take(b);
        h.give();
        CHECK(b.in_use() == 0);
    }
    {   // a waiter is served before the hold is extended
        GroupBudget b;
        RoundHold h;
        h.take(b);
        std::atomic<int> got{0};
        std::thread other([&] {
            b.acquire(10);
            got = 1;
            std::this_thread::sleep_for(std::chrono::milliseconds(50));
            got = 2;
            b.release(10);
        });
        while (!b.contended()) std::this_thread::yield();
        std::thread cb([&] {
            std::this_thread::sleep_for(std::chrono::milliseconds(50));
            CHECK(got == 0);
            h.give();
        });
        h.take(b);   // queues behind the waiter, which holds a share until got == 2
        CHECK(got == 2 && b.in_use() == U);
        cb.join();
        other.join();
        h.give();
        CHECK(b.in_use() == 0);
    }
    {   // rounds, callbacks and small requests from other threads: nothing is lost
        GroupBudget b;
        RoundHold h;
        std::atomic<long long> small{0};
        std::atomic<bool> over{false};
        std::thread others[3];
        for (auto &t : others)
            t = std::thread([&] {
                while (!over) {
                    b.acquire(U / 4);
                    CHECK(b.in_use() <= 3 * (U / 4));
                    ++small;
                    b.release(U / 4);
                }
            });
        for (int i = 0; i < 300; ++i) {
            h.take(b);
            CHECK(b.in_use() == U);
            std::thread([&] { h.give(); }).join();
        }
        over = true;
        for (auto &t : others) t.join();
        CHECK(b.in_use() == 0 && small > 0);
    }
    std::printf("ok\n");
    return 0;
}
