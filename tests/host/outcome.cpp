// The wait for a unit's outcome in the resident pass (adasum_outcome.h): it comes back with what the unit wrote in this call, and it
// ends also where no such word ever comes; and waves that have to agree on what they see.  Built and run by tests/test_outcome_cpu.py.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>

#include "adasum_outcome.h"

using namespace adasum;

#define CHECK(cond)                                                                           \
    do {                                                                                      \
        if (!(cond)) {                                                                        \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);     \
            std::exit(1);                                                                     \
        }                                                                                     \
    } while (0)

int main() {
    for (unsigned tag : {1u, 2u, 5u, 0x1000000u}) {
        // words that are no outcome of this call: none, an older call's, the next one's
        for (int stale : {0, outcome_word(tag, 0), outcome_word(tag + 1, kDone), outcome_word(tag + 1, kGaveUp),
                          tag > 1 ? outcome_word(tag - 1, kGaveUp) : 0, tag > 1 ? outcome_word(tag - 1, kDone) : 0}) {
            int looks = 1000, taken = 0;
            CHECK(await_outcome([&]() { ++taken; return stale; }, tag, [&]() { return --looks > 0; }) == kOverdue);
            CHECK(taken == 1000);
        }
        for (int what : {int(kDone), int(kGaveUp)})
            // the unit's word is there at the n-th look of five, or after them
            for (int n = 1; n <= 7; ++n) {
                int looks = 5, taken = 0;
                const int got = await_outcome([&]() { return ++taken >= n ? outcome_word(tag, what) : 0; }, tag, [&]() { return --looks > 0; });
                CHECK(got == (n <= 5 ? what : static_cast<int>(kOverdue)));
            }
    }
    // a unit beside the wait; and another call that clears the word whenever it is written
    for (int rep = 0; rep < 500; ++rep) {
        std::atomic<int> word{0};
        std::thread unit([&]() { word = outcome_word(7, rep % 2 ? kDone : kGaveUp); });
        CHECK(await_outcome([&]() { return word.load(); }, 7, []() { return true; }) == (rep % 2 ? kDone : kGaveUp));
        unit.join();
    }
    int looks = 100000;
    std::atomic<int> word{0};
    CHECK(await_outcome([&]() { word = outcome_word(3, kDone); word = 0; return word.load(); }, 3, [&]() { return --looks > 0; }) == kOverdue);
    // a wave that looks late, beside one that changes what is looked at as soon as it may
    for (int rep = 0; rep < 5; ++rep) {
        std::atomic<int> late{0}, arrived{0};
        auto barrier = [&]() {
            ++arrived;
            while (arrived < 2) std::this_thread::yield();
        };
        bool first = true, second = true;
        std::thread quick([&]() {
            first = same_answer([&]() { return late != 0; }, barrier);
            late = 1;
        });
        std::this_thread::sleep_for(std::chrono::milliseconds(50));
        second = same_answer([&]() { return late != 0; }, barrier);
        quick.join();
        CHECK(!first && !second);
    }
    std::printf("outcomes ok\n");
    return 0;
}
