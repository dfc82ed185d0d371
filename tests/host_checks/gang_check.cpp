// Host check of a gang's meetings (test program): members that arrive and wait
// as the batch kernel's do, with the counter started short of where 31 and 32
// bits wrap, never pass a meeting before every member has arrived and never
// wait once all have.  Exit status 0 when that holds.
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "../../paper_0710_3747_amd/csrc/device_plan.hpp"

using namespace spinqp;

int main() {
    int bad = 0;
    for (const uint32_t G : {2u, 8u, 64u, 512u})
        for (const uint64_t wrap : {uint64_t(1) << 31, uint64_t(1) << 32}) {
            uint32_t epoch = uint32_t(wrap / G) - 3;      // meetings behind the gang
            uint32_t counter = epoch * G;
            for (int meeting = 0; meeting < 6; ++meeting) {
                const uint32_t target = ++epoch * G;
                for (uint32_t arrived = 0; arrived < G; ++arrived) {
                    if (!gang_waits(counter, target)) ++bad;        // passed too early
                    ++counter;
                }
                // everyone has arrived; the quickest are already at the next meeting
                for (uint32_t ahead = 0; ahead < G; ++ahead)
                    if (gang_waits(counter + ahead, target)) ++bad;
            }
        }
    const uint64_t second = kGangWaitTicks / 20;
    for (const uint64_t every : {1 * second, 15 * second, 19 * second})
        for (const uint64_t ends : {uint64_t(0), 30 * second, 5000 * second}) {
            const uint64_t t0 = 1234567;
            GangClock clock{t0};
            uint64_t gave_up = 0;
            for (uint64_t t = 0; t < 6000 * second && !gave_up; t += second / 4) {
                const uint32_t progress = uint32_t((t < ends ? t : ends) / every);
                if (clock.due(t0 + t) && clock.stalled(t0 + t, progress)) gave_up = t;
            }
            if (gave_up <= ends / every * every || gave_up > ends + 2 * kGangWaitTicks + second) ++bad;
        }
    std::printf("failures %d\n", bad);
    return bad ? 1 : 0;
}
