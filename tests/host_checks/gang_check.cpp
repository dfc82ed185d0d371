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
    std::printf("failures %d\n", bad);
    return bad ? 1 : 0;
}
