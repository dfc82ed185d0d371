// Host check of the batch kernel's LDS buffer (test program): for every
// precision, tile mode and size of a one-workgroup problem, the slots that its
// exchange and its staging in memory order touch, counted one by one, lie
// inside the buffer; so do the gangs' tiles.  Exit status 0 when they do.
#include <algorithm>
#include <cstdio>

#include "../../paper_0710_3747_amd/csrc/device_plan.hpp"

using namespace spinqp;

int main() {
    int bad = 0;
    for (int f32 = 0; f32 < 2; ++f32)
        for (int half = 0; half < 2; ++half) {
            const int eb = f32 ? 8 : 16, nt = half ? 256 : 512, K = f32 ? 14 : 13;
            const int slots = batch_lds_slots(f32 != 0, half != 0);
            int top = 0;
            for (int M = 1; M <= K - 1; ++M) {
                const int r = batch_resident_regs(M, half != 0);
                for (int t = 0; t < nt; ++t)
                    top = std::max(top, ((1 << r) - 1) * exchange_row_slots(nt, eb) + exchange_slot(t, eb));
                top = std::max(top, (nt << r) - 1);
                if ((nt << r) < 1 << M) ++bad;        // the state does not fit the registers
            }
            const int rr = batch_regs(f32 != 0, half != 0);
            if ((nt << rr) != 1 << K) ++bad;
            if (half)
                for (int t = 0; t < nt; ++t)
                    top = std::max(top, ((1 << (rr - 1)) - 1) * exchange_row_slots(nt, eb) + exchange_slot(t, eb));
            else
                top = std::max(top, (1 << K) - 1);
            std::printf("%s %s: %d slots, last one touched %d, %d bytes\n", f32 ? "complex64" : "complex128",
                        half ? "half" : "whole", slots, top, slots * eb);
            // and some room for the sums beside it in the 160 KiB
            if (top >= slots || slots * eb > 152 * 1024) ++bad;
        }
    return bad ? 1 : 0;
}
