// Host check of the single-precision rotation coefficients of a plan (test
// program; links the planner).
//
// Reads "M k r half n_steps" and then K lines "i j b" on stdin, plans and
// encodes the call as the library does (two gates, 4 low bits) and goes over
// its rotations in encoding order.  A rotation with coefficients (t, s) has the
// off-diagonal elements t (2 - t s) and -s; per pair of sites the differences
// of the two (signed by the register bits that hold the sites) and the errors
// of the angle are added up over the passes before the repeated block and over
// the block.  With each coefficient free to move by one unit of the last place
// the sums of two candidates differ by at most 2 ulp(t) + 2 ulp(s), so a sum can
// always be brought back to within that; without the feedback it grows with the
// number of rotations.  Prints the largest sum in those units and the number of
// rotations of a pair; exit status 0 when no sum exceeds one unit.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <map>
#include <utility>
#include <vector>

#include "../../paper_0710_3747_amd/csrc/planner.hpp"

using namespace spinqp;

int main() {
    int M, k, r, half;
    long long steps;
    if (std::scanf("%d %d %d %d %lld", &M, &k, &r, &half, &steps) != 5) return 2;
    std::vector<Coupling> J;
    Coupling x{};
    while (std::scanf("%d %d %lf", &x.i, &x.j, &x.b) == 3) J.push_back(x);
    PassParams pp;
    pp.k = k;
    pp.r = r;
    pp.c = 4;
    pp.half = half != 0;
    pp.once = half == 0;
    pp.gates = kMaxGates;
    const StreamPlan sp = plan_stream_best(M, J, 0.05, steps, 0, true, pp);
    auto ulp = [](float v) { return double(std::nextafter(std::fabs(v), INFINITY)) - std::fabs(v); };
    struct Sum {
        double across = 0, angle = 0;
        int n = 0;
    };
    std::map<std::pair<int, int>, Sum> sums;
    double worst = 0;
    int most = 0, blocks = 0;
    DevTables<float> tb;
    for (const HostPass& hp : sp.passes) {
        if (hp.block_start) {
            ++blocks;
            sums.clear();
        }
        size_t at = tb.ops.size();
        encode_pass<float>(hp, M, 0, tb);
        const DevPass& P = tb.passes.back();
        auto site_at = [&](int64_t offset) {
            for (int p = 0; p < k; ++p)
                if (offset == int64_t(1) << hp.bit_in[p]) return hp.sites[p];
            return -1;
        };
        for (int si = 0; si < P.nstage; ++si, ++at) {
            // the sites on the register and thread bits at the stage's entry
            const DevStage& S = tb.stages[P.stage0 + si];
            std::vector<int> reg(r), lane(k - r);
            for (int b = 0; b < r; ++b) reg[b] = site_at(S.gr_in[b]);
            for (int q = 0; q < k - r; ++q) lane[q] = site_at(S.gt_in[q]);
            // one entry per rotation: angles beyond a quarter turn take several
            std::vector<std::pair<const Op*, double>> factors;
            for (const StageItem& it : hp.stages[si].prog)
                if (it.op >= 0 && hp.ops[it.op].kind == 0) {
                    const double theta = 0.5 * hp.ops[it.op].B;
                    int n = 1;
                    while (std::fabs(theta / n) > 1.5707963267948966) n *= 2;
                    factors.insert(factors.end(), size_t(n), {&hp.ops[it.op], theta / n});
                }
            size_t f = 0;
            for (; tb.ops[at].code != kOpEnd; ++at) {
                const DevOp<float>& op = tb.ops[at];
                if (op.code == kOpMeas) continue;
                if (op.code >= op_gate(0, 0)) {
                    std::swap(reg[(op.code - 16) / 2], lane[4 + (op.code - 16) % 2]);
                    continue;
                }
                int lo = 0, hi = 1;
                while (op_xy(lo, hi) != op.code)
                    if (++lo == hi) lo = 0, ++hi;
                const double theta = factors.at(f).second;
                const Op& h = *factors[f++].first;
                const bool first = reg[lo] == h.i && reg[hi] == h.j;
                if (!first && !(reg[lo] == h.j && reg[hi] == h.i)) {
                    std::printf("rotation on other sites than its factor's\n");
                    return 1;
                }
                const double ts = double(op.t) * op.s, b = op.t * (2.0 - ts);
                Sum& u = sums[{h.i, h.j}];
                u.across += (first ? 1.0 : -1.0) * (b - op.s);
                u.angle += std::atan2(0.5 * (b + op.s), 1.0 - ts) - theta;
                const double unit = 2.0 * ulp(op.t) + 2.0 * ulp(op.s);
                worst = std::fmax(worst, std::fmax(std::fabs(u.across), std::fabs(u.angle)) / unit);
                most = std::max(most, ++u.n);
            }
        }
    }
    std::printf("rotations of a pair %d blocks %d worst %.3f\n", most, blocks, worst);
    return worst <= 1.0 ? 0 : 1;
}
