// Host check of passes that exchange through per-lane slots, with
// register/lane exchanges inside their stages (test program; links the
// planner).
//
// Reads "M prec k r c n_steps observed half" (half 0: whole small tiles, half 2:
// the one-workgroup plan on k bits, run for n_steps steps) and then K lines "i j a b" on stdin,
// plans the call as the library does (two gates), encodes every pass and
// emulates the kernel on one tile, with every lane's registers holding the
// tile-local index of their amplitude:
//  * every factor finds its two sites on its two register bits, every
//    observable its site on the thread, register or address bit it names;
//  * the scatters of an exchange go to distinct slots inside the buffer and
//    the gathers find what they look for there; an exchange marked wave-local
//    reads only slots written by the same wave;
//  * the last stage stores every amplitude at its output address, and a pass
//    no exchange of which crosses waves stores in each wave exactly the
//    addresses it loaded.
// Prints one summary line with the mean number of lanes (of 16) whose gather
// slot shares its bank with another's; exit status 0 when every check holds.
#include <cstdio>
#include <set>
#include <vector>

#include "../../paper_0710_3747_amd/csrc/planner.hpp"

using namespace spinqp;

template <typename T>
static int check(int M, const std::vector<Coupling>& J, int k, int r, int c, int64_t steps, int observed, bool half) {
    PassParams pp;
    pp.k = k;
    pp.r = r;
    pp.c = c;
    pp.half = half;
    pp.once = !half;
    pp.gates = kMaxGates;
    const StreamPlan sp = plan_stream_best(M, J, 0.05, steps, observed, true, pp);
    constexpr int EB = int(sizeof(T)) * 2;
    const uint32_t nt = 1u << (k - r), nr = 1u << r;
    const uint32_t row = uint32_t(exchange_row_slots(int(nt), EB));
    int bad = 0;
    long swaps = 0, factors = 0, exchanges = 0, cross = 0;
    double conflicts = 0, groups = 0;
    auto fail = [&](const char* what) {
        if (bad < 10) std::printf("%s\n", what);
        ++bad;
    };
    for (const HostPass& hp : sp.passes) {
        DevTables<T> tb;
        encode_pass<T>(hp, M, observed, tb);
        const DevPass& P = tb.passes.back();
        std::vector<int> local(kMaxSites, -1);
        for (int p = 0; p < k; ++p) local[hp.sites[p]] = p;
        auto offset = [&](const int64_t* gt, const int64_t* gr, uint32_t t, uint32_t j) {
            int64_t o = 0;
            for (int q = 0; q < k - r; ++q)
                if (t >> q & 1) o += gt[q];
            for (int b = 0; b < r; ++b)
                if (j >> b & 1) o += gr[b];
            return o;
        };
        auto index = [&](int64_t off, const int32_t* tbit) {
            uint32_t x = 0;
            int64_t rest = off;
            for (int p = 0; p < k; ++p)
                if (off >> tbit[p] & 1) {
                    x |= 1u << p;
                    rest &= ~(int64_t(1) << tbit[p]);
                }
            if (rest) fail("offset outside the tile");
            return x;
        };
        const DevStage& S0 = tb.stages[P.stage0];
        std::vector<std::vector<uint32_t>> v(nt, std::vector<uint32_t>(nr));
        std::vector<std::set<int64_t>> loaded(nt / 64), stored(nt / 64);
        for (uint32_t t = 0; t < nt; ++t)
            for (uint32_t j = 0; j < nr; ++j) {
                const int64_t o = offset(S0.gt_in, S0.gr_in, t, j);
                v[t][j] = index(o, P.tbit);
                loaded[t / 64].insert(o);
            }
        std::vector<Op> left = hp.ops;
        bool any_cross = false;
        for (int si = 0; si < P.nstage; ++si) {
            const DevStage& S = tb.stages[P.stage0 + si];
            for (int o = S.op0; o < S.op0 + S.nop; ++o) {
                const DevOp<T>& op = tb.ops[o];
                if (op.code == kOpMeas) continue;
                if (op.code >= op_gate(0, 0) && op.code < kOpEnd) {
                    ++swaps;
                    const uint32_t lane = 1u << (4 + (op.code - 16) % 2), reg = 1u << ((op.code - 16) / 2);
                    for (uint32_t t = 0; t < nt; ++t)
                        if (!(t & lane))
                            for (uint32_t j = 0; j < nr; ++j)
                                if (j & reg) std::swap(v[t][j], v[t | lane][j ^ reg]);
                    continue;
                }
                int lo = -1, hi = -1;
                for (int b = 1; b < r; ++b)
                    for (int a = 0; a < b; ++a)
                        if (op.code == op_xy(a, b) || op.code == op_zz(a, b)) {
                            lo = a;
                            hi = b;
                        }
                if (lo < 0) {
                    fail("unknown op code");
                    continue;
                }
                ++factors;
                // registers 0 and (qa, qb) of every lane differ in two tile
                // positions, the factor's sites: one of the pass's factors
                const uint32_t d = v[0][0] ^ v[0][(1u << hi) | (1u << lo)];
                for (uint32_t t = 0; t < nt; ++t)
                    for (uint32_t j = 0; j < nr; ++j)
                        if ((v[t][j] ^ v[t][j ^ (1u << hi) ^ (1u << lo)]) != d) {
                            fail("register bits do not hold one position each");
                            t = nt - 1;
                            break;
                        }
                bool found = false;
                for (const Op& x : left)
                    found |= x.kind == 0 && d == ((1u << local[x.i]) | (1u << local[x.j]));
                if (!found) fail("factor on sites that the pass has no factor for");
            }
            if (tb.ops[S.op0 + S.nop].code != kOpEnd) fail("stage without an end record");
            for (int o = S.op0; o < S.op0 + S.nop; ++o) {
                // observables at the end of a stage (exit arrangement) only
                const DevOp<T>& op = tb.ops[o];
                if (op.code != kOpMeas) continue;
                bool later = false;
                for (int q = o + 1; q < S.op0 + S.nop; ++q) later |= tb.ops[q].code != kOpMeas;
                const int kind = (op.aux >> 6) & 3, idx = (op.aux >> 8) & 63, p = local[observed];
                if ((kind == 2) != (p < 0)) fail("observed site's kind");
                if (kind == 2 && idx != hp.layout[observed]) fail("observed site's address bit");
                if (kind == 2 || later) continue;
                for (uint32_t t = 0; t < nt; ++t)
                    for (uint32_t j = 0; j < nr; ++j)
                        if ((v[t][j] >> p & 1) != (kind == 0 ? t >> idx & 1 : j >> idx & 1)) {
                            fail("observed site's bit");
                            t = nt - 1;
                            break;
                        }
            }
            if (si + 1 == P.nstage) break;
            ++exchanges;
            cross += S.xnext != 0;
            any_cross |= S.xnext != 0;
            std::vector<std::vector<uint32_t>> w(nt, std::vector<uint32_t>(nr));
            const int rw = half ? r - 1 : r;
            const uint32_t nh = 1u << rw;
            for (uint32_t h = 0; h < nr / nh; ++h) {
                std::vector<int64_t> slot(size_t(row) << rw, -1), owner(slot.size(), -1);
                for (uint32_t t = 0; t < nt; ++t)
                    for (uint32_t i = 0; i < nh; ++i) {
                        const size_t s = size_t(i) * row + size_t(exchange_slot(int(t), EB));
                        if (s >= slot.size() || slot[s] >= 0) fail("scatter slot out of range or taken");
                        else {
                            slot[s] = v[t][h * nh + i];
                            owner[s] = t / 64;
                        }
                    }
                for (uint32_t t = 0; t < nt; ++t)
                    for (uint32_t i = 0; i < nh; ++i) {
                        uint64_t a = 0;
                        for (int q = 0; q < k - r; ++q)
                            if (t >> q & 1) a += S.gw[q];
                        for (int b = 0; b < rw; ++b)
                            if (i >> b & 1) a += S.gr[b];
                        const size_t s = a / EB;
                        if (a % EB || s >= slot.size() || slot[s] < 0) {
                            fail("gather slot out of range or empty");
                            continue;
                        }
                        if (!S.xnext && owner[s] != int64_t(t / 64)) fail("wave-local exchange reads another wave's slot");
                        w[t][h * nh + i] = uint32_t(slot[s]);
                    }
            }
            v.swap(w);
            std::set<uint32_t> res;
            const uint32_t mod = 1u << exchange_pad_shift(EB);
            for (uint32_t t = 0; t < 16; ++t) {
                uint64_t a = 0;
                for (int q = 0; q < 4; ++q)
                    if (t >> q & 1) a += S.gw[q];
                res.insert(uint32_t(a / EB % mod));
            }
            conflicts += 16.0 - double(res.size());
            groups += 1;
        }
        const DevStage& SL = tb.stages[P.stage0 + P.nstage - 1];
        for (uint32_t t = 0; t < nt; ++t)
            for (uint32_t j = 0; j < nr; ++j) {
                const int64_t o = offset(SL.gt_out, SL.gr_out, t, j);
                if (v[t][j] != index(o, P.tbit_out)) {
                    fail("an amplitude is stored at another tile position");
                    t = nt - 1;
                    break;
                }
                stored[t / 64].insert(o);
            }
        if (!any_cross && loaded != stored) fail("pass without barriers: a wave stores offsets it did not load");
    }
    std::printf("templates %zu exchanges %ld cross-wave %ld swaps %ld factors %ld conflicts %.2f failures %d\n",
                sp.passes.size(), exchanges, cross, swaps, factors, groups ? conflicts / groups : 0.0, bad);
    return bad;
}

// One-workgroup plan: the stages run one after the other on one state held in
// registers, with an exchange after each (between steps too).
template <typename T>
static int check_resident(const std::vector<Coupling>& J, int k, int r, int64_t steps, int observed) {
    const ResidentPlan rp = plan_resident(k, J, 0.05, observed, true, r);
    DevTables<T> tb;
    const ResidentStages rs = encode_resident<T>(rp, k, observed, tb, false);
    constexpr int EB = int(sizeof(T)) * 2;
    const uint32_t nt = 1u << (k - r), nr = 1u << r;
    const uint32_t row = uint32_t(exchange_row_slots(int(nt), EB));
    int bad = 0;
    long exchanges = 0, factors = 0, measured = 0;
    auto fail = [&](const char* what) {
        if (bad < 10) std::printf("%s\n", what);
        ++bad;
    };
    auto index = [&](const int64_t* gt, const int64_t* gr, uint32_t t, uint32_t j) {
        int64_t o = 0;
        for (int q = 0; q < k - r; ++q)
            if (t >> q & 1) o += gt[q];
        for (int b = 0; b < r; ++b)
            if (j >> b & 1) o += gr[b];
        return uint32_t(o);
    };
    std::vector<std::vector<uint32_t>> v(nt, std::vector<uint32_t>(nr));
    const int first = steps > 0 ? rs.pro0 : rs.obs0;
    for (uint32_t t = 0; t < nt; ++t)
        for (uint32_t j = 0; j < nr; ++j) v[t][j] = index(tb.stages[first].gt_in, tb.stages[first].gr_in, t, j);
    const DevStage* lastS = nullptr;
    for (int64_t step = 0; step <= steps; ++step) {
        const int st0 = step == 0 ? first : step < steps ? rs.step0 : rs.last0;
        const int nst = step > 0 ? rs.nstep : steps > 0 ? rs.npro : 1;
        for (int si = 0; si < nst; ++si) {
            const DevStage& S = tb.stages[st0 + si];
            lastS = &S;
            for (int o = S.op0; o < S.op0 + S.nop; ++o) {
                const DevOp<T>& op = tb.ops[o];
                if (op.code == kOpMeas) {
                    ++measured;
                    const int kind = (op.aux >> 6) & 3, idx = (op.aux >> 8) & 63;
                    for (uint32_t t = 0; t < nt; ++t)
                        if ((v[t][1] >> observed & 1) != (kind == 0 ? t >> idx & 1 : idx == 0)) {
                            fail("observed site's bit");
                            break;
                        }
                } else if (op.code >= op_gate(0, 0) && op.code < kOpEnd) {
                    const uint32_t lane = 1u << (4 + (op.code - 16) % 2), reg = 1u << ((op.code - 16) / 2);
                    for (uint32_t t = 0; t < nt; ++t)
                        if (!(t & lane))
                            for (uint32_t j = 0; j < nr; ++j)
                                if (j & reg) std::swap(v[t][j], v[t | lane][j ^ reg]);
                } else {
                    ++factors;
                }
            }
            if (step == steps && si + 1 == nst) break;
            if (S.xnext == kNoExchange) continue;
            ++exchanges;
            std::vector<std::vector<uint32_t>> w(nt, std::vector<uint32_t>(nr));
            std::vector<int64_t> slot(size_t(row) << r, -1), owner(slot.size(), -1);
            for (uint32_t t = 0; t < nt; ++t)
                for (uint32_t j = 0; j < nr; ++j) {
                    const size_t s = size_t(j) * row + size_t(exchange_slot(int(t), EB));
                    slot[s] = v[t][j];
                    owner[s] = t / 64;
                }
            for (uint32_t t = 0; t < nt; ++t)
                for (uint32_t j = 0; j < nr; ++j) {
                    uint64_t a = 0;
                    for (int q = 0; q < k - r; ++q)
                        if (t >> q & 1) a += S.gw[q];
                    for (int b = 0; b < r; ++b)
                        if (j >> b & 1) a += S.gr[b];
                    const size_t s = a / EB;
                    if (a % EB || s >= slot.size() || slot[s] < 0) {
                        fail("gather slot out of range or empty");
                        continue;
                    }
                    if (!S.xnext && owner[s] != int64_t(t / 64)) fail("wave-local exchange reads another wave's slot");
                    w[t][j] = uint32_t(slot[s]);
                }
            v.swap(w);
            // the next stage's entry is where the exchange put everything
            const int nx = si + 1 < nst ? st0 + si + 1 : step + 1 < steps ? rs.step0 : rs.last0;
            const DevStage& N = tb.stages[nx];
            for (uint32_t t = 0; t < nt; ++t)
                for (uint32_t j = 0; j < nr; ++j)
                    if (v[t][j] != index(N.gt_in, N.gr_in, t, j)) {
                        fail("exchange does not give the next stage's entry");
                        t = nt - 1;
                        break;
                    }
        }
    }
    for (uint32_t t = 0; t < nt; ++t)
        for (uint32_t j = 0; j < nr; ++j)
            if (v[t][j] != index(lastS->gt_out, lastS->gr_out, t, j)) {
                fail("an amplitude is stored at another index");
                t = nt - 1;
                break;
            }
    if (measured != steps + 1) fail("not one observable per step");
    std::printf("resident exchanges %ld factors %ld failures %d\n", exchanges, factors, bad);
    return bad;
}

int main() {
    int M, prec, k, r, c, observed, half;
    long long steps;
    if (std::scanf("%d %d %d %d %d %lld %d %d", &M, &prec, &k, &r, &c, &steps, &observed, &half) != 8) return 2;
    std::vector<Coupling> J;
    Coupling x;
    while (std::scanf("%d %d %lf %lf", &x.i, &x.j, &x.a, &x.b) == 4) J.push_back(x);
    if (half == 2)
        return (prec == 1 ? check_resident<float>(J, k, r, steps, observed)
                          : check_resident<double>(J, k, r, steps, observed)) ? 1 : 0;
    const int bad = prec == 1 ? check<float>(M, J, k, r, c, steps, observed, half != 0)
                              : check<double>(M, J, k, r, c, steps, observed, half != 0);
    return bad ? 1 : 0;
}
