// device_plan.hpp -- plain-old-data plan records shared by the host planner
// and the gfx950 kernels, plus the LDS address swizzle both sides use.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define SPIN_HD __host__ __device__
#else
#define SPIN_HD
#endif

namespace spinqp {

constexpr int kMaxTileBits = 14;    // 2^14 amplitudes: 128 KiB of complex64 in LDS
constexpr int kMaxRegBits = 6;      // at most 64 amplitudes per lane
constexpr int kMaxMeas = 4;         // observable slots one pass can hold
constexpr int kMaxSites = 40;
constexpr int kBatchRing = 16;      // observable slots per gang problem (steps mod 16)
constexpr int kMaxMeasProfile = 64; // per-site observables one pass can hold (all-site profile)

// Op codes.  A two-spin factor on register bits a < b of a stage is one op
// op_xy(a, b) and, when it carries an I^z I^z phase, a second one op_zz(a, b).
// op_gate(q, g) exchanges register bit q with lane bit 4 + g (g = 0, 1):
// register q = 1 of the lanes with the lane bit clear trades places with
// register q = 0 of the lanes with it set, so the site on the lane bit
// becomes a register site and the other way round, without LDS.  kOpMeas
// accumulates the observable of the state at that point; kOpEnd ends every
// stage's ops (not counted in DevStage::nop).  The codes are the slots of the
// kernels' handlers (a phase's takes four).
constexpr int32_t op_xy(int a, int b) { return b * (b - 1) / 2 + a; }
constexpr int32_t op_gate(int q, int g) { return 16 + 2 * q + g; }
constexpr int32_t op_zz(int a, int b) { return 32 + 4 * op_xy(a, b); }
constexpr int32_t kOpEnd = 28;
constexpr int32_t kOpMeas = 29;
constexpr int kMaxGates = 2;        // lane bits 4 and 5
// kOpMat (matrix engine, 32 registers per lane): multiply the lane's
// registers by a dense 32 x 32 complex matrix, the product of consecutive
// factors of the stage, on MFMA.  aux = index of the matrix in the matrix
// table: kMatFloats floats per matrix, the real 64 x 64 form
// W = [[Re U, -Im U], [Im U, Re U]] in MFMA A-operand order
// (W[32 b + (l % 32)][2 p + l / 32] at float (32 b + p) * 64 + l).
constexpr int32_t kOpMat = 30;
constexpr int kMatFloats = 64 * 64;

// One op of a stage.  For a factor with integrated strengths
// (A, B) = (sum a*tau, sum b*tau) over the merged two-spin propagators:
//   op_xy: theta = B/2, (t, s) = (tan(theta/2), sin(theta)) for the three-shear
//          rotation, and their negatives (nt, ns)
//   op_zz: (t, s) = (cos, sin)(A/4), the anti-aligned phase exp(+i A/4)
// For kOpMeas, aux = slot | kind << 6 | index << 8: the observed site's bit is
// thread bit `index` (kind 0), register bit `index` (kind 1) or global address
// bit `index` of the tile base (kind 2) at that point of the stage; slot is
// the pass's measurement slot (one-workgroup plans: unused).  In all-site
// profile plans every site has its own kOpMeas and aux also holds
// (norm slot + 1) << 14 | site << 17; norm slot + 1 = 0 when this observable
// does not also carry the norm.
// 32 (48) bytes, so that a record is one aligned scalar load.
template <typename T>
struct alignas(sizeof(T) == 4 ? 32 : 16) DevOp {
    T t, s, nt, ns;
    int32_t code;
    int32_t aux;
};

// One stage: the amplitudes of a tile are gathered from LDS into registers
// (thread bit q and register bit q of a lane hold one tile-local position
// each), the stage's ops run on registers, and the registers are scattered
// back.  Ops that exchange a register bit with lane bit 4 or 5 leave other
// positions there: gt_in/gr_in describe the stage's entry, gt_out/gr_out its
// exit.  tmask/rbit are the layout of passes that keep one layout for all
// stages (bits xor-ed).
struct DevStage {
    int32_t op0, nop;         // op range
    int32_t xnext;            // 1: the exchange after this stage moves amplitudes between
                              // waves (workgroup barrier); 0: within each wave only;
                              // kNoExchange (one-workgroup plans): there is none
    int32_t pad_;
    uint32_t tmask[16];       // LDS byte offset of thread bit q (zero past the last)
    uint32_t rbit[8];         // LDS byte offset of register bit q
    // Exchange through per-lane slots after this stage: LDS byte weight of
    // thread bit q / register bit q of the next stage's entry (see
    // exchange_row_slots).
    uint32_t gw[10], gr[6];
    // Global element offsets of thread bit q / register bit q, for the first
    // stage of a pass (loaded straight from HBM, input layout, entry) and the
    // last (stored straight to HBM, output layout, exit).  One-workgroup plans:
    // offsets in the state, where it is staged through LDS.
    int64_t gt_in[16], gr_in[8], gt_out[16], gr_out[8];
};

constexpr int32_t kNoExchange = 2;

// One tiled pass over the whole state.
struct DevPass {
    int32_t k;                // tile bits
    int32_t stage0, nstage;   // stage range (at least one stage)
    int32_t writes;           // 0: read-only pass (observable only)
    int32_t nfree;            // number of non-tile bits
    int32_t nmeas;            // measurements in this pass
    int32_t tile_barrier;     // 1: workgroup barrier after each tile's stores
    int32_t half;             // 1: half-tile exchanges (the top register bit of every stage
                              // is the same tile position, which has no LDS image)
    int64_t meas_step[kMaxMeas];   // step label of measurement slot m (plus launch offset)
    int64_t free_mask;        // mask of the global bits not in the tile
    int32_t tbit[16];         // global bit of tile-local position p (input layout)
    int32_t tbit_out[16];     // global bit of tile-local position p (output layout)
    // All-site profile plans: per-site measurement slots and norm slots.
    int32_t pmeas, pnorm;
    int64_t pmeas_step[kMaxMeasProfile];   // step label of slot m
    int8_t pmeas_site[kMaxMeasProfile];    // site of slot m
    int32_t pnorm_meas[kMaxMeas];          // measurement slot whose step the norm slot carries
};

// Per-lane LDS slots of an exchange.  The amplitude that lane `tid` holds in
// register j (in a half-tile exchange: of the half's registers) goes to slot
//     j * exchange_row_slots + tid + (tid >> P),
// P = 5 for 8-byte and 4 for 16-byte amplitudes: an address of the lane's own
// plus a constant per register, so the scatter needs no address arithmetic.
// The next stage's lanes gather with one weight per thread and register bit,
// added up.  Modulo the 2^P slots of a 256-byte bank row, lane bits 0 to 3 (3
// are enough at P = 4) and register bits 0, 1, 2, .. weigh 1, 2, 4, 8, .., lane
// and wave bits from P on start again at 1: any four positions get distinct
// weights by ordering the registers and lanes of the stage before, which makes
// the gather's groups of 16 lanes conflict-free.
SPIN_HD constexpr int exchange_pad_shift(int elem_bytes) { return elem_bytes == 8 ? 5 : 4; }
SPIN_HD constexpr int exchange_slot(int tid, int elem_bytes) {
    return tid + (tid >> exchange_pad_shift(elem_bytes));
}
SPIN_HD constexpr int exchange_row_slots(int nt, int elem_bytes) {
    const int n = 1 << exchange_pad_shift(elem_bytes);
    return (exchange_slot(nt - 1, elem_bytes) + n - 1) / n * n + 1;
}

// Whether a gang's member still waits: its counter of arrivals has not reached
// `target`, the arrivals up to this meeting.  Both wrap after 2^32 arrivals (a
// gang of 512 makes that many in 8.4 million meetings); at most a gang's
// arrivals apart, their difference does not.
SPIN_HD constexpr bool gang_waits(uint32_t arrived, uint32_t target) { return int32_t(arrived - target) < 0; }

// Bound of a member's wait.  Before a gang's first meeting a member may wait for
// others that are still busy with earlier problems, as long as those take, so the
// time counts from the last progress anywhere in the launch (meetings passed,
// one-workgroup problems ended and steps of theirs).
constexpr uint64_t kGangWaitTicks = 20ull * 100000000ull;   // 20 s of the 100 MHz real-time counter
struct GangClock {
    uint64_t since;
    uint32_t seen = 0;
    SPIN_HD constexpr bool due(uint64_t now) const { return now - since > kGangWaitTicks; }
    // To be asked with the launch's progress when due: whether it stands still.
    SPIN_HD constexpr bool stalled(uint64_t now, uint32_t progress) {
        if (progress == seen) return true;
        seen = progress;
        since = now;
        return false;
    }
};

// The integers that a batch launch's workgroups share: the error flag, their
// number, the movements of one-workgroup problems, and a counter of arrivals per
// gang.  One array, so that the kernel keeps one pointer.
constexpr int kSyncError = 0, kSyncCount = 1, kSyncProgress = 2, kSyncGangs = 3;

// LDS slots of a workgroup that holds a whole state, 2^r amplitudes on each of
// nt lanes: it is exchanged in padded rows and staged in memory order.
SPIN_HD constexpr int resident_slots(int r, int nt, int elem_bytes) {
    const int rows = exchange_row_slots(nt, elem_bytes) << r, order = nt << r;
    return rows > order ? rows : order;
}

// Register bits and lanes of the batch kernel's tiles (see batch_shape).
SPIN_HD constexpr int batch_regs(bool f32, bool half) { return (f32 ? 5 : 4) + (half ? 1 : 0); }
SPIN_HD constexpr int batch_lanes(bool half) { return half ? 256 : 512; }
// Amplitudes per lane, as a power of two, of its one-workgroup problems: 16, and
// 32 for M = 13 on 256 lanes.
SPIN_HD constexpr int batch_resident_regs(int M, bool half) { return half && M > 12 ? 5 : 4; }
// LDS slots of the batch kernel: the tiles of its gangs (whole ones in one
// layout, or half of them in padded rows) and its one-workgroup problems, up to
// half a tile.
SPIN_HD constexpr int batch_lds_slots(bool f32, bool half) {
    const int eb = f32 ? 8 : 16, r = batch_regs(f32, half), nt = batch_lanes(half);
    const int tile = half ? exchange_row_slots(nt, eb) << (r - 1) : nt << r;
    const int most = f32 ? 13 : 12;
    const int whole = resident_slots(batch_resident_regs(most, half), nt, eb);
    return tile > whole ? tile : whole;
}

}  // namespace spinqp
