// rsos.hip -- host runtime and C ABI of librsos.so (see include/rsos.h).
//
// Launch plan per sweep: one block_sweep launch over every tile block of
// every active surface (the last block of each surface also folds its
// exact sums into the per-sweep log), or, where a launch's latency is the
// bound, one block_sweep2 launch for two sweeps.  The kernels read the
// surface time t from device memory, so a captured hipGraph of K sweeps
// replays for any t.  Surfaces whose L^2 int32 fit in LDS run all their
// sweeps in one lds_run launch instead.
#include "rsos.h"
#include "rsos_host.hpp"
#include "rsos_kernels.hpp"
#include "rsos_moments.hpp"
#include "rsos_ms.hpp"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <deque>
#include <map>
#include <new>
#include <string>
#include <vector>

using rsosk::SurfDev;
using rsosh::check_overflow;
using rsosh::fail;
using rsosh::g_last_error;
using rsosh::validate_h0;
using rsosh::w2_of;

namespace {

// Every HIP runtime call of the library goes through HIP_TRY.  A test can
// make the n-th next one on its thread report a failure (rsos_debug_fail)
// to exercise the error paths without a real device error.
#define HIP_TRY(expr)                                                                       \
    do {                                                                                    \
        if (rsosh::g_fail_countdown > 0 && --rsosh::g_fail_countdown == 0)                  \
            return fail(RSOS_E_DEVICE, "%s: failure injected by rsos_debug_fail", #expr);   \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess) return fail(RSOS_E_DEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr int kLdsMaxBytes = 64 * 1024;  // surfaces of at most this many bytes of int32 run whole in LDS
constexpr int kGraphSweeps = 32;
constexpr long long kNoEnd = 0x7FFFFFFFFFFFFFFFll;  // t_end of a surface with no bound
constexpr long long kBesideSweeps = 4;  // least sweeps for which a batch's LDS path takes a stream of its own
constexpr int kCUs = 256;           // of an MI355X
constexpr size_t kLdsOfCU = 160 * 1024, kLdsStatic = 1024;  // LDS of a CU; of an LDS-path kernel's static arrays, at most about
constexpr int kPsGrid = 2048;       // workgroups of the power-sum reduction
constexpr size_t kStagingBytes = 4096;      // least size of a pinned staging buffer
constexpr long long kReadRecords = 1 << 15; // most log records copied at once (768 KiB pinned)

// ---------------------------------------------------------------------------
// Block-kernel variants.  The tile block shape never changes results.  On
// int32 storage a shape serves every lattice of at least its tiles and its
// region's sites a side (where it does not divide them, the last blocks
// overlap the ones before); on 16-bit storage T % TX == 0 and T % TY == 0.
// ---------------------------------------------------------------------------
// e0 / e1: events recorded by the runtime when the kernel starts / ends
// (hipExtLaunchKernel), for the timing mode; nullptr otherwise.
typedef void (*BlockLaunch)(dim3, hipStream_t, SurfDev *, int, const int *, int, int, hipEvent_t, hipEvent_t);

// E: LDS element type; EW: wider type for the blocks whose range does not
// fit E (void: E always fits); SCHED 1: the double-tiling schedule
template <int D, int TX, int TY, int NT, typename E, typename EW, int SCHED>
void launch_block(dim3 grid, hipStream_t st, SurfDev *d, int n, const int *owner, int xmode, int xnbx, hipEvent_t e0,
                  hipEvent_t e1)
{
    if (e0 || e1)
        hipExtLaunchKernelGGL((rsosk::block_sweep<D, TX, TY, NT, E, EW, SCHED>), grid, dim3(NT), 0, st, e0, e1, 0, d,
                              n, owner, xmode, xnbx);
    else
        hipLaunchKernelGGL((rsosk::block_sweep<D, TX, TY, NT, E, EW, SCHED>), grid, dim3(NT), 0, st, d, n, owner,
                           xmode, xnbx);
}

template <int D, int TX, int TY, int NT>
void launch_block16(dim3 grid, hipStream_t st, SurfDev *d, int n, const int *owner, int xmode, int xnbx, hipEvent_t e0,
                    hipEvent_t e1)
{
    if (e0 || e1)
        hipExtLaunchKernelGGL((rsosk::block_sweep16<D, TX, TY, NT>), grid, dim3(NT), 0, st, e0, e1, 0, d, n, owner,
                              xmode, xnbx);
    else
        hipLaunchKernelGGL((rsosk::block_sweep16<D, TX, TY, NT>), grid, dim3(NT), 0, st, d, n, owner, xmode, xnbx);
}

// The double-tiling schedule is built for the domain sizes the paper
// compares (8 and 16) on int32 storage.
template <int D, int TX, int TY, int NT, typename E, typename EW>
constexpr BlockLaunch dt_launcher()
{
    if constexpr (D == 8 || D == 16) return launch_block<D, TX, TY, NT, E, EW, 1>;
    else return nullptr;
}

struct Variant {
    int D, TX, TY, NT, elem;  // elem: LDS bytes per site (1 and 2: offsets from a block reference)
    BlockLaunch launch;       // int32 storage (elem 1: int16 sub-blocks where int8 does not fit)
    BlockLaunch launch16;     // 16-bit storage, uint8 staging with int16 sub-blocks (nullptr: not offered)
    BlockLaunch launch_dt;    // double-tiling schedule, int32 storage (nullptr: not offered)
    bool steps = false;       // attempts in steps: for launches that leave most lanes idle
};

#define P16(D, TX, TY, NT) launch_block16<D, TX, TY, NT>
#define V8(D, TX, TY, NT)                                                                     \
    {D, TX, TY, NT, 1, launch_block<D, TX, TY, NT, int8_t, int16_t, 0>, P16(D, TX, TY, NT),    \
     dt_launcher<D, TX, TY, NT, int8_t, int16_t>()}
#define V8N(D, TX, TY, NT)                                                                     \
    {D, TX, TY, NT, 1, launch_block<D, TX, TY, NT, int8_t, int16_t, 0>, nullptr,                \
     dt_launcher<D, TX, TY, NT, int8_t, int16_t>()}
#define V16(D, TX, TY, NT) \
    {D, TX, TY, NT, 2, launch_block<D, TX, TY, NT, int16_t, void, 0>, nullptr, dt_launcher<D, TX, TY, NT, int16_t, void>()}
#define V16P(D, TX, TY, NT) \
    {D, TX, TY, NT, 2, launch_block<D, TX, TY, NT, int16_t, void, 0>, P16(D, TX, TY, NT), \
     dt_launcher<D, TX, TY, NT, int16_t, void>()}
#define V32(D, TX, TY, NT) \
    {D, TX, TY, NT, 4, launch_block<D, TX, TY, NT, int32_t, void, 0>, nullptr, dt_launcher<D, TX, TY, NT, int32_t, void>()}
// Attempts in steps (int16 staging): checkerboard on int32 storage only.
#define VS(D, TX, TY, NT) {D, TX, TY, NT, 2, launch_block<D, TX, TY, NT, int16_t, void, 2>, nullptr, nullptr, true}
// In order of preference; without a tuned choice the first one that fits
// every surface is used.
// (V8N: the same int8 kernel without a 16-bit storage instance, where a
// V16P entry of the same shape already provides it.)  The autotuner times
// every entry that fits.
const Variant kVariants[] = {
    V16P(2, 32, 32, 256), V32(2, 16, 16, 128), V32(2, 2, 2, 64), V8(2, 64, 32, 256),
    V16P(4, 16, 16, 128), V32(4, 16, 16, 128), V32(4, 2, 2, 64), V8(4, 32, 16, 256),
    V8(8, 32, 8, 256), V16P(8, 16, 8, 128), V16(8, 8, 8, 64), V32(8, 16, 8, 128),
    V32(8, 8, 8, 64), V32(8, 2, 2, 64), V8(8, 16, 16, 256), V8N(8, 16, 8, 128),
    V16P(16, 4, 4, 64), V32(16, 4, 4, 64), V32(16, 2, 2, 64), V8(16, 4, 4, 64), V8(16, 8, 8, 256),
    V8(32, 2, 2, 64), V32(32, 2, 2, 64),
    VS(8, 8, 8, 256), VS(8, 16, 8, 512), VS(16, 4, 4, 384),
};
#undef P16
#undef V8
#undef V8N
#undef V16
#undef V16P
#undef V32
#undef VS

bool variant_fits(const Variant &v, int L, int N, bool packed, bool dt = false)
{
    if (dt && (packed || !v.launch_dt)) return false;
    const int T = L / v.D;
    const int rw = v.TX * v.D + 2 * (v.D + 1), rh = v.TY * v.D + 2 * (v.D + 1);
    const int rwl = packed ? (rw + 14) & ~7 : (rw + 6) & ~3;
    if (T < v.TX || T < v.TY || rh > L) return false;
    // 16-bit storage keeps to the lattices that the shape tiles
    if (packed && (T % v.TX != 0 || T % v.TY != 0)) return false;
    // a region wider than the lattice only for a block as wide as the
    // lattice (its ring columns are copies of its own far edge, recomputed
    // from the same inputs)
    if (rwl > L && !(v.TX * v.D == L && rwl <= 2 * L)) return false;
    // int16 staging: every staged value within 32767 of the block reference
    // (the int16 sub-blocks of a block that int8 staging does not fit are
    // smaller than the block, so the block's bound covers them)
    const bool i16_ok = (long long)N * (rw + rh + 4) + v.D * v.D <= 32767;
    // 16-bit storage: uint8 staging (N D <= 96) and the int16 sub-blocks
    if (packed) return v.launch16 && L % 8 == 0 && (long long)N * v.D <= 96 && i16_ok;
    if (v.elem == 2 && !i16_ok) return false;
    // int8 staging: the sweep's growth N D must leave room in the byte
    if (v.elem == 1 && ((long long)N * v.D > 96 || !i16_ok)) return false;
    return true;
}

// Blocks of a variant along one side of T tiles.
int blocks_along(int T, int tiles) { return (T + tiles - 1) / tiles; }

// The variant for D without a tuned choice: the first one that fits every
// (L, N) and sweeps at most 4/3 of its tiles (blocks that overlap at the
// lattice's edges sweep tiles twice; the variants' own times differ by less
// than that), else the fitting one that stages the fewest sites.
// (Optionally forced by the RSOS_VARIANT environment variable
// "TXxTYxNTxELEM", e.g. "16x8x128x2"; ELEM is 16 for the 16-bit storage
// kernels.)
const Variant *pick_variant(int D, const std::vector<std::pair<int, int>> &LN, bool packed = false,
                            bool dt = false)
{
    const char *force = getenv("RSOS_VARIANT");
    // Attempts in steps where a whole sweep is at most one such workgroup
    // per CU: L = 256 18.2 -> 14.0 us per sweep, L = 1024 20.6 -> 16.8,
    // L = 1360 20.6 -> 18.4 (16 x 8 blocks), D = 16, L = 1024: 54.8 -> 29.0.
    // With more blocks the lists cost more than the idle lanes: 64 surfaces
    // of L = 256, four 8 x 8 blocks per CU, 21.1 -> 31.3.
    if (!force && !packed && !dt)
        for (const Variant &v : kVariants) {
            if (v.D != D || !v.steps) continue;
            bool ok = true;
            long long blocks = 0;
            for (auto &ln : LN) {
                ok = ok && variant_fits(v, ln.first, ln.second, false, false);
                blocks += (long long)blocks_along(ln.first / D, v.TX) * blocks_along(ln.first / D, v.TY);
            }
            if (ok && blocks <= kCUs) return &v;
        }
    const Variant *least = nullptr;
    double least_staged = 0;
    for (const Variant &v : kVariants) {
        if (v.D != D || (v.steps && !force)) continue;
        if (force) {
            char want[48];
            snprintf(want, sizeof want, "%dx%dx%dx%d", v.TX, v.TY, v.NT, packed ? 16 : v.elem);
            if (strcmp(force, want) != 0) continue;
        }
        bool ok = true;
        double tiles = 0, blocks = 0;
        for (auto &ln : LN) {
            ok = ok && variant_fits(v, ln.first, ln.second, packed, dt);
            const int T = ln.first / D;
            tiles += (double)T * T;
            blocks += (double)blocks_along(T, v.TX) * blocks_along(T, v.TY);
        }
        if (!ok) continue;
        if (3 * blocks * v.TX * v.TY <= 4 * tiles) return &v;
        const double staged = blocks * (v.TX * D + 2 * (D + 1)) * (v.TY * D + 2 * (D + 1));
        if (!least || staged < least_staged) {
            least = &v;
            least_staged = staged;
        }
    }
    return least;
}

// Block shapes of the launches of two sweeps (int32 storage, tile
// checkerboard, D = 8), each for up to per_cu blocks per CU, in order of the
// time that a pair takes at that count.  Per sweep, two per launch against
// one (us):
//     8 x 8 in steps      L = 256: 11.3 / 13.9, L = 512: 11.5 / 14.2, L = 1024: 12.9 / 17.1
//                         (without steps, 32 x 8 tiles: 16.5 at 512, 17.0 at 1024)
//     32 x 8,  1 per CU   L = 1360: 16.7 / 18.8, L = 2048: 18.8 / 23.2, 64 surfaces of 256: 18.9 / 20.7
//     32 x 16, 1 per CU   L = 2560: 22.8 / 27.4, 8 surfaces of 1024: 23.3 / 28.7
//     32 x 8,  3 per CU   L = 3072: 32.7 / 34.6
//     32 x 16, 2 per CU   L = 4096: 36.4 / 42.4, 64 surfaces of 512: 35.6 / 43.1
// With more blocks the attempts themselves are the bound, of which a pair
// makes more: L = 5120 60.9 / 59.3, L = 8192 118.4 / 116.5, L = 16384
// 431 / 406.
struct Pair {
    int D, TX, TY, NT, per_cu;
    bool steps;  // attempts in steps
    void (*launch)(dim3, hipStream_t, SurfDev *, int, const int *, int, int);
};

template <int D, int TX, int TY, int NT, bool STEPS>
void launch_pair(dim3 grid, hipStream_t st, SurfDev *d, int n, const int *owner, int xmode, int xnbx)
{
    hipLaunchKernelGGL((rsosk::block_sweep2<D, TX, TY, NT, STEPS>), grid, dim3(NT), 0, st, d, n, owner, xmode, xnbx);
}

#define PAIR(D, TX, TY, NT, PER, STEPS) {D, TX, TY, NT, PER, STEPS, launch_pair<D, TX, TY, NT, STEPS>}
const Pair kPairs[] = {PAIR(8, 8, 8, 512, 1, true), PAIR(8, 32, 8, 256, 1, false), PAIR(8, 32, 16, 512, 1, false),
                       PAIR(8, 32, 8, 256, 3, false), PAIR(8, 32, 16, 512, 2, false)};
#undef PAIR

bool pair_fits(const Pair &q, int L, int N)
{
    const int ring = 2 * (q.D + 1), rw = (q.TX + rsosk::kTwoMargin) * q.D + ring, rh = (q.TY + rsosk::kTwoMargin) * q.D + ring;
    const int rwl = (rw + 6) & ~3;
    // (as in variant_fits)
    if (L < q.TX * q.D || rh > L || (rwl > L && !(q.TX * q.D == L && rwl <= 2 * L))) return false;
    return (q.steps || 2ll * N * q.D <= 96) && (long long)N * (rw + rh + 4) + 2 * q.D * q.D <= 32767;
}

// Whether row q takes the surfaces (L, N) in one launch.
bool pair_takes(const Pair &q, const std::vector<std::pair<int, int>> &LN)
{
    bool ok = true;
    long long blocks = 0;
    for (auto &ln : LN) {
        ok = ok && pair_fits(q, ln.first, ln.second);
        blocks += (long long)blocks_along(ln.first / q.D, q.TX) * blocks_along(ln.first / q.D, q.TY);
    }
    return ok && blocks <= q.per_cu * kCUs;
}

// The shape for two sweeps per launch of surfaces (L, N), or nullptr (also
// where RSOS_VARIANT names the kernel to run).
const Pair *pick_pair(int D, const std::vector<std::pair<int, int>> &LN)
{
    if (getenv("RSOS_VARIANT")) return nullptr;
    for (const Pair &q : kPairs)
        if (q.D == D && pair_takes(q, LN)) return &q;
    return nullptr;
}

// The blocks of shape q of a surface.
int pair_blocks(const Pair &q, int T) { return blocks_along(T, q.TX) * blocks_along(T, q.TY); }

bool uses_lds(int L);

// 16-bit storage is exact while every height of a sweep stays within 2^15
// of floor(mean): N L <= 32766 (the torus spread is at most N L, the mean
// moves by at most one per sweep).
rsos_status check_packed(const rsos_params *p)
{
    if (uses_lds(p->L))
        return fail(RSOS_E_INVAL, "16-bit storage: L=%d is small enough for the LDS path, which keeps int32", p->L);
    if ((long long)p->N * p->L > 32766)
        return fail(RSOS_E_INVAL, "16-bit storage needs N*L <= 32766 (N=%d, L=%d)", p->N, p->L);
    if (!pick_variant(p->D, {{p->L, p->N}}, true))
        return fail(RSOS_E_INVAL, "16-bit storage: no tile-block shape fits L=%d, N=%d, D=%d", p->L, p->N, p->D);
    return RSOS_OK;
}

// How a launch runs surfaces that live in LDS: attempts in steps, with the
// next sweep's steps laid out ahead where that is offered or with one phase's
// at a time (lds_run), or one lane per tile (lds_run32).
enum class LdsMode { kAhead, kSteps, kLane };
struct LdsPlan {
    LdsMode mode = LdsMode::kLane;
    size_t bytes = 0;  // of dynamic LDS per workgroup
};
typedef void (*LdsLaunch)(dim3, const LdsPlan &, hipStream_t, SurfDev *, const int *);
template <int D, int SCHED>
void launch_lds(dim3 grid, const LdsPlan &pl, hipStream_t st, SurfDev *d, const int *w)
{
    constexpr int NT = rsosk::kLdsThreads;
    if (pl.mode == LdsMode::kLane)
        hipLaunchKernelGGL((rsosk::lds_run32<D, 256, SCHED>), grid, dim3(256), pl.bytes, st, d, w);
    else if constexpr (D > 2) {
        if (pl.mode == LdsMode::kAhead) hipLaunchKernelGGL((rsosk::lds_run<D, NT, SCHED>), grid, dim3(NT), pl.bytes, st, d, w);
        else hipLaunchKernelGGL((rsosk::lds_run<D, NT, SCHED, false>), grid, dim3(NT), pl.bytes, st, d, w);
    }
}
LdsLaunch lds_launcher(int D, int sched = 0)
{
    if (sched == 1) {
        switch (D) {
        case 8: return launch_lds<8, 1>;
        case 16: return launch_lds<16, 1>;
        }
        return nullptr;
    }
    switch (D) {
    case 2: return launch_lds<2, 0>;
    case 4: return launch_lds<4, 0>;
    case 8: return launch_lds<8, 0>;
    case 16: return launch_lds<16, 0>;
    case 32: return launch_lds<32, 0>;
    }
    return nullptr;
}

// The steps are for few tiles with long chains of attempts: where small tiles
// fill the lanes, one lane each does better (us per sweep, steps / one lane:
// D = 2, L = 32: 3.6 / 3.2, L = 128: 21.0 / 15.2; D = 4, L = 16: 4.0 / 5.8,
// L = 32: 4.2 / 6.0, L = 64: 7.2 / 6.7, L = 128: 19.0 / 13.2; D = 8, L = 128:
// 14.6 / 24.2).
bool lds_wide(int D, int L, int N)
{
    return D == 2 || (D == 4 && L > 32) || (long long)N * L > rsosk::kLdsRunMaxNL;
}

// LDS of one workgroup that runs a surface of side L.
size_t lds_bytes_of(int D, int sched, int L, LdsMode mode)
{
    if (mode == LdsMode::kLane) return (size_t)L * L * 4;
    const int ph = sched == 1 ? 4 : 2;
    const bool ahead = mode == LdsMode::kAhead;
    switch (D) {
    case 4: return (size_t)(ahead ? rsosk::LdsRun<4>::bytes(L, ph) : rsosk::LdsRun<4, false>::bytes(L, ph));
    case 8: return (size_t)(ahead ? rsosk::LdsRun<8>::bytes(L, ph) : rsosk::LdsRun<8, false>::bytes(L, ph));
    case 16: return (size_t)(ahead ? rsosk::LdsRun<16>::bytes(L, ph) : rsosk::LdsRun<16, false>::bytes(L, ph));
    }
    return (size_t)(ahead ? rsosk::LdsRun<32>::bytes(L, ph) : rsosk::LdsRun<32, false>::bytes(L, ph));
}

// What a sweep of one surface takes alone on its CU, by mode (us; columns:
// L up to 64, 80, 96, 112, 128), and the workgroups per CU that the registers
// allow.  Measured with 256 surfaces of one size per launch.
struct LdsCost {
    int D, sched, steps_per_cu, lane_per_cu;
    float ahead, steps[5], lane[5];
};
const LdsCost kLdsCosts[] = {
    {4, 0, 2, 4, 4.6f, {6.2f, 6.2f, 6.2f, 6.2f, 6.2f}, {6.6f, 6.6f, 6.6f, 6.6f, 6.6f}},  // (in steps up to L = 32 only)
    {8, 0, 3, 8, 7.6f, {10.5f, 11.4f, 12.3f, 14.5f, 15.9f}, {23.f, 21.6f, 25.5f, 25.8f, 26.8f}},
    {8, 1, 3, 8, 12.3f, {17.8f, 18.7f, 19.3f, 20.3f, 20.9f}, {45.f, 45.f, 40.f, 42.f, 43.f}},
    {16, 0, 2, 4, 19.f, {20.f, 23.f, 25.8f, 28.f, 29.9f}, {76.f, 76.f, 76.f, 76.f, 76.f}},
    {16, 1, 2, 4, 32.f, {34.f, 36.f, 38.4f, 42.f, 45.f}, {152.f, 152.f, 152.f, 152.f, 152.f}},
    {32, 0, 3, 8, 70.f, {71.f, 72.f, 73.f, 73.f, 74.f}, {355.f, 355.f, 355.f, 355.f, 355.f}},
};

// The plan of one launch of surfaces (L, N): the mode with the least time by
// the table.  A workgroup makes all its sweeps before the next takes its
// place, so beyond what is resident at once the launch takes rounds (a last
// one with fewer workgroups per CU is the shorter), and one of several
// workgroups per CU takes c times as long.  The
// steps are the shorter chain, but need more LDS and registers: with the
// lists of two sweeps (ahead) 90 KB at L = 64, one workgroup per CU, with one
// phase's 41 KB, three, with one lane per tile 16 KB, eight.  Measured, us per
// sweep of the launch (ahead / steps / one lane; D = 8):
//     L = 32:  n = 256 7.4 / 10.2 / 23.0, 1024 14.4 / 20.1 / 25.4, 4096 43 / 58 / 58
//     L = 64:  n = 256 8.2 / 10.7 / 22.9, 768 22.5 / 14.1 / 23.3, 1024 29.2 / 22.0 / 23.5, 2048 57 / 37 / 32, 4096 114 / 68 / 60
//     L = 80:  n = 768 - / 23.2 / 24.7, 1024 - / 27.3 / 25.1, 4096 - / 101 / 77
//     L = 112: n = 512 - / 27.8 / 31.7, 768 - / 41.5 / 33.3, 4096 - / 211 / 163
//     L = 128: n = 256 - / 15.9 / 26.9, 1024 - / 58.5 / 62.5, 4096 - / 231 / 232
//     n each of L = 32 and 64: 342 21.5 / 13.6 / 24.4, 1024 54.5 / 33.6 / 31.6
//     n each of L = 32, 64, 128: 1024 112 / 133 / 157
// and D = 16, L = 64, n = 1024: 79 / 45 / 98, D = 4, L = 32: n = 512 5.9 / 7.2 / 7.4, 1024 10.5 / 13.2 / 8.9.
LdsPlan lds_plan(int D, int sched, const std::vector<std::pair<int, int>> &LN)
{
    const LdsCost *cost = nullptr;
    for (const LdsCost &c : kLdsCosts)
        if (c.D == D && c.sched == sched) cost = &c;
    for (auto &x : LN)
        if (lds_wide(D, x.first, x.second)) cost = nullptr;
    LdsPlan best;
    double best_time = 0.0;
    for (LdsMode mode : {LdsMode::kAhead, LdsMode::kSteps, LdsMode::kLane}) {
        if (!cost && mode != LdsMode::kLane) continue;  // one lane per tile only
        LdsPlan pl;
        pl.mode = mode;
        double sum = 0.0, most = 0.0;
        bool ahead = true;
        for (auto &x : LN) {
            ahead = ahead && x.first <= 64;
            pl.bytes = std::max(pl.bytes, lds_bytes_of(D, sched, x.first, mode));
            if (!cost) continue;
            const int col = x.first <= 64 ? 0 : std::min((x.first - 49) / 16, 4);
            const double t = mode == LdsMode::kLane ? cost->lane[col]
                             : mode == LdsMode::kAhead && x.first <= 64 ? cost->ahead : cost->steps[col];
            sum += t;
            most = std::max(most, t);
        }
        if (!cost) return pl;
        const int fit = std::max(1, std::min((int)(kLdsOfCU / (pl.bytes + kLdsStatic)),
                                             mode == LdsMode::kLane ? cost->lane_per_cu : cost->steps_per_cu));
        const int per_cu = ((int)LN.size() + kCUs - 1) / kCUs, here = std::min(fit, per_cu);
        const double load = (double)per_cu / fit, rounds = std::max(1.0, (std::ceil(load) + load) / 2);
        const double c = here == 1 ? 1.0 : mode == LdsMode::kAhead && here == 2 && ahead ? 1.12 : here == 2 ? 1.25 : 1.3;
        const double time = std::max(most, sum / LN.size() * rounds) * c;
        if (best.bytes == 0 || time < best_time) {
            best = pl;
            best_time = time;
        }
    }
    return best;
}

bool valid_D(int D) { return D == 2 || D == 4 || D == 8 || D == 16 || D == 32; }

rsos_status check_params(const rsos_params *p)
{
    if (!p) return fail(RSOS_E_INVAL, "params is NULL");
    if (!valid_D(p->D)) return fail(RSOS_E_INVAL, "D=%d: must be 2, 4, 8, 16 or 32", p->D);
    if (p->L < 2 * p->D || p->L > 65536 || p->L % (2 * p->D) != 0)
        return fail(RSOS_E_INVAL, "L=%d: must be a multiple of 2D=%d in [2D, 65536]", p->L, 2 * p->D);
    if (p->N < 1) return fail(RSOS_E_INVAL, "N=%d: must be >= 1", p->N);
    if (p->flags & ~(RSOS_FLAG_PACKED16 | RSOS_FLAG_DT4 | RSOS_FLAG_TUNE))
        return fail(RSOS_E_INVAL, "unknown flags 0x%x", (unsigned)p->flags);
    if (p->flags & RSOS_FLAG_DT4) {
        if (p->flags & RSOS_FLAG_PACKED16)
            return fail(RSOS_E_INVAL, "the double-tiling schedule runs on int32 storage");
        if (p->D != 8 && p->D != 16) return fail(RSOS_E_INVAL, "double tiling: D must be 8 or 16");
        if (!uses_lds(p->L) && !pick_variant(p->D, {{p->L, p->N}}, false, true))
            return fail(RSOS_E_INVAL, "double tiling: no tile-block shape fits L=%d, N=%d", p->L, p->N);
    }
    if (p->flags & RSOS_FLAG_PACKED16) return check_packed(p);
    return RSOS_OK;
}

bool uses_lds(int L) { return (long long)L * L * 4 <= kLdsMaxBytes; }

// Pinned staging for small host->device descriptor updates; the event makes
// sure the previous copy is done before the buffer is rewritten.
struct Staging {
    void *host = nullptr;
    size_t bytes = 0;
    hipEvent_t done = nullptr;
    bool pending = false;

    rsos_status ensure(size_t n)
    {
        if (!done) HIP_TRY(hipEventCreateWithFlags(&done, hipEventDisableTiming));
        if (pending) {
            HIP_TRY(hipEventSynchronize(done));
            pending = false;
        }
        if (n > bytes) {
            if (host) HIP_TRY(hipHostFree(host));
            host = nullptr;
            n = std::max(n, kStagingBytes);
            HIP_TRY(hipHostMalloc(&host, n, hipHostMallocDefault));
            bytes = n;
        }
        return RSOS_OK;
    }
    // Copies n bytes from the device into the buffer and waits for them and
    // for everything before them on the stream.
    rsos_status copy_from(const void *dev, size_t n, hipStream_t st)
    {
        rsos_status r = ensure(n);
        if (r != RSOS_OK) return r;
        HIP_TRY(hipMemcpyAsync(host, dev, n, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        return RSOS_OK;
    }
    rsos_status copy_to(void *dev, size_t n, hipStream_t st)
    {
        HIP_TRY(hipMemcpyAsync(dev, host, n, hipMemcpyHostToDevice, st));
        HIP_TRY(hipEventRecord(done, st));
        pending = true;
        return RSOS_OK;
    }
    void release()
    {
        if (pending && done) (void)hipEventSynchronize(done);
        if (host) (void)hipHostFree(host);
        if (done) (void)hipEventDestroy(done);
        host = nullptr;
        done = nullptr;
    }
};

}  // namespace

// Block-path surfaces swept by one kernel instance: rows [first, first +
// count) of the descriptor table, blocks numbered from 0 within the shape.
struct Shape {
    const Variant *variant = nullptr;
    int xmode = 1;
    int first = 0, count = 0;
    int total_blocks = 0;
    int *d_owner = nullptr;  // block -> row within the shape (count > 1)
    const Pair *pair = nullptr;  // blocks of its launches of two sweeps (nullptr: none)
    int pair_blocks = 0, pair_xmode = 1;
    int *d_owner2 = nullptr; // as d_owner
};

// A launch choice for one surface: the kernel variant, or the blocks of two
// sweeps per launch (with the first variant that fits for single sweeps), the
// block order and the sweeps per captured graph (none of them changes
// results).
struct Choice {
    const Variant *v = nullptr;
    const Pair *pair = nullptr;
    int xmode = 1;
    int graph_k = 0;
    bool entered = false;  // by rsos_tune_set, not timed

    bool made() const { return v || pair; }
    bool same_kernel(const Choice &o) const { return v == o.v && pair == o.pair && xmode == o.xmode; }
};

// ---------------------------------------------------------------------------
// A group of surfaces sharing one D: the common core of the single-surface,
// batch and engine front ends.
// ---------------------------------------------------------------------------
struct SurfaceGroup {
    int D = 8;
    bool packed = false;               // heights kept as 16-bit residues
    int sched = 0;                     // 0: tile checkerboard, 1: double tiling
    hipStream_t stream = nullptr;
    bool failed = false;
    std::vector<SurfDev> host;         // host mirror (t, t_end kept current)
    std::vector<long long> dev_t_end;  // t_end values last uploaded
    std::vector<long long> max_h0, t0; // per surface
    SurfDev *d_desc = nullptr;
    long long *d_acc = nullptr;        // kAccWords per block-path surface
    std::vector<int32_t *> readout;    // 16-bit storage: int32[L^2] device scratch per surface
    long long *d_ps = nullptr;         // power sums: per-workgroup partials, then the result
    long long *d_rec = nullptr;        // the surfaces' current records (read_widths; batches)
    int xmode = 1;                     // workgroup -> block order (rsosk::block_map) without a choice
    std::vector<Shape> shapes;         // block-path surfaces by kernel instance
    std::vector<Choice> want;          // per surface: a tuned launch choice (or none); read by setup()
    std::vector<int> rows;             // device-table row -> surface index
    std::vector<int> lds_idx, blk_idx; // surfaces on each path
    int *d_lds_idx = nullptr;
    int graph_k = kGraphSweeps;        // sweeps per captured graph
    LdsPlan lds;
    // groups with surfaces on both paths: the LDS path's launch runs beside
    // the tile blocks on a stream of its own, forked from the group's stream
    // and joined to it within the call
    hipStream_t lds_stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    Staging staging;
    bool any_pair = false;             // two sweeps share a launch, in some shape
    hipGraphExec_t graph = nullptr;    // graph_k sweeps that every block-path surface makes
    hipGraphExec_t graph1 = nullptr;   // as many, one per launch, each bounded by t_end (where it differs)
    bool timing = false;                             // bracket block launches with events
    std::vector<std::pair<hipEvent_t, hipEvent_t>> timed;
    std::vector<void *> owned;         // library-owned device allocations

    rsos_status dev_alloc(void **p, size_t n)
    {
        hipError_t e = hipMalloc(p, n);
        if (e != hipSuccess) return fail(RSOS_E_NOMEM, "hipMalloc(%zu): %s", n, hipGetErrorString(e));
        owned.push_back(*p);
        return RSOS_OK;
    }

    // Builds the descriptor table (host side must be filled: buf, log, L, N,
    // key, t, t_end).  Groups the block-path surfaces by kernel instance:
    // each surface's tuned choice where want[] holds one for every
    // block-path surface, else one first-fit variant for all of them.
    rsos_status setup()
    {
        const int n = (int)host.size();
        std::vector<std::pair<int, int>> LN;
        for (int i = 0; i < n; ++i) {
            if (uses_lds(host[i].L)) lds_idx.push_back(i);
            else { blk_idx.push_back(i); LN.push_back({host[i].L, host[i].N}); }
            for (int k = 0; k < 2; ++k)
                if (((uintptr_t)host[i].buf[k] & 15) != 0)
                    return fail(RSOS_E_INVAL, "height buffers must be 16-byte aligned");
        }
        if (packed && !lds_idx.empty()) return fail(RSOS_E_INVAL, "16-bit storage needs the tile-block path");
        if (const char *xm = getenv("RSOS_XMODE")) xmode = atoi(xm) == 0 ? 0 : atoi(xm) == 2 ? 2 : 1;
        bool tuned = !blk_idx.empty() && want.size() == host.size();
        for (int i : blk_idx) tuned = tuned && want[i].made();
        std::vector<std::vector<int>> members;
        if (tuned) {
            for (int i : blk_idx) {
                size_t g = 0;
                while (g < shapes.size() && !want[members[g][0]].same_kernel(want[i])) ++g;
                if (g == shapes.size()) {
                    shapes.push_back(Shape());
                    shapes.back().variant = want[i].v;
                    shapes.back().pair = want[i].pair;
                    shapes.back().xmode = want[i].xmode;
                    members.emplace_back();
                }
                members[g].push_back(i);
            }
            for (size_t g = 0; g < shapes.size(); ++g) {
                if (shapes[g].variant) continue;
                std::vector<std::pair<int, int>> ln;
                for (int i : members[g]) ln.push_back({host[i].L, host[i].N});
                if (!(shapes[g].variant = pick_variant(D, ln))) return fail(RSOS_E_INVAL, "no tile-block shape fits these lattice sizes");
            }
            graph_k = 0;
            for (int i : blk_idx) graph_k = std::max(graph_k, want[i].graph_k);
            if (graph_k < 1) graph_k = kGraphSweeps;
        } else if (!blk_idx.empty()) {
            const Variant *v = pick_variant(D, LN, packed, sched == 1);
            if (!v) return fail(RSOS_E_INVAL, "no tile-block shape fits these lattice sizes");
            shapes.push_back(Shape());
            shapes.back().variant = v;
            if (!packed && sched == 0) shapes.back().pair = pick_pair(D, LN);
            shapes.back().xmode = xmode;
            members.push_back(blk_idx);
        }
        // rows: each shape's surfaces in turn (block numbers restart at 0 in
        // every shape), then the LDS-path surfaces
        rows.clear();
        for (size_t g = 0; g < shapes.size(); ++g) {
            Shape &sh = shapes[g];
            sh.first = (int)rows.size();
            sh.count = (int)members[g].size();
            long long blocks = 0;
            long long blocks2 = 0;
            any_pair = any_pair || sh.pair;
            for (int i : members[g]) {
                SurfDev &sd = host[i];
                const int T = sd.L / D;
                sd.nbx = blocks_along(T, sh.variant->TX);
                sd.nblocks = sd.nbx * blocks_along(T, sh.variant->TY);
                sd.block_start = (int)blocks;
                blocks += sd.nblocks;
                sd.block_start2 = (int)blocks2;
                if (sh.pair) blocks2 += pair_blocks(*sh.pair, T);
                if (blocks > (1ll << 30)) return fail(RSOS_E_INVAL, "too many tile blocks");
                rows.push_back(i);
            }
            sh.total_blocks = (int)blocks;
            sh.pair_blocks = (int)blocks2;
            sh.pair_xmode = sh.xmode == 2 && sh.pair && !(sh.count == 1 && blocks_along(host[members[g][0]].T, sh.pair->TX) % 8 == 0) ? 1 : sh.xmode;
            if (sh.xmode == 2 && !(sh.count == 1 && host[members[g][0]].nbx % 8 == 0)) sh.xmode = 1;
        }
        const int nblk_rows = (int)rows.size();
        for (int i : lds_idx) {
            host[i].nbx = 0;
            host[i].nblocks = 0;
            host[i].block_start = 1 << 30;  // never matched by a block workgroup
            rows.push_back(i);
        }
        rsos_status st;
        if ((st = dev_alloc((void **)&d_desc, sizeof(SurfDev) * n)) != RSOS_OK) return st;
        if (nblk_rows) {
            const size_t bytes = sizeof(long long) * rsosk::kAccWords * nblk_rows;
            if ((st = dev_alloc((void **)&d_acc, bytes)) != RSOS_OK) return st;
            HIP_TRY(hipMemset(d_acc, 0, bytes));
            for (int r = 0; r < nblk_rows; ++r) host[rows[r]].acc = d_acc + rsosk::kAccWords * r;
        }
        for (Shape &sh : shapes) {
            if (sh.count < 2) continue;
            // owner of every block of the shape: its row within the shape
            // (and of every block of two sweeps)
            std::vector<int> own((size_t)sh.total_blocks + sh.pair_blocks);
            for (int k = 0; k < sh.count; ++k) {
                const SurfDev &sd = host[rows[sh.first + k]];
                for (int b = 0; b < sd.nblocks; ++b) own[(size_t)sd.block_start + b] = k;
                for (int b = 0; sh.pair && b < pair_blocks(*sh.pair, sd.T); ++b)
                    own[(size_t)sh.total_blocks + sd.block_start2 + b] = k;
            }
            if ((st = dev_alloc((void **)&sh.d_owner, sizeof(int) * own.size())) != RSOS_OK) return st;
            HIP_TRY(hipMemcpy(sh.d_owner, own.data(), sizeof(int) * own.size(), hipMemcpyHostToDevice));
            sh.d_owner2 = sh.d_owner + sh.total_blocks;
        }
        if (!lds_idx.empty()) {
            if ((st = dev_alloc((void **)&d_lds_idx, sizeof(int) * lds_idx.size())) != RSOS_OK) return st;
            std::vector<int> pos(lds_idx.size());
            for (size_t k = 0; k < pos.size(); ++k) pos[k] = nblk_rows + (int)k;
            HIP_TRY(hipMemcpy(d_lds_idx, pos.data(), sizeof(int) * pos.size(), hipMemcpyHostToDevice));
            std::vector<std::pair<int, int>> ln;
            for (int i : lds_idx) ln.push_back({host[i].L, host[i].N});
            lds = lds_plan(D, sched, ln);
            if (!blk_idx.empty()) {
                HIP_TRY(hipStreamCreateWithFlags(&lds_stream, hipStreamNonBlocking));
                HIP_TRY(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
                HIP_TRY(hipEventCreateWithFlags(&join, hipEventDisableTiming));
            }
        }
        return upload_all();
    }

    rsos_status upload_all()
    {
        const int n = (int)host.size();
        rsos_status st = staging.ensure(sizeof(SurfDev) * n);
        if (st != RSOS_OK) return st;
        SurfDev *h = (SurfDev *)staging.host;
        for (int k = 0; k < n; ++k) {
            h[k] = host[rows[k]];
            // (most surfaces of a batch are at one time: no division for these)
            h[k].slot = k && h[k].t == h[k - 1].t && h[k].log_cap == h[k - 1].log_cap ? h[k - 1].slot : h[k].t % h[k].log_cap;
        }
        return staging.copy_to(d_desc, sizeof(SurfDev) * n, stream);
    }

    // Sets every surface's end time for the next launch_sweeps(n).  A
    // block-path surface that advances by all n sweeps needs no bound (the
    // launch count is the bound) and keeps an unbounded t_end on the device,
    // so a run of such calls rewrites nothing; the others, and LDS-path
    // surfaces (which run to their t_end in one launch), get their exact
    // t_end.  A rewrite uploads the whole (small) table, t included: the
    // host mirror of t is exact, since sweep counts are deterministic.
    rsos_status set_t_end(const std::vector<long long> &t_end, long long n)
    {
        bool changed = dev_t_end.size() != host.size();
        for (size_t i = 0; i < host.size(); ++i) {
            const bool blk = !uses_lds(host[i].L);
            host[i].t_end = (blk && t_end[i] - host[i].t == n) ? kNoEnd : t_end[i];
            changed = changed || host[i].t_end != dev_t_end[i];
        }
        if (!changed) return RSOS_OK;
        dev_t_end.resize(host.size());
        for (size_t i = 0; i < host.size(); ++i) dev_t_end[i] = host[i].t_end;
        return upload_all();
    }

    rsos_status launch_sweeps(long long n)
    {
        if (n <= 0) return RSOS_OK;
        // Beside the blocks from kBesideSweeps sweeps on: the fork and the join
        // cost about 10 us (2 surfaces of 64 and 256, one sweep 42 -> 55 us),
        // four sweeps take 92 -> 82 us and 64 sweeps 1165 -> 753, 300 surfaces
        // of 64 beside one of 2048 163 -> 128 and 2069 -> 1366.
        // (Where the runtime puts both streams on one hardware queue, 1 of the
        // 12 measured, they run in turn and 304 us become 325.)
        const bool beside = lds_stream && n >= kBesideSweeps;
        if (!lds_idx.empty()) {
            if (beside) {
                HIP_TRY(hipEventRecord(fork, stream));
                HIP_TRY(hipStreamWaitEvent(lds_stream, fork, 0));
            }
            lds_launcher(D, sched)(dim3((unsigned)lds_idx.size()), lds, beside ? lds_stream : stream, d_desc, d_lds_idx);
            HIP_TRY(hipGetLastError());
            if (beside) HIP_TRY(hipEventRecord(join, lds_stream));
        }
        if (blk_idx.empty()) return RSOS_OK;
        // sweeps that every block-path surface makes: only these may be
        // launched two at a time
        long long every = n;
        if (any_pair)
            for (int i : blk_idx) every = std::min(every, host[i].t_end - host[i].t);
        rsos_status st = run_block(every, &graph, any_pair);
        if (st == RSOS_OK) st = run_block(n - every, &graph1, false);
        if (beside) HIP_TRY(hipStreamWaitEvent(stream, join, 0));
        return st;
    }

    // n sweeps of the tile blocks, as replays of a graph of graph_k sweeps
    // where there are enough of them, four: in pairs per launch.
    rsos_status run_block(long long n, hipGraphExec_t *gr, bool four)
    {
        long long left = n;
        if (stream != nullptr && n >= 2 * graph_k && !timing) {
            if (!*gr) {
                rsos_status st = capture_graph(graph_k, gr, four);
                if (st != RSOS_OK) return st;
            }
            for (; left >= graph_k; left -= graph_k) HIP_TRY(hipGraphLaunch(*gr, stream));
        }
        for (; four && !timing && left >= 4; left -= 4) launch_four();
        HIP_TRY(hipGetLastError());
        for (; left > 0; --left) {
            rsos_status st = enqueue_one();
            if (st != RSOS_OK) return st;
        }
        return RSOS_OK;
    }

    // four sweeps of every surface, two per launch where the shape takes them
    void launch_four()
    {
        for (const Shape &sh : shapes) {
            const int nbx2 = sh.count == 1 && sh.pair ? blocks_along(host[rows[sh.first]].T, sh.pair->TX) : 0;
            for (int i = 0; i < 4; ++i)
                if (!sh.pair) launch_shape(sh);
                else if (i % 2 == 0)
                    sh.pair->launch(dim3(sh.pair_blocks), stream, d_desc + sh.first, sh.count, sh.d_owner2, sh.pair_xmode, nbx2);
        }
    }

    void launch_shape(const Shape &sh, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr)
    {
        const Variant *v = sh.variant;
        BlockLaunch k = packed ? v->launch16 : sched == 1 ? v->launch_dt : v->launch;
        const int nbx = sh.count == 1 ? host[rows[sh.first]].nbx : 0;
        k(dim3(sh.total_blocks), stream, d_desc + sh.first, sh.count, sh.d_owner, sh.xmode, nbx, e0, e1);
    }

    // the tile-block sweep proper: one workgroup per block, the whole sweep
    // in one launch per kernel instance
    void launch_block_sweep(hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr)
    {
        for (size_t i = 0; i < shapes.size(); ++i)
            launch_shape(shapes[i], i == 0 ? e0 : nullptr, i + 1 == shapes.size() ? e1 : nullptr);
    }

    rsos_status enqueue_one()
    {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (timing) {
            // recorded by the runtime at the start of the sweep's first
            // kernel and the end of its last
            HIP_TRY(hipEventCreate(&e0));
            HIP_TRY(hipEventCreate(&e1));
            timed.push_back({e0, e1});
        }
        launch_block_sweep(e0, e1);
        HIP_TRY(hipGetLastError());
        return RSOS_OK;
    }

    // Captures the graphs of graph_k sweeps when the group is created, so
    // that no sweep call pays for a capture (surfaces on a stream): the second
    // one for the sweeps that only some of several surfaces make.
    rsos_status prepare_graph()
    {
        if (stream == nullptr || blk_idx.empty() || graph) return RSOS_OK;
        rsos_status st = capture_graph(graph_k, &graph, any_pair);
        if (st == RSOS_OK && any_pair && blk_idx.size() > 1) st = capture_graph(graph_k, &graph1, false);
        return st;
    }

    rsos_status capture_graph(int k, hipGraphExec_t *gr, bool four)
    {
        hipGraph_t g = nullptr;
        HIP_TRY(hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal));
        for (; four && k >= 4; k -= 4) launch_four();
        for (; k > 0; --k) launch_block_sweep();
        HIP_TRY(hipStreamEndCapture(stream, &g));
        HIP_TRY(hipGraphInstantiate(gr, g, nullptr, nullptr, 0));
        HIP_TRY(hipGraphDestroy(g));
        return RSOS_OK;
    }

    // Reads log records of surface i for times [t_from, t_from + n).
    rsos_status read_log(int i, long long t_from, long long n, rsos_width_t *out)
    {
        const SurfDev &s = host[i];
        if (n < 0 || t_from < t0[i] || t_from + n > s.t + 1)
            return fail(RSOS_E_INVAL, "times [%lld, %lld) outside [t0=%lld, t=%lld]", t_from,
                        t_from + n, t0[i], s.t);
        if (t_from + s.log_cap <= s.t && n > 0)
            return fail(RSOS_E_INVAL, "records before t=%lld are no longer kept", s.t - s.log_cap + 1);
        if (n == 0) {
            HIP_TRY(hipStreamSynchronize(stream));
            return RSOS_OK;
        }
        for (long long k = 0; k < n;) {
            const long long slot = (t_from + k) % s.log_cap, run = std::min({n - k, s.log_cap - slot, kReadRecords});
            rsos_status st = staging.copy_from(s.log + 3 * slot, sizeof(long long) * 3 * run, stream);
            if (st != RSOS_OK) return st;
            const long long *r = (const long long *)staging.host;
            for (long long i = 0; i < run; ++i, ++k)
                out[k] = {t_from + k, r[3 * i], r[3 * i + 1], r[3 * i + 2], w2_of(s.L, r[3 * i], r[3 * i + 1])};
        }
        return RSOS_OK;
    }

    // The current record of every surface: gathered into one array on the
    // device and copied once (one copy per surface cost about 12 us each,
    // 3 ms of a 256-surface call).
    rsos_status read_widths(rsos_width_t *out)
    {
        const int n = (int)host.size();
        rsos_status st;
        hipLaunchKernelGGL(rsosk::gather_records, dim3((unsigned)(n + 255) / 256), dim3(256), 0, stream, d_desc, n, d_rec);
        HIP_TRY(hipGetLastError());
        if ((st = staging.copy_from(d_rec, sizeof(long long) * 3 * n, stream)) != RSOS_OK) return st;
        const long long *r = (const long long *)staging.host;
        for (int k = 0; k < n; ++k) {
            const SurfDev &s = host[rows[k]];
            out[rows[k]] = {s.t, r[3 * k], r[3 * k + 1], r[3 * k + 2], w2_of(s.L, r[3 * k], r[3 * k + 1])};
        }
        return RSOS_OK;
    }

    rsos_status copy_heights(int i, int32_t *dst, int dst_is_device)
    {
        const SurfDev &s = host[i];
        const size_t n = (size_t)s.L * s.L;
        if (packed) {
            // residues -> int32 on the device (needs floor(S1 / L^2) of time t)
            int32_t *out = dst_is_device ? dst : readout[i];
            hipLaunchKernelGGL((long long)n > rsosk::kStreamSites ? rsosk::unpack16<true> : rsosk::unpack16<false>,
                               dim3(grid_for(n)), dim3(256), 0, stream,
                               (const uint16_t *)s.buf[s.t & 1], out, (long long)n,
                               (const long long *)(s.acc + rsosk::kMeanWord));
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipStreamSynchronize(stream));
            if (!dst_is_device) HIP_TRY(hipMemcpy(dst, out, n * 4, hipMemcpyDeviceToHost));
            return RSOS_OK;
        }
        HIP_TRY(hipStreamSynchronize(stream));
        HIP_TRY(hipMemcpy(dst, s.buf[s.t & 1], n * 4,
                          dst_is_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost));
        return RSOS_OK;
    }

    // Initial state of surface i into its buffer of parity t: int32 heights
    // from host memory (nullptr: flat), as residues in 16-bit storage, and
    // floor(S1 / L^2) into the accumulator area.
    rsos_status load_initial(int i, const int32_t *h0_host, long long s1)
    {
        const SurfDev &s = host[i];
        const size_t n = (size_t)s.L * s.L;
        int32_t *cur = s.buf[s.t & 1];
        if (!packed) {
            HIP_TRY(h0_host ? hipMemcpyAsync(cur, h0_host, n * 4, hipMemcpyHostToDevice, stream)
                            : hipMemsetAsync(cur, 0, n * 4, stream));
        } else if (h0_host) {
            HIP_TRY(hipMemcpyAsync(readout[i], h0_host, n * 4, hipMemcpyHostToDevice, stream));
            hipLaunchKernelGGL(rsosk::pack16, dim3(grid_for(n)), dim3(256), 0, stream,
                               (const int32_t *)readout[i], (uint16_t *)cur, (long long)n);
            HIP_TRY(hipGetLastError());
        } else {
            HIP_TRY(hipMemsetAsync(cur, 0, n * 2, stream));
        }
        if (s.acc) {
            const long long m0 = s1 / ((long long)s.L * s.L);
            HIP_TRY(hipMemcpyAsync(s.acc + rsosk::kMeanWord, &m0, sizeof m0, hipMemcpyHostToDevice, stream));
        }
        HIP_TRY(hipStreamSynchronize(stream));
        return RSOS_OK;
    }

    static unsigned grid_for(size_t n) { return (unsigned)std::min<size_t>((n + 255) / 256, 8192); }

    // Exact power sums of surface i's current heights about floor(S1/L^2)
    // (rsosk::power_sums_partial / power_sums_final), then the central
    // moments from them.
    rsos_status moments(int i, rsos_moments_t *out)
    {
        const SurfDev &s = host[i];
        const long long n = (long long)s.L * s.L;
        // at most 2^16 sites per thread: grid >= n / 2^24
        const int grid = (int)std::min<long long>(kPsGrid, std::max<long long>(1, n / (256 * 32)));
        rsos_status st;
        if (!d_ps && (st = dev_alloc((void **)&d_ps, sizeof(long long) * (8 * (size_t)kPsGrid + 9))) != RSOS_OK)
            return st;
        const long long *rec = s.log + 3 * (s.t % s.log_cap);
        if (packed)
            hipLaunchKernelGGL(rsosk::power_sums_partial<uint16_t>, dim3(grid), dim3(256), 0, stream,
                               (const uint16_t *)s.buf[s.t & 1], n, rec, d_ps);
        else
            hipLaunchKernelGGL(rsosk::power_sums_partial<int32_t>, dim3(grid), dim3(256), 0, stream,
                               (const int32_t *)s.buf[s.t & 1], n, rec, d_ps);
        HIP_TRY(hipGetLastError());
        long long *total = d_ps + 8 * (size_t)kPsGrid;  // 4 int128, then S1
        hipLaunchKernelGGL(rsosk::power_sums_final, dim3(1), dim3(256), 0, stream, d_ps, grid, rec, total);
        HIP_TRY(hipGetLastError());
        if ((st = staging.copy_from(total, sizeof(long long) * 9, stream)) != RSOS_OK) return st;
        unsigned long long r[9];
        memcpy(r, staging.host, sizeof r);
        __int128 c[4];
        for (int k = 0; k < 4; ++k) c[k] = (__int128)(((unsigned __int128)r[2 * k + 1] << 64) | r[2 * k]);
        out->t = s.t;
        out->ref = (long long)r[8] / n;
        out->c1 = (int64_t)c[0];
        out->c2 = (int64_t)c[1];
        out->c3[0] = r[4];
        out->c3[1] = r[5];
        out->c4[0] = r[6];
        out->c4[1] = r[7];
        // central moments: with d = c1/n in [0, 1), expand (h - ref - d)^k
        const long double N_ = (long double)n, d = (long double)c[0] / N_;
        const long double m2 = (long double)c[1] / N_, m3 = (long double)c[2] / N_, m4 = (long double)c[3] / N_;
        out->phi2 = (double)(m2 - d * d);
        out->phi3 = (double)(m3 - 3 * d * m2 + 2 * d * d * d);
        out->phi4 = (double)(m4 - 4 * d * m3 + 6 * d * d * m2 - 3 * d * d * d * d);
        return RSOS_OK;
    }

    // Writes the initial log record (time t0) of surface i.
    rsos_status init_record(int i, long long s1, long long s2)
    {
        long long rec[3] = {s1, s2, 0};
        const SurfDev &s = host[i];
        HIP_TRY(hipMemcpy(s.log + 3 * (s.t % s.log_cap), rec, sizeof rec, hipMemcpyHostToDevice));
        return RSOS_OK;
    }

    rsos_status read_timing(int64_t *launches, double *mean_ms, double *total_ms)
    {
        HIP_TRY(hipStreamSynchronize(stream));
        double tot = 0.0;
        for (auto &pr : timed) {
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, pr.first, pr.second));
            tot += ms;
        }
        if (launches) *launches = (int64_t)timed.size();
        if (total_ms) *total_ms = tot;
        if (mean_ms) *mean_ms = timed.empty() ? 0.0 : tot / (double)timed.size();
        clear_timing();
        return RSOS_OK;
    }

    void clear_timing()
    {
        for (auto &pr : timed) {
            (void)hipEventDestroy(pr.first);
            (void)hipEventDestroy(pr.second);
        }
        timed.clear();
    }

    void destroy()
    {
        if (stream) (void)hipStreamSynchronize(stream);
        else (void)hipDeviceSynchronize();
        if (lds_stream) {
            (void)hipStreamSynchronize(lds_stream);
            (void)hipStreamDestroy(lds_stream);
        }
        if (fork) (void)hipEventDestroy(fork);
        if (join) (void)hipEventDestroy(join);
        clear_timing();
        if (graph) (void)hipGraphExecDestroy(graph);
        if (graph1) (void)hipGraphExecDestroy(graph1);
        staging.release();
        for (void *p : owned) (void)hipFree(p);
        owned.clear();
    }
};

struct rsos_surface {
    rsos_params p;
    SurfaceGroup g;
};

struct rsos_batch {
    std::vector<rsos_params> p;
    SurfaceGroup g;
};

// ---------------------------------------------------------------------------
// autotuner of the launch knobs -- see rsos_tune.inc
// ---------------------------------------------------------------------------
#include "rsos_tune.inc"

#define CHECK_HANDLE(h, grp)                                                           \
    do {                                                                               \
        if (!(h)) return fail(RSOS_E_INVAL, "NULL handle");                           \
        if ((grp).failed) return fail(RSOS_E_STATE, "handle failed after a device error"); \
    } while (0)

static rsos_status mark(SurfaceGroup &g, rsos_status st)
{
    if (st == RSOS_E_DEVICE) g.failed = true;
    return st;
}

extern "C" {

const char *rsos_version(void) { return "rsos-gfx950 1.0"; }

const char *rsos_strerror(rsos_status st)
{
    switch (st) {
    case RSOS_OK: return "ok";
    case RSOS_E_INVAL: return "invalid argument";
    case RSOS_E_RSOS: return "initial heights violate the RSOS restriction";
    case RSOS_E_OVERFLOW: return "heights or sums could overflow";
    case RSOS_E_DEVICE: return "HIP runtime error";
    case RSOS_E_NOMEM: return "out of memory";
    case RSOS_E_STATE: return "handle failed or call out of sequence";
    case RSOS_E_BUSY: return "no room for the job now";
    }
    return "unknown status";
}

const char *rsos_last_error(void) { return g_last_error.c_str(); }

rsos_status rsos_debug_fail(int32_t after)
{
    if (after < 0) return fail(RSOS_E_INVAL, "after < 0");
    rsosh::g_fail_countdown = after;
    return RSOS_OK;
}

void rsos_philox4x32_10(const uint32_t ctr[4], const uint32_t key[2], uint32_t out[4])
{
    const rsosk::u32x4 r = rsosk::philox4x32_10(ctr[0], ctr[1], ctr[2], ctr[3], key[0], key[1]);
    for (int i = 0; i < 4; ++i) out[i] = r.v[i];
}

double rsos_w2(int32_t L, int64_t s1, int64_t s2) { return w2_of(L, s1, s2); }

rsos_status rsos_init(rsos_surface **out, const rsos_params *p, int32_t *d_h, int32_t *d_work,
                      const int32_t *h0_host, int64_t t0, int64_t log_cap, void *stream)
{
    if (!out) return fail(RSOS_E_INVAL, "out is NULL");
    *out = nullptr;
    rsos_status st = check_params(p);
    if (st != RSOS_OK) return st;
    if (!d_h) return fail(RSOS_E_INVAL, "d_h is NULL");
    if (t0 < 0 || t0 >= (1ll << 32)) return fail(RSOS_E_INVAL, "t0 outside [0, 2^32)");
    if (log_cap < 0) return fail(RSOS_E_INVAL, "log_cap < 0");
    if (log_cap == 0) log_cap = 65536;
    long long max_h = 0, s1 = 0, s2 = 0;
    if (h0_host && (st = validate_h0(h0_host, p->L, p->N, &max_h, &s1, &s2)) != RSOS_OK) return st;
    if ((st = check_overflow(*p, max_h, 0)) != RSOS_OK) return st;

    rsos_surface *s = new (std::nothrow) rsos_surface();
    if (!s) return fail(RSOS_E_NOMEM, "host allocation failed");
    s->p = *p;
    SurfaceGroup &g = s->g;
    g.D = p->D;
    g.packed = (p->flags & RSOS_FLAG_PACKED16) != 0;
    g.sched = (p->flags & RSOS_FLAG_DT4) ? 1 : 0;
    g.stream = (hipStream_t)stream;
    const size_t n = (size_t)p->L * p->L;
    SurfDev d = {};
    int32_t *work = d_work;
    if (!work && (st = g.dev_alloc((void **)&work, n * 4)) != RSOS_OK) { g.destroy(); delete s; return st; }
    if (g.packed) {
        // both residue buffers in d_h; d_work receives int32 heights on readout
        d.buf[0] = d_h;
        d.buf[1] = (int32_t *)((uint16_t *)d_h + n);
        g.readout.push_back(work);
    } else {
        d.buf[0] = d_h;
        d.buf[1] = work;
    }
    if ((st = g.dev_alloc((void **)&d.log, sizeof(long long) * 3 * log_cap)) != RSOS_OK) { g.destroy(); delete s; return st; }
    d.log_cap = log_cap;
    d.t = t0;
    d.t_end = t0;
    d.key0 = (uint32_t)(p->seed & 0xFFFFFFFFu);
    d.key1 = (uint32_t)(p->seed >> 32);
    d.L = p->L;
    d.N = p->N;
    d.T = p->L / p->D;
    g.host.push_back(d);
    g.max_h0.push_back(max_h);
    g.t0.push_back(t0);
    if (tuning_wanted(p) && !uses_lds(p->L)) {
        Choice c;
        if ((st = tuned_choice(p, 0, &c)) != RSOS_OK) { g.destroy(); delete s; return st; }
        g.want.assign(1, c);
    }
    if ((st = mark(g, g.setup())) != RSOS_OK) { g.destroy(); delete s; return st; }
    // initial state into the buffer of parity t0
    if ((st = g.load_initial(0, h0_host, s1)) != RSOS_OK) { g.destroy(); delete s; return st; }
    if ((st = g.init_record(0, s1, s2)) != RSOS_OK) { g.destroy(); delete s; return st; }
    if ((st = mark(g, g.prepare_graph())) != RSOS_OK) { g.destroy(); delete s; return st; }
    *out = s;
    return RSOS_OK;
}

rsos_status rsos_sweep(rsos_surface *s, int64_t n_mcs)
{
    CHECK_HANDLE(s, s->g);
    if (n_mcs < 0) return fail(RSOS_E_INVAL, "n_mcs < 0");
    if (n_mcs == 0) return RSOS_OK;
    SurfaceGroup &g = s->g;
    const long long t = g.host[0].t;
    if (t + n_mcs > (1ll << 32)) return fail(RSOS_E_INVAL, "sweep index would exceed 2^32");
    rsos_status st = check_overflow(s->p, g.max_h0[0], t + n_mcs - g.t0[0]);
    if (st != RSOS_OK) return st;
    if ((st = mark(g, g.set_t_end({t + n_mcs}, n_mcs))) != RSOS_OK) return st;
    if ((st = mark(g, g.launch_sweeps(n_mcs))) != RSOS_OK) return st;
    g.host[0].t = t + n_mcs;
    return RSOS_OK;
}

rsos_status rsos_width(rsos_surface *s, rsos_width_t *out)
{
    CHECK_HANDLE(s, s->g);
    if (!out) return fail(RSOS_E_INVAL, "out is NULL");
    return mark(s->g, s->g.read_log(0, s->g.host[0].t, 1, out));
}

rsos_status rsos_log(rsos_surface *s, int64_t t_from, int64_t n, rsos_width_t *out)
{
    CHECK_HANDLE(s, s->g);
    if (!out && n > 0) return fail(RSOS_E_INVAL, "out is NULL");
    return mark(s->g, s->g.read_log(0, t_from, n, out));
}

rsos_status rsos_heights(rsos_surface *s, int32_t *dst, int dst_is_device)
{
    CHECK_HANDLE(s, s->g);
    if (!dst) return fail(RSOS_E_INVAL, "dst is NULL");
    return mark(s->g, s->g.copy_heights(0, dst, dst_is_device));
}

rsos_status rsos_moments(rsos_surface *s, rsos_moments_t *out)
{
    CHECK_HANDLE(s, s->g);
    if (!out) return fail(RSOS_E_INVAL, "out is NULL");
    return mark(s->g, s->g.moments(0, out));
}

rsos_status rsos_time(rsos_surface *s, int64_t *t, int32_t **d_current)
{
    CHECK_HANDLE(s, s->g);
    const SurfDev &d = s->g.host[0];
    if (t) *t = d.t;
    if (d_current) *d_current = s->g.packed ? nullptr : d.buf[d.t & 1];
    return RSOS_OK;
}

rsos_status rsos_timing(rsos_surface *s, int enable)
{
    CHECK_HANDLE(s, s->g);
    s->g.timing = enable != 0;
    return RSOS_OK;
}

rsos_status rsos_timing_read(rsos_surface *s, int64_t *launches, double *mean_ms, double *total_ms)
{
    CHECK_HANDLE(s, s->g);
    return mark(s->g, s->g.read_timing(launches, mean_ms, total_ms));
}

rsos_status rsos_kernel_name(rsos_surface *s, char *buf, int32_t len)
{
    CHECK_HANDLE(s, s->g);
    if (!buf || len < 1) return fail(RSOS_E_INVAL, "bad buffer");
    const SurfaceGroup &g = s->g;
    const Variant *v = g.shapes.empty() ? nullptr : g.shapes[0].variant;
    const Pair *q = v && !g.timing ? g.shapes[0].pair : nullptr;  // (timed launches are of single sweeps)
    if (q)
        snprintf(buf, (size_t)len, "block_sweep2<%d,%d,%d,%d,%s>", q->D, q->TX, q->TY, q->NT, q->steps ? "true" : "false");
    else if (v && g.packed)
        snprintf(buf, (size_t)len, "block_sweep16<%d,%d,%d,%d,0>", v->D, v->TX, v->TY, v->NT);
    else if (v)
        snprintf(buf, (size_t)len, "block_sweep<%d,%d,%d,%d,%s,%d>", v->D, v->TX, v->TY, v->NT,
                 v->elem == 1 ? "int8,int16" : v->elem == 2 ? "int16,void" : "int32,void", v->steps ? 2 : g.sched);
    else
        snprintf(buf, (size_t)len, g.lds.mode == LdsMode::kLane ? "lds_run32<%d,256,%d>" : "lds_run<%d,512,%d,true>", g.D, g.sched);
    return RSOS_OK;
}

rsos_status rsos_free(rsos_surface *s)
{
    if (!s) return RSOS_OK;
    s->g.destroy();
    delete s;
    return RSOS_OK;
}

// ---------------------------------------------------------------------------
// batch
// ---------------------------------------------------------------------------
rsos_status rsos_batch_init(rsos_batch **out, int32_t n, const rsos_params *p, int32_t *d_pool,
                            int32_t *d_work_pool, const int64_t *offsets, int64_t log_cap,
                            void *stream)
{
    if (!out) return fail(RSOS_E_INVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || !p || !d_pool || !offsets) return fail(RSOS_E_INVAL, "bad batch arguments");
    if (log_cap < 0) return fail(RSOS_E_INVAL, "log_cap < 0");
    if (log_cap == 0) log_cap = 65536;
    rsos_status st;
    for (int i = 0; i < n; ++i) {
        if ((st = check_params(&p[i])) != RSOS_OK) return fail(st, "surface %d: %s", i, g_last_error.c_str());
        if (p[i].D != p[0].D) return fail(RSOS_E_INVAL, "all surfaces of a batch share one D");
        if (p[i].flags != p[0].flags) return fail(RSOS_E_INVAL, "all surfaces of a batch share one storage mode");
        if (offsets[i] < 0) return fail(RSOS_E_INVAL, "negative offset");
    }
    // surfaces must not overlap in the pool
    {
        std::vector<std::pair<long long, long long>> iv;
        for (int i = 0; i < n; ++i) iv.push_back({offsets[i], offsets[i] + (long long)p[i].L * p[i].L});
        std::sort(iv.begin(), iv.end());
        for (int i = 1; i < n; ++i)
            if (iv[i].first < iv[i - 1].second) return fail(RSOS_E_INVAL, "surfaces overlap in the pool");
    }
    rsos_batch *b = new (std::nothrow) rsos_batch();
    if (!b) return fail(RSOS_E_NOMEM, "host allocation failed");
    b->p.assign(p, p + n);
    SurfaceGroup &g = b->g;
    g.D = p[0].D;
    g.packed = (p[0].flags & RSOS_FLAG_PACKED16) != 0;
    g.sched = (p[0].flags & RSOS_FLAG_DT4) ? 1 : 0;
    g.stream = (hipStream_t)stream;
    long long pool_elems = 0;
    for (int i = 0; i < n; ++i) pool_elems = std::max(pool_elems, offsets[i] + (long long)p[i].L * p[i].L);
    int32_t *work = d_work_pool;
    if (!work && (st = g.dev_alloc((void **)&work, (size_t)pool_elems * 4)) != RSOS_OK) { delete b; return st; }
    long long *logs = nullptr;
    if ((st = g.dev_alloc((void **)&logs, sizeof(long long) * 3 * log_cap * n)) != RSOS_OK) { g.destroy(); delete b; return st; }
    for (int i = 0; i < n; ++i) {
        SurfDev d = {};
        if (g.packed) {
            // the surface's int32[L^2] of the pool holds both residue buffers
            d.buf[0] = d_pool + offsets[i];
            d.buf[1] = (int32_t *)((uint16_t *)(d_pool + offsets[i]) + (size_t)p[i].L * p[i].L);
            g.readout.push_back(work + offsets[i]);
        } else {
            d.buf[0] = d_pool + offsets[i];
            d.buf[1] = work + offsets[i];
        }
        d.log = logs + 3 * log_cap * i;
        d.log_cap = log_cap;
        d.key0 = (uint32_t)(p[i].seed & 0xFFFFFFFFu);
        d.key1 = (uint32_t)(p[i].seed >> 32);
        d.L = p[i].L;
        d.N = p[i].N;
        d.T = p[i].L / p[i].D;
        g.host.push_back(d);
        g.max_h0.push_back(0);
        g.t0.push_back(0);
    }
    if (tuning_wanted(&p[0])) {
        // one tuned choice per (L, N) class, grouped into kernel instances,
        // unless one variant for all times faster on this mix
        g.want.assign(n, Choice());
        std::vector<std::pair<int, int>> LN;
        std::vector<Choice> plan;
        for (int i = 0; i < n; ++i) {
            if (uses_lds(p[i].L)) continue;
            if ((st = tuned_choice(&p[i], 1, &g.want[i])) != RSOS_OK) {
                g.destroy();
                delete b;
                return st;
            }
            LN.push_back({p[i].L, p[i].N});
            plan.push_back(g.want[i]);
        }
        {
            std::lock_guard<std::mutex> lock(g_tune_mu);
            st = batch_plan(p[0].D, (int)p[0].flags, LN, &plan);
        }
        if (st != RSOS_OK) { g.destroy(); delete b; return st; }
        for (int i = 0, k = 0; i < n; ++i)
            if (!uses_lds(p[i].L)) g.want[i] = plan[k++];
    }
    if ((st = mark(g, g.setup())) != RSOS_OK) { g.destroy(); delete b; return st; }
    if ((st = g.dev_alloc((void **)&g.d_rec, sizeof(long long) * 3 * n)) != RSOS_OK) { g.destroy(); delete b; return st; }
    for (int i = 0; i < n; ++i)
        if ((st = g.load_initial(i, nullptr, 0)) != RSOS_OK || (st = g.init_record(i, 0, 0)) != RSOS_OK) {
            g.destroy();
            delete b;
            return st;
        }
    if ((st = mark(g, g.prepare_graph())) != RSOS_OK) { g.destroy(); delete b; return st; }
    *out = b;
    return RSOS_OK;
}

rsos_status rsos_batch_sweep(rsos_batch *b, const int64_t *n_mcs, int64_t n_all)
{
    CHECK_HANDLE(b, b->g);
    SurfaceGroup &g = b->g;
    const int n = (int)g.host.size();
    std::vector<long long> t_end(n);
    long long most = 0;
    for (int i = 0; i < n; ++i) {
        const long long k = n_mcs ? n_mcs[i] : n_all;
        if (k < 0) return fail(RSOS_E_INVAL, "negative sweep count for surface %d", i);
        if (g.host[i].t + k > (1ll << 32)) return fail(RSOS_E_INVAL, "sweep index would exceed 2^32");
        rsos_status st = check_overflow(b->p[i], g.max_h0[i], g.host[i].t + k - g.t0[i]);
        if (st != RSOS_OK) return st;
        t_end[i] = g.host[i].t + k;
        most = std::max(most, k);
    }
    if (most == 0) return RSOS_OK;
    rsos_status st;
    if ((st = mark(g, g.set_t_end(t_end, most))) != RSOS_OK) return st;
    if ((st = mark(g, g.launch_sweeps(most))) != RSOS_OK) return st;
    for (int i = 0; i < n; ++i) g.host[i].t = t_end[i];
    return RSOS_OK;
}

rsos_status rsos_batch_width(rsos_batch *b, rsos_width_t *out)
{
    CHECK_HANDLE(b, b->g);
    if (!out) return fail(RSOS_E_INVAL, "out is NULL");
    return mark(b->g, b->g.read_widths(out));
}

rsos_status rsos_batch_log(rsos_batch *b, int32_t i, int64_t t_from, int64_t n, rsos_width_t *out)
{
    CHECK_HANDLE(b, b->g);
    if (i < 0 || i >= (int)b->g.host.size()) return fail(RSOS_E_INVAL, "surface index out of range");
    if (!out && n > 0) return fail(RSOS_E_INVAL, "out is NULL");
    return mark(b->g, b->g.read_log(i, t_from, n, out));
}

rsos_status rsos_batch_moments(rsos_batch *b, int32_t i, rsos_moments_t *out)
{
    CHECK_HANDLE(b, b->g);
    if (i < 0 || i >= (int)b->g.host.size()) return fail(RSOS_E_INVAL, "surface index out of range");
    if (!out) return fail(RSOS_E_INVAL, "out is NULL");
    return mark(b->g, b->g.moments(i, out));
}

rsos_status rsos_batch_heights(rsos_batch *b, int32_t i, int32_t *dst, int dst_is_device)
{
    CHECK_HANDLE(b, b->g);
    if (i < 0 || i >= (int)b->g.host.size()) return fail(RSOS_E_INVAL, "surface index out of range");
    if (!dst) return fail(RSOS_E_INVAL, "dst is NULL");
    return mark(b->g, b->g.copy_heights(i, dst, dst_is_device));
}

rsos_status rsos_batch_free(rsos_batch *b)
{
    if (!b) return RSOS_OK;
    b->g.destroy();
    delete b;
    return RSOS_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Sweeps without any allocation (rsos_sweep_static).  The descriptor, the
// accumulator area and the log ring of the one surface live in `scratch`, a
// file-scope device array that every GPU the library runs on holds once
// until the process ends.  In host code its name is a host-side stand-in;
// the entry point takes the array's device address on each device with
// hipGetSymbolAddress the first time it runs there and uses that address
// only.  Calls on one GPU share the array: they must not overlap.
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kScratchBytes = 128 * 1024;
constexpr size_t kScratchDesc = 0;      // SurfDev
constexpr size_t kScratchIdx = 128;     // int 0: the LDS-path kernel's descriptor index
constexpr size_t kScratchAcc = 256;     // kAccWords int64
constexpr size_t kScratchLog = 4096;    // log ring of kStaticLogCap records of 3 int64
constexpr long long kStaticLogCap = RSOS_STATIC_MAX_SWEEPS + 1;
static_assert(sizeof(SurfDev) <= kScratchIdx, "descriptor slot");
static_assert(kScratchAcc + 8 * rsosk::kAccWords <= kScratchLog, "accumulator slot");
static_assert(kScratchLog + 24 * (size_t)kStaticLogCap <= kScratchBytes, "log ring");

__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch[kMaxDevices] = {};

// Device address of `scratch` on the current device.
rsos_status scratch_ptr(unsigned char **out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(RSOS_E_INVAL, "device %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(RSOS_E_DEVICE, "no device address for the scratch array");
        g_scratch[dev] = (unsigned char *)p;
    }
    *out = g_scratch[dev];
    return RSOS_OK;
}

}  // namespace

// Writes the descriptor, clears the accumulators and stores the record of
// time t0 (a fill kernel, not a memset: callers may capture the launches).
// Surfaces in LDS (`sum`) get the sums of the lattice itself, whatever the
// caller's are: lds_run goes on from the record, and lds_run32, which sums
// the lattice after each sweep, does not need it.
__global__ __launch_bounds__(256) void static_setup(SurfDev d, unsigned char *base, long long s1, long long s2, int sum)
{
    long long *acc = (long long *)(base + kScratchAcc);
    for (int i = threadIdx.x; i < rsosk::kAccWords; i += blockDim.x) acc[i] = 0;
    if (sum) {
        long long unused = 0;
        s1 = s2 = 0;
        const int32_t *h = d.buf[d.t & 1];
        for (int i = threadIdx.x; i < d.L * d.L; i += 256) {
            const long long v = h[i];
            s1 += v;
            s2 += v * v;
        }
        rsosk::block_reduce3<256>(s1, s2, unused);
    }
    __syncthreads();  // the accumulators are clear
    if (threadIdx.x == 0) {
        *(int *)(base + kScratchIdx) = 0;
        const long long L2 = (long long)d.L * d.L;
        acc[rsosk::kMeanWord] = s1 / L2;
        long long *rec = d.log + 3 * d.slot;
        rec[0] = s1;
        rec[1] = s2;
        rec[2] = 0;
        *(SurfDev *)(base + kScratchDesc) = d;
    }
}

// Records of times t0+1 .. t0+n from the ring into the caller's int64[3n].
__global__ void static_copy_log(const unsigned char *base, long long t0, long long n, long long *out)
{
    const long long *ring = (const long long *)(base + kScratchLog);
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < 3 * n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long k = i / 3, w = i % 3;
        out[i] = ring[3 * ((t0 + 1 + k) % kStaticLogCap) + w];
    }
}

extern "C" rsos_status rsos_sweep_static(const rsos_params *p, int32_t *d_h, int32_t *d_work, int64_t t0,
                                         int64_t s1, int64_t s2, int64_t n_mcs, int64_t *d_log, void *stream)
{
    rsos_status st = check_params(p);
    if (st != RSOS_OK) return st;
    if (p->flags & ~RSOS_FLAG_DT4)
        return fail(RSOS_E_INVAL, "rsos_sweep_static: flags may only select the schedule (RSOS_FLAG_DT4)");
    if (!d_h || !d_work || (n_mcs > 0 && !d_log)) return fail(RSOS_E_INVAL, "NULL buffer");
    if (n_mcs < 0 || n_mcs > RSOS_STATIC_MAX_SWEEPS)
        return fail(RSOS_E_INVAL, "n_mcs=%lld outside [0, %d]", (long long)n_mcs, RSOS_STATIC_MAX_SWEEPS);
    if (t0 < 0 || t0 + n_mcs > (1ll << 32)) return fail(RSOS_E_INVAL, "sweep index would exceed 2^32");
    if ((((uintptr_t)d_h) | ((uintptr_t)d_work)) & 15) return fail(RSOS_E_INVAL, "height buffers must be 16-byte aligned");
    const long long L2 = (long long)p->L * p->L;
    if (s1 < 0 || s2 < 0 || (__int128)s1 * s1 > (__int128)L2 * s2)
        return fail(RSOS_E_INVAL, "s1, s2 are not the sums of any heights (need 0 <= s1, s1^2 <= L^2 s2)");
    // every height is within N L of the mean s1 / L^2
    if ((st = check_overflow(*p, s1 / L2 + 1 + (long long)p->N * p->L, n_mcs)) != RSOS_OK) return st;
    if (n_mcs == 0) return RSOS_OK;
    unsigned char *base = nullptr;
    if ((st = scratch_ptr(&base)) != RSOS_OK) return st;
    const int D = p->D, sched = (p->flags & RSOS_FLAG_DT4) ? 1 : 0;
    SurfDev d = {};
    d.buf[0] = d_h;
    d.buf[1] = d_work;
    d.log = (long long *)(base + kScratchLog);
    d.acc = (long long *)(base + kScratchAcc);
    d.log_cap = kStaticLogCap;
    d.t = t0;
    d.slot = t0 % kStaticLogCap;
    d.t_end = t0 + n_mcs;
    d.key0 = (uint32_t)(p->seed & 0xFFFFFFFFu);
    d.key1 = (uint32_t)(p->seed >> 32);
    d.L = p->L;
    d.N = p->N;
    d.T = p->L / D;
    const Variant *v = nullptr;
    const Pair *pair = nullptr;
    if (!uses_lds(p->L)) {
        v = pick_variant(D, {{p->L, p->N}}, false, sched == 1);
        if (!v) return fail(RSOS_E_INVAL, "no tile-block shape fits L=%d, N=%d, D=%d", p->L, p->N, D);
        d.nbx = blocks_along(d.T, v->TX);
        d.nblocks = d.nbx * blocks_along(d.T, v->TY);
        d.block_start = 0;
        if (sched == 0) pair = pick_pair(D, {{p->L, p->N}});
    }
    hipStream_t s = (hipStream_t)stream;
    SurfDev *dd = (SurfDev *)(base + kScratchDesc);
    hipLaunchKernelGGL(static_setup, dim3(1), dim3(256), 0, s, d, base, (long long)s1, (long long)s2, v ? 0 : 1);
    HIP_TRY(hipGetLastError());
    if (!v) {
        // the whole surface in one workgroup's LDS, all sweeps in one launch
        lds_launcher(D, sched)(dim3(1), lds_plan(D, sched, {{p->L, p->N}}), s, dd, (const int *)(base + kScratchIdx));
        HIP_TRY(hipGetLastError());
    } else {
        BlockLaunch k = sched == 1 ? v->launch_dt : v->launch;
        long long left = n_mcs;
        for (; pair && left >= 4; left -= 4)
            for (int i = 0; i < 2; ++i)
                pair->launch(dim3(pair_blocks(*pair, d.T)), s, dd, 1, nullptr, 1, blocks_along(d.T, pair->TX));
        for (; left > 0; --left) k(dim3(d.nblocks), s, dd, 1, nullptr, 1, d.nbx, nullptr, nullptr);
        HIP_TRY(hipGetLastError());
    }
    const unsigned grid = (unsigned)std::min<long long>((3 * n_mcs + 255) / 256, 64);
    hipLaunchKernelGGL(static_copy_log, dim3(grid), dim3(256), 0, s, base, (long long)t0, (long long)n_mcs,
                       (long long *)d_log);
    HIP_TRY(hipGetLastError());
    return RSOS_OK;
}

// ---------------------------------------------------------------------------
// serving engine (continuous batching) -- see rsos_engine.inc
// ---------------------------------------------------------------------------
#include "rsos_engine.inc"

// ---------------------------------------------------------------------------
// multisurface lock-step mode -- see rsos_ms.inc
// ---------------------------------------------------------------------------
#include "rsos_ms.inc"
