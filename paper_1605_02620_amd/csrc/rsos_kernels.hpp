// rsos_kernels.hpp -- gfx950 kernels of the RSOS deposition sweep.
//
// Model (Kelling, Odor & Gemming): RSOS deposition on an L x L periodic
// lattice, accepted iff afterwards |h_i - h_j| <= N for the 4 nearest
// neighbours (Sec. I); one sweep = L^2 attempts scheduled over D x D domains
// whose origin moves randomly each sweep (Sec. II); per-sweep exact sums
// S1 = sum h, S2 = sum h^2 for Eq. (2).
//
// Schedule of one sweep s (identical bits for any launch shape):
//   origin (ox, oy) = Philox(0, 0, s, 2) words 0, 1 mod 2D;
//   colour-0 tiles of the shifted frame make D^2 attempts each, then the
//   colour-1 tiles; tile tile_id = ty*T + tx (T = L/D) in phase p takes its
//   sites from Philox counters (j, tile_id, s, p).
//
// Kernels:
//   block_sweep  one workgroup owns a TX x TY tile block of the shifted frame
//                plus a ring of D+1 sites.  It loads the block and ring from
//                the input buffer into LDS (aligned 16-byte chunks, stored
//                as int8 or int16 offsets from a per-block reference height
//                when they fit), recomputes the phase-0 update of the
//                colour-0 tiles just outside the block (their inputs are all
//                in the ring, and the update is a pure function of them),
//                runs phase 1 on the block, stores the block into the output
//                buffer and adds its (S1, S2, A) increments to one of the
//                surface's 64 accumulator slots; the surface's last block
//                folds them into the per-sweep log.  A sweep, sums included,
//                is one launch and costs one read and one write of every
//                site.  An int8 block whose range does not fit is swept
//                again by the same workgroup as int16 sub-blocks.
//   block_sweep16  the same on heights kept in HBM as 16-bit residues
//                (half the bytes per sweep) when N L <= 32766.
//   block_sweep2   two sweeps in one pass over the lattice, for launches that
//                are bound by their latency.
//   lds_run, lds_run32   a whole small surface (L^2 * 4 bytes fits in LDS)
//                lives in one workgroup's LDS for many sweeps; no per-sweep
//                launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace rsosk {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11).  Ten rounds; each round multiplies
// counter words 0 and 2 by the two round multipliers, mixes the high halves
// with words 1, 3 and the key, and the key advances by the two Weyl
// increments between rounds.
// ---------------------------------------------------------------------------
struct u32x4 {
    uint32_t v[4];
};

__host__ __device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                         uint32_t c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = (uint64_t)c0 * 0xD2511F53ull;
        const uint64_t m1 = (uint64_t)c2 * 0xCD9E8D57ull;
        const uint32_t n0 = (uint32_t)(m1 >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(m0 >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)m1;
        c3 = (uint32_t)m0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    u32x4 o;
    o.v[0] = c0; o.v[1] = c1; o.v[2] = c2; o.v[3] = c3;
    return o;
}

// ---------------------------------------------------------------------------
// Per-surface state shared by the kernels.  Lives in device memory; the
// host writes it at setup and sets t_end before a run; the sweep's last
// block (or lds_run) advances t.
// ---------------------------------------------------------------------------
constexpr int kAccSlots = 64;  // per-surface spread of the (S1, S2) atomics
// Per-surface accumulator area: 4 * kAccSlots words of increments (two pairs
// for a launch of two sweeps), then
// word kMeanWord = floor(S1 / L^2) of the current time (16-bit storage only,
// which recovers true heights from it: kept by the sweep's last block, read
// by every block) and, in a 128-byte line of its own so that the blocks'
// atomic additions to it do not stall those reads, word kDoneWord, the
// blocks of the running sweep that have committed.  All words but
// kMeanWord are zero between sweeps.  Areas are 128-byte aligned.
constexpr int kMeanWord = 4 * kAccSlots;
constexpr int kDoneWord = kMeanWord + 16;
constexpr int kAccWords = kDoneWord + 16;

// Lattice pointers reach the kernels through descriptors in memory, so the
// compiler sees generic pointers and would emit flat memory instructions
// (which also count against the LDS wait counter).  They always point to
// device global memory: accesses go through these global-address-space
// views.
typedef __attribute__((address_space(1))) int32_t gint32;
typedef __attribute__((address_space(1))) unsigned long long gu64;
typedef __attribute__((address_space(1))) long long gi64;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) v4i gv4i;

__device__ __forceinline__ const gint32 *as_global(const int32_t *p) { return (const gint32 *)p; }
__device__ __forceinline__ gint32 *as_global(int32_t *p) { return (gint32 *)p; }

__device__ __forceinline__ int4 load4(const gint32 *p)
{
    const v4i x = *reinterpret_cast<const gv4i *>(p);
    return make_int4(x.x, x.y, x.z, x.w);
}

__device__ __forceinline__ void store4(gint32 *p, const int4 v)
{
    const v4i x = {v.x, v.y, v.z, v.w};
    *reinterpret_cast<gv4i *>(p) = x;
}

struct SurfDev {
    int32_t *buf[2];      // state after t sweeps is in buf[t & 1] (see flip)
    long long *log;       // 3 * log_cap int64: (S1, S2, A) of time tau at slot tau % log_cap
    long long *acc;       // kAccWords int64: accumulators (zero between sweeps), mean floor
    long long log_cap;
    long long t;          // sweeps done
    long long slot;       // t % log_cap
    long long t_end;      // run while t < t_end
    uint32_t flip;        // the state of time t is in buf[(t + flip) & 1]; 0 but between two launches of two sweeps
    int block_start2;     // as block_start for the launches of two sweeps, whose blocks have a shape of their own
    uint32_t key0, key1;  // Philox key = seed
    int L, N, T;          // T = L / D
    int nbx;              // blocks along x (block path)
    int nblocks;          // blocks of this surface (block path)
    int block_start;      // first global block index of this surface
};

template <int D>
struct TileBits {
    static constexpr int LOG2D = (D == 2) ? 1 : (D == 4) ? 2 : (D == 8) ? 3 : (D == 16) ? 4 : 5;
    static constexpr int B = 2 * LOG2D;               // bits per site field
    static constexpr int F = 32 / B;                  // fields per 32-bit word
    static constexpr int PER = 4 * F;                 // attempts per Philox call
    static constexpr int NCALL = (D * D + PER - 1) / PER;
};

// Geometry of a TX x TY tile block with its ring of D+1 sites, as staged in
// LDS: region rows of RW sites in RWL elements (CH chunks; the rows are laid
// RWL elements apart, or RowPitch below for byte staging), shifted right by
// the alignment pad (0..CPC-1) of the region's first column so that every
// global load is an aligned 16-byte chunk of CPC cells (4 int32 or 8 uint16).
template <int D, int TX, int TY, int CPC = 4>
struct BlockGeom {
    static constexpr int RING = D + 1;
    static constexpr int RW = TX * D + 2 * RING;
    static constexpr int RH = TY * D + 2 * RING;
    static constexpr int RWL = (RW + 2 * (CPC - 1)) & ~(CPC - 1);
    static constexpr int CH = RWL / CPC;
    static constexpr int HALF = TX * TY / 2;
    static constexpr int P0 = HALF + TX + TY;
    static constexpr int BW = TX * D, BH = TY * D;
};

// One attempt on the site at field f of a tile whose site (u, v) sits at LDS
// index base + v*P + u (neighbours at +-1 and +-P).  E is the LDS element
// type: narrow types hold heights relative to a per-block base, int32 raw
// heights.  Adds the acceptance to acc (minus the acceptance with unsigned
// byte staging) and, when accepted, the staged value c before the deposit
// to q (a deposit on height h raises sum h^2 by 2h + 1).
template <int D, int P, typename E, typename Q>
__device__ __forceinline__ void attempt(E *lds, int base, uint32_t f, int N, int &acc, Q &q)
{
    constexpr int LOG2D = TileBits<D>::LOG2D;
    const int idx = base + (int)(f >> LOG2D) * P + (int)(f & (D - 1));
    if constexpr (std::is_same<E, uint8_t>::value) {
        // unsigned byte staging (LDS-bound): the left neighbour, the site and
        // the right neighbour from one read of the two aligned words around
        // them (measured slower on the HBM-bound int8 path, so not used there).
        // Every access is addressed from i1 = idx - 1; the byte shift of
        // v_alignbyte uses the low two bits of its operand only.
        const int i1 = (base - 1) + (int)__umul24(f >> LOG2D, (uint32_t)P) + (int)(f & (D - 1));
        const uint32_t *w = reinterpret_cast<const uint32_t *>(lds + (i1 & ~3));
        const uint32_t t3 = __builtin_amdgcn_alignbyte(w[1], w[0], (uint32_t)i1);
        // min(left, right) straight from bytes 0 and 2 of t3 (one instruction
        // where the compiler would extract both bytes first)
        uint32_t lr;
        asm("v_min_u16_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0 src1_sel:BYTE_2"
            : "=v"(lr) : "v"(t3));
        const int d1 = (int)lds[i1 + 1 - P], d2 = (int)lds[i1 + 1 + P];
        // the new height is min(c + 1, m + N), m the least neighbour: accepted
        // iff c + 1 <= m + N, and c <= m + N always
        int n1;
        asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1"
            : "=v"(n1) : "v"(1 - N), "v"(t3));
        n1 = min(min(min(n1, (int)lr), d1), d2) + N;
        lds[i1 + 1] = (E)n1;
        // all ones if accepted, else zero; then c where accepted
        int nok, qc;
        asm("v_sub_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD"
            : "=v"(nok) : "v"(t3), "v"(n1));
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1"
            : "=v"(qc) : "v"(nok), "v"(t3));
        q += qc;
        // this staging counts acceptances negatively (one instruction less
        // per attempt); region_sweep16 negates the block's count
        acc += nok;
        return;
    } else {
        const int c = lds[idx], l = lds[idx - 1], r = lds[idx + 1], u = lds[idx - P], w = lds[idx + P];
        if constexpr (sizeof(E) <= 2) {
            // narrow staging: N is far inside int range (see above)
            const int n1 = min(min(min(min(c + 1 - N, l), r), u), w) + N;
            lds[idx] = (E)n1;
            const int ok = n1 - c;
            q += __mul24(c, ok);
            acc += ok;
        } else {
            // h_c + 1 - h_j <= N for every neighbour j; the lower side cannot
            // fail because |h_c - h_j| <= N held before
            const int ok = (c - min(min(l, r), min(u, w))) < N;
            q += ok ? (Q)c : (Q)0;
            lds[idx] = (E)(c + ok);
            acc += ok;
        }
    }
}

// D^2 sequential attempts of one tile: the Philox calls whose fields are
// all used, then the call that holds the last D^2 mod (fields per call).
template <int D, int P, typename E, typename Q>
__device__ __forceinline__ void tile_attempts(E *lds, int base, uint32_t tile_id, uint32_t s,
                                              uint32_t p, int N, uint32_t k0, uint32_t k1,
                                              int &acc, Q &q)
{
    using TB = TileBits<D>;
    constexpr int NFULL = (D * D) / TB::PER, TAIL = (D * D) % TB::PER;
    constexpr uint32_t MASK = (uint32_t)(D * D - 1);
#pragma unroll 1
    for (int j = 0; j < NFULL; ++j) {
        const u32x4 r = philox4x32_10((uint32_t)j, tile_id, s, p, k0, k1);
#pragma unroll
        for (int k = 0; k < TB::PER; ++k)
            attempt<D, P, E, Q>(lds, base, (r.v[k / TB::F] >> ((k % TB::F) * TB::B)) & MASK, N, acc, q);
    }
    if constexpr (TAIL > 0) {
        const u32x4 r = philox4x32_10((uint32_t)NFULL, tile_id, s, p, k0, k1);
#pragma unroll
        for (int k = 0; k < TAIL; ++k)
            attempt<D, P, E, Q>(lds, base, (r.v[k / TB::F] >> ((k % TB::F) * TB::B)) & MASK, N, acc, q);
    }
}

__device__ __forceinline__ void wave_reduce3(long long &a, long long &b, long long &c)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
        c += __shfl_xor(c, off, 64);
    }
}

// Result valid in thread 0.
template <int NT>
__device__ __forceinline__ void block_reduce3(long long &a, long long &b, long long &c)
{
    __shared__ long long red[3][NT / 64 > 0 ? NT / 64 : 1];
    wave_reduce3(a, b, c);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (NT > 64) {
        if (l == 0) { red[0][w] = a; red[1][w] = b; red[2][w] = c; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < NT / 64; ++i) { a += red[0][i]; b += red[1][i]; c += red[2][i]; }
        }
    }
}

template <typename E>
__device__ __forceinline__ void lds_put4(E *dst, const int4 v, int ref);

template <>
__device__ __forceinline__ void lds_put4<int16_t>(int16_t *dst, const int4 v, int ref)
{
    const uint32_t lo = (uint32_t)(uint16_t)(v.x - ref) | ((uint32_t)(uint16_t)(v.y - ref) << 16);
    const uint32_t hi = (uint32_t)(uint16_t)(v.z - ref) | ((uint32_t)(uint16_t)(v.w - ref) << 16);
    *reinterpret_cast<uint2 *>(dst) = make_uint2(lo, hi);
}

template <>
__device__ __forceinline__ void lds_put4<int8_t>(int8_t *dst, const int4 v, int ref)
{
    const uint32_t w = (uint32_t)(uint8_t)(v.x - ref) | ((uint32_t)(uint8_t)(v.y - ref) << 8) |
                       ((uint32_t)(uint8_t)(v.z - ref) << 16) | ((uint32_t)(uint8_t)(v.w - ref) << 24);
    *reinterpret_cast<uint32_t *>(dst) = w;
}

template <>
__device__ __forceinline__ void lds_put4<int32_t>(int32_t *dst, const int4 v, int)
{
    *reinterpret_cast<int4 *>(dst) = v;
}

template <typename E> struct Lds4;
template <> struct Lds4<int16_t> {
    typedef uint2 raw;
    __device__ static int4 widen(const uint2 w, int ref)
    {
        return make_int4(ref + (int)(int16_t)(w.x & 0xFFFF), ref + (int)(int16_t)(w.x >> 16),
                         ref + (int)(int16_t)(w.y & 0xFFFF), ref + (int)(int16_t)(w.y >> 16));
    }
};
template <> struct Lds4<int8_t> {
    typedef uint32_t raw;
    __device__ static int4 widen(const uint32_t w, int ref)
    {
        return make_int4(ref + (int)(int8_t)(w & 0xFF), ref + (int)(int8_t)((w >> 8) & 0xFF),
                         ref + (int)(int8_t)((w >> 16) & 0xFF), ref + (int)(int8_t)(w >> 24));
    }
};
template <> struct Lds4<int32_t> {
    typedef int4 raw;
    __device__ static int4 widen(const int4 w, int) { return w; }
};





// The next sweep reads the output from HBM long after this one wrote it:
// stream the full 16-byte chunks past the caches.
__device__ __forceinline__ void store4_stream(gint32 *dst, const int4 v)
{
    const v4i x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<gv4i *>(dst));
}

// Descriptor index of the surface that owns global block lb: from the
// host-built table when there is one (one load), else by binary search over
// the descriptors (sorted by block_start).
template <bool TWO = false>
__device__ __forceinline__ int find_surface(const SurfDev *descs, int nsurf, const int *owner, int lb)
{
    if (owner) return owner[lb];
    int lo = 0, hi = nsurf - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((TWO ? descs[mid].block_start2 : descs[mid].block_start) <= lb) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Place of a TX x TY tile block: the tile of its upper left corner.  Blocks
// tile the lattice where its T x T tiles divide; where they do not, the last
// block of a row (column) is moved back to end with the lattice, and its
// first dupx columns (dupy rows) of tiles are the previous block's too: both
// compute the same bits from the same inputs and write them, the previous
// block counts them.  So one shape serves every T: before, only blocks of
// 2 x 2 tiles divided most of the sizes that are no power of two (L = 1360,
// T = 170: 113 us per sweep, with 32 x 8 blocks 23 us).
struct BlockPos {
    int tx, ty, dupx, dupy;
    __device__ __forceinline__ bool counts(int ltx, int lty) const { return ltx >= dupx && lty >= dupy; }
};

template <int TX, int TY>
__device__ __forceinline__ BlockPos block_pos(int bx, int by, int T)
{
    const int tx = min(bx * TX, T - TX), ty = min(by * TY, T - TY);
    return {tx, ty, bx * TX - tx, by * TY - ty};
}

// Both phases of one sweep on a block staged in LDS with row pitch RWL and
// block column 0 at column off of region row RING.  Phase 0: the colour-0
// tiles of the block, then the colour-0 ring tiles that touch the block's
// colour-1 border tiles (their counts belong to the neighbouring blocks and
// are dropped); phase 1: the colour-1 tiles of the block.  acc and q receive
// this thread's accepted count and sum of accepted staged values.
template <int D, int TX, int TY, int NT, int RWL, typename E, typename Q>
__device__ __forceinline__ void block_phases(E *lds, int off, BlockPos bp, int T, uint32_t s, int N,
                                             uint32_t k0, uint32_t k1, int &acc, Q &q)
{
    constexpr int RING = D + 1, HALF = TX * TY / 2, P0 = HALF + TX + TY;
    for (int k = threadIdx.x; k < P0; k += NT) {
        int ltx, lty;
        if (k < HALF) {
            lty = k / (TX / 2);
            ltx = 2 * (k % (TX / 2)) + (lty & 1);
        } else {
            const int g = k - HALF;
            if (g < TX / 2) { lty = -1; ltx = 2 * g + 1; }
            else if (g < TX) { lty = TY; ltx = 2 * (g - TX / 2); }
            else if (g < TX + TY / 2) { ltx = -1; lty = 2 * (g - TX) + 1; }
            else { ltx = TX; lty = 2 * (g - TX - TY / 2); }
        }
        int gtx = bp.tx + ltx, gty = bp.ty + lty;
        gtx = gtx < 0 ? gtx + T : (gtx >= T ? gtx - T : gtx);
        gty = gty < 0 ? gty + T : (gty >= T ? gty - T : gty);
        const int base = (lty * D + RING) * RWL + ltx * D + off;
        int a = 0;
        Q qq = 0;
        tile_attempts<D, RWL, E, Q>(lds, base, (uint32_t)(gty * T + gtx), s, 0u, N, k0, k1, a, qq);
        if (k < HALF && bp.counts(ltx, lty)) { acc += a; q += qq; }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < HALF; k += NT) {
        const int lty = k / (TX / 2);
        const int ltx = 2 * (k % (TX / 2)) + 1 - (lty & 1);
        const int gtx = bp.tx + ltx, gty = bp.ty + lty;
        const int base = (lty * D + RING) * RWL + ltx * D + off;
        int a = 0;
        Q qq = 0;
        tile_attempts<D, RWL, E, Q>(lds, base, (uint32_t)(gty * T + gtx), s, 1u, N, k0, k1, a, qq);
        if (bp.counts(ltx, lty)) { acc += a; q += qq; }
    }
    __syncthreads();
}

// The double-tiling schedule on the same block (TX x TY sub-tiles of D,
// TX and TY even, so a block holds whole 2 x 2 tiles).  Set k = (sx mod 2)
// + 2 (sy mod 2) is updated in phase k with Philox phase code 4 + k.  The
// block's border sub-tiles read sub-tiles of the neighbouring blocks; those
// updated in an earlier phase are recomputed here, in their phase: the
// set-0 sub-tiles of the frame column right of the block and of the frame
// row below it (and the corner between them) in phase 0, the set-1
// sub-tiles of the row below in phase 1, the set-2 sub-tiles of the column
// to the right in phase 2.  Their inputs are original values or values
// this block has already brought to the same phase; the frames above and
// to the left are read only before their own updates.  Counts of frame
// sub-tiles are dropped.
template <int D, int TX, int TY, int NT, int RWL, typename E, typename Q>
__device__ __forceinline__ void block_phases_dt(E *lds, int off, BlockPos bp, int T, uint32_t s, int N,
                                                uint32_t k0, uint32_t k1, int &acc, Q &q)
{
    static_assert(TX % 2 == 0 && TY % 2 == 0, "blocks hold whole 2 x 2 tiles");
    constexpr int RING = D + 1, Q4 = TX * TY / 4;
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
        const int extra = k == 0 ? TX / 2 + TY / 2 + 1 : k == 1 ? TX / 2 : k == 2 ? TY / 2 : 0;
        for (int i = threadIdx.x; i < Q4 + extra; i += NT) {
            int ltx, lty;
            if (i < Q4) {
                lty = 2 * (i / (TX / 2)) + (k >> 1);
                ltx = 2 * (i % (TX / 2)) + (k & 1);
            } else {
                const int g = i - Q4;
                if (k == 0) {
                    if (g < TY / 2) { ltx = TX; lty = 2 * g; }
                    else if (g < TY / 2 + TX / 2) { lty = TY; ltx = 2 * (g - TY / 2); }
                    else { ltx = TX; lty = TY; }
                } else if (k == 1) {
                    lty = TY;
                    ltx = 2 * g + 1;
                } else {
                    ltx = TX;
                    lty = 2 * g + 1;
                }
            }
            int gsx = bp.tx + ltx, gsy = bp.ty + lty;
            if (gsx >= T) gsx -= T;
            if (gsy >= T) gsy -= T;
            const int base = (lty * D + RING) * RWL + ltx * D + off;
            int a = 0;
            Q qq = 0;
            tile_attempts<D, RWL, E, Q>(lds, base, (uint32_t)(gsy * T + gsx), s, 4u + (uint32_t)k, N, k0, k1, a, qq);
            if (i < Q4 && bp.counts(ltx, lty)) { acc += a; q += qq; }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Attempts in steps.  Attempts commute unless their sites are the same or
// neighbours, so where too few tiles are at work to fill the lanes, a tile's
// attempts are laid out in steps of up to kLdsWin pairwise independent ones
// that keep their order across steps (one lane per tile and Philox call; the
// site sequence does not depend on the heights), and kLdsWin lanes of a tile
// make the attempts of a step together: for D = 8 about 27 steps, each one
// LDS round trip, instead of 64.  Used on int16 staging.
// ---------------------------------------------------------------------------
constexpr int kLdsWin = 4;        // attempts per step

// Attempts of one Philox call, and of the last one of a tile.  Every lane of
// a tile has its own list of that many entries per call (a call may need a
// step for each of its attempts); an entry is the LDS address of the site
// above the attempt's (in units of 2^SHIFT bytes, in 16 bits).
template <int D>
struct StepList {
    using TB = TileBits<D>;
    static constexpr int NPER = TB::PER < D * D ? TB::PER : D * D;
    static constexpr int NLAST = D * D - (TB::NCALL - 1) * NPER;
    static_assert(NPER % 2 == 0 && NLAST % 2 == 0, "entries are read in pairs");
};

typedef __attribute__((address_space(3))) int16_t l16;
__device__ __forceinline__ uint32_t lds_address(const int16_t *p) { return (uint32_t)(uintptr_t)(const l16 *)p; }

// a / d for 0 <= a < 2^20 with r = 1.0f / d: (a + 1/2) / d is at least
// 1 / (2 d) from every integer, far more than the float error.
__device__ __forceinline__ int div_by(int a, float r) { return (int)(((float)a + 0.5f) * r); }

// Sum over the wavefront, in lane 63 (six dependent adds; an LDS atomic from
// every lane took 9000 cycles per sweep).
__device__ __forceinline__ int wave_sum63(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, true);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, true);   // row_bcast:31
    return v;
}

// Lays out the attempts of Philox call j of one tile in steps: the k-th step
// takes entry k of the lists of the tile's kLdsWin lanes (`stride` entries
// apart, 16-byte aligned); the entries that are not used name the idle site
// (idle2: its entry twice).  `above` is the site above the tile's corner.
// Returns the number of steps.
template <int D, int P, int SHIFT>
__device__ __forceinline__ int lay_out_steps(uint16_t *list, int stride, const int16_t *above, uint32_t idle2, int j,
                                             uint32_t tile_id, uint32_t s, uint32_t p, uint32_t k0, uint32_t k1)
{
    using R = StepList<D>;
    using TB = TileBits<D>;
    const u32x4 r = philox4x32_10((uint32_t)j, tile_id, s, p, k0, k1);
    const int n = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
#pragma unroll
    for (int i = 0; i < R::NPER / 2; ++i)
        if (i < n / 2) ((uint4 *)list)[i] = make_uint4(idle2, idle2, idle2, idle2);
    const uint32_t a0 = lds_address(above) >> SHIFT;
    constexpr uint32_t FAR = 0x8080u;            // further than one bond from every site
    uint32_t w1 = FAR, w2 = FAR, w3 = FAR;       // the step's sites so far, x + 256 y
    int at = 0;                                  // entry of the next site
    int used = 0, steps = 0;                     // sites of the current step, steps before it
    static_assert(kLdsWin == 4, "three earlier sites are compared");
#pragma unroll
    for (int k = 0; k < R::NPER; ++k) {
        if (k < n) {
            const uint32_t f = (r.v[k / TB::F] >> ((k % TB::F) * TB::B)) & (uint32_t)(D * D - 1);
            const uint32_t x = f & (uint32_t)(D - 1), y = f >> TB::LOG2D;
            const uint32_t xy = x | (y << 8);
            const uint32_t near = min(min(__builtin_amdgcn_sad_u8(xy, w1, 0), __builtin_amdgcn_sad_u8(xy, w2, 0)),
                                      __builtin_amdgcn_sad_u8(xy, w3, 0));
            const bool next = near <= 1u || used == kLdsWin;
            w3 = next ? FAR : w2;
            w2 = next ? FAR : w1;
            w1 = xy;
            steps += next;
            at = next ? steps : at;
            used = next ? 1 : used + 1;
            list[at] = (uint16_t)(a0 + (__umul24(y, (uint32_t)P) + x) * 2 / (1 << SHIFT));
            at += stride;
        }
    }
    return steps + 1;
}

// The attempts of one lane's list of a call: n steps (rounded up to pairs)
// on staging with row pitch P.
template <int P, int SHIFT>
__device__ __forceinline__ void make_steps(const uint32_t *e, int n, int N, int &acc, int &q)
{
    auto attempt1 = [&](uint32_t a) {
        // the site above, then the site and its neighbours at constant offsets
        l16 *c = (l16 *)(uintptr_t)(a << SHIFT);
        const int u = c[0], l = c[P - 1], v = c[P], r = c[P + 1], w = c[2 * P];
        // a deposit is accepted iff v + 1 <= m + N, and v <= m + N always
        const int n1 = min(v + 1, min(min(l, r), min(u, w)) + N);
        c[P] = (int16_t)n1;
        const int ok = n1 - v;
        acc += ok;
        q += __mul24(v, ok);
        // the next step's reads stay behind these writes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    uint32_t two = *e;
#pragma unroll 1
    for (int step = 0; step < n; step += 2) {
        const uint32_t cur = two;
        two = *++e;  // (one pair beyond the last step's is read, and not used)
        attempt1(cur & 0xFFFFu);
        attempt1(cur >> 16);
    }
}

// Both phases of block_phases on int16 staging, in steps.  lay_out_block
// fills the lists (it reads no height, so it runs while the region's loads
// are on their way), block_phases_steps makes the attempts.
template <int D, int TX, int TY, int NT, int RWL, int RH>
struct BlockSteps {
    using TB = TileBits<D>;
    using R = StepList<D>;
    static constexpr int RING = D + 1, HALF = TX * TY / 2, P0 = HALF + TX + TY, ALL = P0 + HALF;
    static constexpr int G0 = (P0 + 15) / 16, GROUPS = G0 + (HALF + 15) / 16;
    // after the region: the idle site with its neighbours, the lists, the
    // longest number of steps of each 16 tiles by call
    static constexpr int IDLE = (RWL * RH + 7) & ~7;                // element
    static constexpr int LISTS = (IDLE + 2 * RWL + 2 + 7) & ~7;     // element
    static constexpr int STEPS = LISTS + ALL * D * D * kLdsWin + 8; // element (a pair is read beyond the lists)
    static constexpr int BYTES = 2 * STEPS + 4 * TB::NCALL * GROUPS;

    // tile k of the list: phase 0's (block_phases' order), then phase 1's
    static __device__ __forceinline__ void tile(int k, int &ltx, int &lty)
    {
        const int p = k >= P0;
        const int i = p ? k - P0 : k;
        lty = i / (TX / 2);
        ltx = 2 * (i % (TX / 2)) + ((lty + p) & 1);
        if (!p && i >= HALF) {
            const int g = i - HALF;
            if (g < TX / 2) { lty = -1; ltx = 2 * g + 1; }
            else if (g < TX) { lty = TY; ltx = 2 * (g - TX / 2); }
            else if (g < TX + TY / 2) { ltx = -1; lty = 2 * (g - TX) + 1; }
            else { ltx = TX; lty = 2 * (g - TX - TY / 2); }
        }
    }
    static __device__ __forceinline__ uint32_t idle2(int16_t *lds) { return lds_address(lds + IDLE + 1) * 0x10001u; }

    // before the workgroup's first barrier
    static __device__ __forceinline__ void clear(int16_t *lds, int N)
    {
        int *steps = (int *)(lds + STEPS);
        for (int i = threadIdx.x; i < TB::NCALL * GROUPS; i += NT) steps[i] = 0;
        if (threadIdx.x == 0) {
            // N above its neighbours: never changes
            int16_t *c = lds + IDLE + 1 + RWL;
            c[0] = 0;
            c[-1] = c[1] = c[-RWL] = c[RWL] = (int16_t)-N;
        }
    }
    static __device__ __forceinline__ void lay_out(int16_t *lds, int off, BlockPos bp, int T, uint32_t s, uint32_t k0,
                                                   uint32_t k1)
    {
        int *steps = (int *)(lds + STEPS);
        for (int i = threadIdx.x; i < ALL * TB::NCALL; i += NT) {
            const int j = i / ALL, k = i - j * ALL;  // consecutive lanes take consecutive tiles
            int ltx, lty;
            tile(k, ltx, lty);
            int gtx = bp.tx + ltx, gty = bp.ty + lty;
            gtx = gtx < 0 ? gtx + T : (gtx >= T ? gtx - T : gtx);
            gty = gty < 0 ? gty + T : (gty >= T ? gty - T : gty);
            const int stride = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
            const int16_t *above = lds + (lty * D + RING - 1) * RWL + ltx * D + off;
            const int n = lay_out_steps<D, RWL, 0>((uint16_t *)(lds + LISTS) + (j * R::NPER * ALL + k * stride) * kLdsWin,
                                                   stride, above, idle2(lds), j, (uint32_t)(gty * T + gtx), s, k >= P0 ? 1u : 0u, k0, k1);
            atomicMax(&steps[j * GROUPS + (k < P0 ? k / 16 : G0 + (k - P0) / 16)], n);
        }
    }
    static __device__ __forceinline__ void phases(int16_t *lds, BlockPos bp, int N, int &acc, int &q)
    {
        const int *steps = (const int *)(lds + STEPS);
#pragma unroll 1
        for (int p = 0; p < 2; ++p) {
            for (int i = threadIdx.x / kLdsWin; i < (p ? HALF : P0); i += NT / kLdsWin) {
                const int k = p ? P0 + i : i;
                int a = 0, qq = 0;
#pragma unroll 1
                for (int j = 0; j < TB::NCALL; ++j) {
                    const int n = __builtin_amdgcn_readfirstlane(steps[j * GROUPS + (p ? G0 : 0) + i / 16]);
                    const int stride = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
                    const uint16_t *e = (const uint16_t *)(lds + LISTS) + (j * R::NPER * ALL + k * stride) * kLdsWin +
                                  (threadIdx.x & (kLdsWin - 1)) * stride;
                    make_steps<RWL, 0>((const uint32_t *)e, n, N, a, qq);
                }
                int ltx, lty;
                tile(k, ltx, lty);
                if ((p || i < HALF) && bp.counts(ltx, lty)) { acc += a; q += qq; }
            }
            __syncthreads();
        }
    }
};

// Schedule selector: 0 = tile checkerboard, 1 = double tiling.  (The kernels'
// schedule 2, the checkerboard in steps on int16 staging, has its phases in
// BlockSteps.)
template <int SCHED, int D, int TX, int TY, int NT, int RWL, typename E, typename Q>
__device__ __forceinline__ void sweep_phases(E *lds, int off, BlockPos bp, int T, uint32_t s, int N,
                                             uint32_t k0, uint32_t k1, int &acc, Q &q)
{
    if constexpr (SCHED == 0)
        block_phases<D, TX, TY, NT, RWL, E, Q>(lds, off, bp, T, s, N, k0, k1, acc, q);
    else
        block_phases_dt<D, TX, TY, NT, RWL, E, Q>(lds, off, bp, T, s, N, k0, k1, acc, q);
}

// ---------------------------------------------------------------------------
// End of a sweep.  Every block adds its increments (A, sum(2h + 1) over its
// accepted deposits) of S1 and S2 to one of the surface's 64 accumulator
// slots and counts itself in the surface's done word; the block that
// completes the count folds the slots into the record of time t + 1 (the
// record of t plus the increments), clears them, keeps floor(S1 / L^2) where
// the storage needs it and advances the surface's time.  So one launch is a
// whole sweep, and the sums are exact whatever order the blocks finish in.
// All of it uses device-scope atomics without fences (an acquire or release
// at device scope would write back or invalidate the XCD's whole L2 in
// every block): a block counts itself only after its two slot additions
// have been performed (it waits for them), and the last block reads the
// slots with device-scope atomic loads.  Its plain stores (time, log
// record, mean) are read by later launches only.
//
// Each of these steps is a round trip of the order of a microsecond, which
// small lattices cannot hide: in the attempts-in-steps kernel only wave 0
// takes them, while the others make their stores.  Reductions are DPP additions (a 64-bit shuffle
// is two LDS permutes), and nothing divides: the log slot is kept in the
// descriptor.
// ---------------------------------------------------------------------------

// Sum over the wavefront, in lane 63.
template <int CTRL, int MASK>
__device__ __forceinline__ long long dpp_add64(long long v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, MASK, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((unsigned long long)v >> 32), CTRL, MASK, 0xF, true);
    return v + (long long)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ long long wave_sum63_64(long long v)
{
    v = dpp_add64<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8
    v = dpp_add64<0x112, 0xF>(v);
    v = dpp_add64<0x114, 0xF>(v);
    v = dpp_add64<0x118, 0xF>(v);
    v = dpp_add64<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add64<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Wave 0 of the block that completed the count of a launch of NS sweeps (of
// two: flip is the descriptor's).
template <bool MEAN, int NS = 1>
__device__ __forceinline__ void finish_sweep(SurfDev &d, long long t, uint32_t flip = 0)
{
    const int lane = threadIdx.x;  // < 64
    const gi64 *prev = (const gi64 *)(d.log + 3 * d.slot);
    long long S1 = prev[0], S2 = prev[1];
    gu64 *a = (gu64 *)(d.acc + 4 * lane);
    long long x[2 * NS];
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i) x[i] = (long long)__hip_atomic_load(a + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i) __hip_atomic_store(a + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i) x[i] = wave_sum63_64(x[i]);
    if (lane == 63) {
        long long slot = d.slot;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            slot = slot + 1 == d.log_cap ? 0 : slot + 1;
            gi64 *e = (gi64 *)(d.log + 3 * slot);
            e[0] = S1 += x[2 * k];
            e[1] = S2 += x[2 * k + 1];
            e[2] = x[2 * k];
        }
        if constexpr (MEAN) *(gi64 *)(d.acc + kMeanWord) = S1 / ((long long)d.L * d.L);
        __hip_atomic_store((gu64 *)(d.acc + kDoneWord), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *(gi64 *)&d.t = t + NS;
        *(gi64 *)&d.slot = slot;
        if (NS == 2) *(gint32 *)&d.flip = (int32_t)(flip ^ 1u);
    }
}

// inc: this thread's accepted count and its share of the S2 increment, for
// each sweep of the launch.  Called by the whole workgroup once its sums are
// final.  Returns, in thread 0, the number of the surface's blocks counted
// before this one.
template <int NT, int NS = 1>
__device__ __forceinline__ unsigned long long commit_sweep(SurfDev &d, int b, long long (&inc)[2 * NS])
{
    __shared__ long long red[2 * NS][NT / 64];
#pragma unroll
    for (int i = 0; i < 2 * NS; ++i) {
        inc[i] = wave_sum63_64(inc[i]);
        if ((threadIdx.x & 63) == 63) red[i][threadIdx.x >> 6] = inc[i];
    }
    __syncthreads();
    unsigned long long before = 0;
    if (threadIdx.x == 0) {
        gu64 *slot = (gu64 *)(d.acc + 4 * (b & (kAccSlots - 1)));
#pragma unroll
        for (int i = 0; i < 2 * NS; ++i) {
            long long v = red[i][0];
            for (int w = 1; w < NT / 64; ++w) v += red[i][w];
            __hip_atomic_fetch_add(slot + i, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // the additions are performed before the block is counted
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        before = __hip_atomic_fetch_add((gu64 *)(d.acc + kDoneWord), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return before;
}

// Whether this block completed the count (wave 0; false in the others).
// Waits for the count, and for every store that wave 0 has made before.
__device__ __forceinline__ bool is_last(int nblocks, unsigned long long before)
{
    return threadIdx.x < 64 && __builtin_amdgcn_readfirstlane((int)(before + 1 == (unsigned long long)nblocks)) != 0;
}

// Workgroup -> global block.  Mode 1: the dispatcher hands consecutive
// workgroup ids to the 8 XCDs in turn; each XCD takes runs of 16 consecutive
// blocks (left and right neighbours share its L2 for their ring columns)
// while the 8 XCDs together walk the lattice in memory order; blocks beyond
// the last whole group of 8 x 16 keep their number.  Mode 2 (one surface,
// nbx % 8 == 0): XCD x owns the block columns [x nbx/8, (x+1) nbx/8) and
// walks them row by row, so a block's upper and lower neighbours, whose
// regions overlap its ring rows, run on the same XCD; all XCDs still move
// down the lattice together.  Mode 0: identity.
__device__ __forceinline__ int block_map(int wg, int n, int mode, int nbx)
{
    if (mode == 1) {
        constexpr int C = 16;
        const int full = n - n % (8 * C);
        if (wg >= full) return wg;
        const int x = wg & 7, j = wg >> 3;
        return (j / C) * (8 * C) + x * C + (j % C);
    }
    if (mode == 2) {
        const int sw = nbx >> 3, x = wg & 7, j = wg >> 3;
        return (j / sw) * nbx + x * sw + j % sw;
    }
    return wg;
}

// LDS row pitch of a byte-staged region.  Rounded up to a multiple of 64
// bytes (half the 32 banks) it spreads the lanes of a wavefront over the
// banks more evenly than the bare row length does, at the price of LDS per
// block: done for the tile checkerboard where that price is at most 15%
// (rows of 32 tiles at D = 8: 280 or 288 -> 320 bytes; measured faster),
// not for narrower rows or the double-tiling schedule, whose latency-bound
// phases need the blocks per CU more (measured slower).
template <int ES, int RWL, int SCHED>
struct RowPitch {
    static constexpr int padded = (RWL + 63) & ~63;
    static constexpr int v = (ES == 1 && SCHED == 0 && 100 * padded <= 115 * RWL) ? padded : RWL;
};

// LDS bytes of a block's narrow staging with its row pitch.
template <int D, int TX, int TY, int CPC, int ES, int SCHED>
struct NarrowBytes {
    using G = BlockGeom<D, TX, TY, CPC>;
    static constexpr int v = RowPitch<ES, G::RWL, SCHED>::v * G::RH * ES;
};

// Where a block's staging does not fit its narrow element type, the same
// workgroup sweeps it again as SX x SY sub-blocks with the wide type EW.
// The tile block shape never changes results (each sub-block recomputes the
// ring tiles it reads), so the sub-blocks reproduce the block's bits.  The
// split is the smallest one whose wide staging fits the LDS of the narrow
// one (sub-blocks keep whole checkerboard pairs: even tile counts, and rows
// the store can tile); with no such split the LDS is the larger of the two.
template <int D, int TX, int TY, int NT, int CPC, int ES, int EWS>
struct WideSplit {
    template <int SX, int SY>
    static constexpr bool ok()
    {
        return TX % SX == 0 && TY % SY == 0 && (TX / SX) % 2 == 0 && (TY / SY) % 2 == 0 &&
               ((TX / SX) * D) % CPC == 0 && NT % ((TX / SX) * D / CPC) == 0;
    }
    template <int SX, int SY>
    static constexpr int bytes()
    {
        using G = BlockGeom<D, TX / SX, TY / SY, CPC>;
        return G::RWL * G::RH * EWS;
    }
    static constexpr int MAIN = BlockGeom<D, TX, TY, CPC>::RWL * BlockGeom<D, TX, TY, CPC>::RH * ES;
    static constexpr int pick()  // 0: 1x1, 1: 2x1, 2: 1x2, 3: 2x2
    {
        if (EWS == 0) return 0;
        if (bytes<1, 1>() <= MAIN) return 0;
        if (ok<2, 1>() && bytes<2, 1>() <= MAIN) return 1;
        if (ok<1, 2>() && bytes<1, 2>() <= MAIN) return 2;
        if (ok<2, 2>() && bytes<2, 2>() <= MAIN) return 3;
        if (ok<2, 2>()) return 3;
        return 0;
    }
    static constexpr int K = pick();
    static constexpr int SX = (K & 1) ? 2 : 1, SY = (K & 2) ? 2 : 1;
    static constexpr int WIDE = EWS == 0 ? 0 : bytes<(K & 1) ? 2 : 1, (K & 2) ? 2 : 1>();
    static constexpr int BYTES = MAIN > WIDE ? MAIN : WIDE;
};

template <typename EW> struct WideSize { static constexpr int v = sizeof(EW); };
template <> struct WideSize<void> { static constexpr int v = 0; };

// Waves per SIMD that the LDS of a kernel with a wide path allows (the
// larger of its narrow staging, with its row pitch, and its wide sub-blocks;
// 160 KB per CU, 4 SIMDs, at most 7).  For D = 8 the register budget is held to
// it, so that the rarely taken wide path (whose registers the compiler then
// spills, in that path only) does not lower the occupancy of the main one;
// for the other domain sizes the budget would force spills into the main
// path, and the compiler's own allocation is kept.  A workgroup of NT
// threads puts NT / 256 waves on each SIMD, so the count is a multiple of
// that; 256 bytes stand for the kernel's small static arrays.
template <int D, int TX, int TY, int NT, int CPC, int ES, int EWS, int SCHED = 0>
struct WideOcc {
    static constexpr int W = WideSplit<D, TX, TY, NT, CPC, ES, EWS>::BYTES;
    static constexpr int N = NarrowBytes<D, TX, TY, CPC, ES, SCHED>::v;
    static constexpr int lds = (W > N ? W : N) + 256;
    static constexpr int per = NT >= 256 ? NT / 256 : 1;
    static constexpr int w0 = (163840 / lds) * (NT / 64) / 4;
    static constexpr int w = ((w0 > 7 ? 7 : w0) / per) * per;
    static constexpr int v = (EWS == 0 || D != 8) ? 1 : (w < 1 ? 1 : w);
};

// Stores a staged block of TX x TY tiles: its first site is at LDS row row0
// and column off (row pitch PP), lattice row gyb (below 2 L) and column gxa +
// off.
template <int D, int TX, int TY, int NT, typename E, int PP>
__device__ __forceinline__ void store_block(const E *lds, int off, int row0, int gxa, int gyb, int L,
                                            gint32 *__restrict__ hout, int ref)
{
    // ---- store the block: aligned 16-byte chunks (LDS and global columns
    // share their alignment), masked single stores in the partial chunks
    {
        constexpr int SPR = (TX * D) / 4;  // chunk slots per row, from the first (maybe partial) one
        static_assert(NT % SPR == 0, "threads must tile whole block rows");
        constexpr int RPP = NT / SPR;   // rows per pass of the workgroup
        const int m = off & 3;
        const int slot = threadIdx.x % SPR;
        const int kslot = (off >> 2) + slot;  // LDS chunk index of this thread
        int gc = gxa + 4 * kslot;
        if (gc >= L) gc -= L;
        if (gc >= L) gc -= L;
        const bool partial = slot == 0 && m != 0;
        // chunks whose 128-byte line lies wholly inside the block row are
        // streamed past the caches; lines shared with the neighbouring block
        // go through L2, where the two halves merge (row bases are
        // line-aligned when L % 32 == 0)
        const int row_lo = 4 * (gxa + off), row_hi = row_lo + 4 * (TX * D);
        const int line = (4 * (gxa + 4 * kslot)) & ~127;
        const bool whole_line = (L % 32 == 0) && line >= row_lo && line + 128 <= row_hi &&
                                gxa + off + (TX * D) <= L;
        // (separate loops: the compiler would otherwise merge the two kinds
        // of store into one plain store)
        if (whole_line) {
            for (int r = threadIdx.x / SPR; r < (TY * D); r += RPP) {
                int gy = gyb + r;
                if (gy >= L) gy -= L;
                const E *src = lds + (row0 + r) * PP + 4 * kslot;
                store4_stream(hout + (size_t)gy * L + gc,
                              Lds4<E>::widen(*reinterpret_cast<const typename Lds4<E>::raw *>(src), ref));
            }
        } else {
            for (int r = threadIdx.x / SPR; r < (TY * D); r += RPP) {
                int gy = gyb + r;
                if (gy >= L) gy -= L;
                gint32 *row = hout + (size_t)gy * L;
                const E *src = lds + (row0 + r) * PP + 4 * kslot;
                const int4 v = Lds4<E>::widen(*reinterpret_cast<const typename Lds4<E>::raw *>(src), ref);
                if (!partial) {
                    store4(row + gc, v);
                } else {
                    if (m <= 1) row[gc + 1] = v.y;
                    if (m <= 2) row[gc + 2] = v.z;
                    row[gc + 3] = v.w;
                }
            }
        }
        // the trailing partial chunk of each row (cells 0 .. m-1)
        if (m != 0) {
            const int kt = (off >> 2) + SPR;
            int gct = gxa + 4 * kt;
            if (gct >= L) gct -= L;
            if (gct >= L) gct -= L;
            for (int r = threadIdx.x; r < (TY * D); r += NT) {
                int gy = gyb + r;
                if (gy >= L) gy -= L;
                gint32 *row = hout + (size_t)gy * L;
                const E *src = lds + (row0 + r) * PP + 4 * kt;
                row[gct] = ref + (int)src[0];
                if (m >= 2) row[gct + 1] = ref + (int)src[1];
                if (m >= 3) row[gct + 2] = ref + (int)src[2];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// One region (the TX x TY tiles of the shifted frame at bp) of sweep s, int32 heights in HBM: stage
// the region and its ring of D+1 sites in LDS, run both phases, store the
// region's tiles.  With a narrow element type that is range-checked (int8)
// it returns false, having written nothing, when some staged value could
// leave the type during the sweep.  Adds the thread's accepted count to ca
// and its share of the S2 increment to cs2.
// Host requirements: T >= TX, T >= TY, TX and TY even, RWL <= L,
// RH <= L, 16-byte aligned buffers, and for E = int16
// N * (RW + RH + 4) + D^2 <= 32767 (every staged value stays within int16
// of the reference: any two region sites are joined by a path of at most
// RW + RH - 2 bonds, each of height difference <= N, and no site gains
// more than D^2 in a sweep).
// ---------------------------------------------------------------------------
template <int D, int TX, int TY, int NT, typename E, int SCHED, int U = 8>
__device__ __forceinline__ bool region_sweep(E *lds, SurfDev &d, BlockPos bp, long long t, int ox, int oy,
                                             int *s_bad, long long &ca, long long &cs2, bool commit_here, int b)
{
    constexpr int PP = RowPitch<(int)sizeof(E), BlockGeom<D, TX, TY, 4>::RWL, SCHED>::v;
    const uint32_t s = (uint32_t)t;
    using G = BlockGeom<D, TX, TY>;
    using Q = typename std::conditional<sizeof(E) <= 2, int, long long>::type;
    constexpr bool checked = sizeof(E) == 1;
    const int L = d.L, N = d.N, T = d.T;
    const uint32_t k0 = d.key0, k1 = d.key1;
    const gint32 *__restrict__ hin = as_global(d.buf[s & 1u]);
    gint32 *__restrict__ hout = as_global(d.buf[(s + 1u) & 1u]);

    int gx0 = ox + bp.tx * D - G::RING;
    int gy0 = oy + bp.ty * D - G::RING;
    if (gx0 < 0) gx0 += L;
    if (gy0 < 0) gy0 += L;
    const int cpad = gx0 & 3;
    const int gxa = gx0 - cpad;  // LDS column c holds global column gxa + c (mod L)
    const int ref = (sizeof(E) <= 2) ? hin[(size_t)gy0 * L + gx0] : 0;

    const int off = G::RING + cpad;  // LDS column of block column 0

    int vmin = 0x7FFFFFFF, vmax = -0x7FFFFFFF;  // range of the staged heights (int8 staging)
    // ---- load the region in aligned 16-byte chunks, consecutive threads on
    // consecutive chunks (rows run on into the next), U chunks in flight per
    // thread; chunk i sits at region row i / CH, chunk column i % CH
    {
        constexpr int NCH = G::CH * G::RH;
        constexpr int FULL = NCH / (NT * U);  // groups in which every thread has U chunks
        auto fetch = [&](int i) {
            const int r = i / G::CH, cc = i - r * G::CH;
            int gy = gy0 + r;
            if (gy >= L) gy -= L;
            int gx = gxa + 4 * cc;
            if (gx >= L) gx -= L;
            if (gx >= L) gx -= L;  // a block as wide as the lattice: the region wraps twice
            return load4(hin + (size_t)gy * L + gx);
        };
        auto stage = [&](int i, const int4 &v) {
            const int r = i / G::CH, cc = i - r * G::CH;
            lds_put4<E>(lds + r * PP + 4 * cc, v, ref);
            if (checked) {
                vmin = min(vmin, min(min(v.x, v.y), min(v.z, v.w)));
                vmax = max(vmax, max(max(v.x, v.y), max(v.z, v.w)));
            }
        };
#pragma unroll 1
        for (int g = 0; g < FULL; ++g) {
            const int i0 = g * NT * U + threadIdx.x;
            int4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = fetch(i0 + u * NT);
#pragma unroll
            for (int u = 0; u < U; ++u) stage(i0 + u * NT, v[u]);
        }
        {
            const int i0 = FULL * NT * U + threadIdx.x;
            int4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * NT < NCH) v[u] = fetch(i0 + u * NT);
            // (no height is read: the loads are on their way meanwhile)
            if constexpr (SCHED == 2) BlockSteps<D, TX, TY, NT, PP, G::RH>::lay_out(lds, off, bp, T, s, k0, k1);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * NT < NCH) stage(i0 + u * NT, v[u]);
        }
    }
    if (checked) {
        // every value of the sweep stays in [min, max + N D]: heights never
        // decrease, and a tile site is never more than N D/2 above the
        // frozen sites around its tile (a path of at most D/2 bonds), whose
        // values grow by at most N D/2 in the first phase
        if (vmin - ref < -128 || (long long)vmax - ref + (long long)N * D > 127) *s_bad = 1;
    }
    __syncthreads();
    if (checked && *(volatile int *)s_bad) return false;  // uniform: the whole workgroup

    int acc = 0;
    Q q = 0;
    if constexpr (SCHED == 2) BlockSteps<D, TX, TY, NT, PP, G::RH>::phases(lds, bp, N, acc, q);
    else sweep_phases<SCHED, D, TX, TY, NT, PP, E, Q>(lds, off, bp, T, s, N, k0, k1, acc, q);
    // a deposit on h raises S2 by 2h + 1; the staged value c stands for ref + c
    ca += acc;
    cs2 += 2ll * (long long)q + (long long)acc + 2ll * (long long)ref * acc;
    // the block's sums are final: commit them before the stores
    unsigned long long before = 0;
    bool last = false;
    if (commit_here) {
        long long inc[2] = {ca, cs2};
        before = commit_sweep<NT>(d, b, inc);
    }
    // Many blocks in flight: better to wait for the count here than for the
    // stores at the block's end, and to start the block's stores together
    // (16 sweeps at L = 16384: 6.63 ms with waves 1..3 ahead, 6.50 ms so).
    if (SCHED != 2 && commit_here) {
        last = is_last(d.nblocks, before);
        __syncthreads();
    }

    store_block<D, TX, TY, NT, E, PP>(lds, off, G::RING, gxa, gy0 + G::RING, L, hout, ref);
    if (SCHED == 2 && commit_here) last = is_last(d.nblocks, before);
    if (last) finish_sweep<false>(d, t);
    return true;
}

// The SX x SY sub-blocks (shape TX x TY each) of the block at bp with wide
// staging.
template <int D, int TX, int TY, int NT, typename E, int SCHED, int SX, int SY>
__device__ __forceinline__ void wide_sweep(E *lds, SurfDev &d, BlockPos bp, long long t, int ox, int oy,
                                           int *s_bad, long long &ca, long long &cs2, int b)
{
#pragma unroll 1
    for (int j = 0; j < SY; ++j)
#pragma unroll 1
        for (int i = 0; i < SX; ++i) {
            __syncthreads();  // the previous stores have read the LDS
            region_sweep<D, TX, TY, NT, E, SCHED, 4>(lds, d, BlockPos{bp.tx + i * TX, bp.ty + j * TY, bp.dupx - i * TX, bp.dupy - j * TY}, t, ox, oy, s_bad, ca, cs2,
                                                     i == SX - 1 && j == SY - 1, b);
        }
}

// ---------------------------------------------------------------------------
// block_sweep: one sweep for every active surface of the descriptor table,
// int32 heights in HBM; one workgroup per tile block, E the LDS element
// type, EW the wider type for blocks whose range does not fit E (void: E
// always fits).  The whole sweep, its exact sums included, is this one
// launch.
// ---------------------------------------------------------------------------
template <int D, int TX, int TY, int NT, typename E, typename EW, int SCHED = 0>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(
    WideOcc<D, TX, TY, NT, 4, (int)sizeof(E), WideSize<EW>::v, SCHED>::v))) void block_sweep(SurfDev *__restrict__ descs, int nsurf,
                                                  const int *__restrict__ owner, int xmode, int xnbx)
{
    using W = WideSplit<D, TX, TY, NT, 4, (int)sizeof(E), WideSize<EW>::v>;
    using G = BlockGeom<D, TX, TY>;
    constexpr int NB = SCHED == 2 ? BlockSteps<D, TX, TY, NT, G::RWL, G::RH>::BYTES
                                  : NarrowBytes<D, TX, TY, 4, (int)sizeof(E), SCHED>::v;
    __shared__ __attribute__((aligned(16))) uint8_t lds_raw[NB > W::BYTES ? NB : W::BYTES];
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;

    const int lb = block_map(blockIdx.x, gridDim.x, xmode, xnbx);
    SurfDev &d = descs[find_surface(descs, nsurf, owner, lb)];
    const long long t = d.t;
    if (t >= d.t_end) return;
    const uint32_t s = (uint32_t)t;
    const u32x4 org = philox4x32_10(0u, 0u, s, 2u, d.key0, d.key1);
    const int ox = (int)(org.v[0] % (2u * D));
    const int oy = (int)(org.v[1] % (2u * D));
    const int b = lb - d.block_start;
    const BlockPos bp = block_pos<TX, TY>(b % d.nbx, b / d.nbx, d.T);
    long long ca = 0, cs2 = 0;
    if constexpr (SCHED == 2) BlockSteps<D, TX, TY, NT, G::RWL, G::RH>::clear((int16_t *)lds_raw, d.N);
    __syncthreads();  // s_bad (and the counts of steps) cleared
    if (__builtin_expect(!region_sweep<D, TX, TY, NT, E, SCHED>((E *)lds_raw, d, bp, t, ox, oy, &s_bad, ca, cs2,
                                                                 true, b), 0)) {
        if constexpr (!std::is_void<EW>::value)
            wide_sweep<D, TX / W::SX, TY / W::SY, NT, EW, SCHED, W::SX, W::SY>((EW *)lds_raw, d, bp, t, ox, oy,
                                                                           &s_bad, ca, cs2, b);
    }
}

// ---------------------------------------------------------------------------
// Two sweeps in one pass over the lattice.  A block of the second sweep's
// frame needs the first sweep's result on itself and RING sites around it:
// the tiles of the first frame that cover those are (TX + 4) x (TY + 3 or 4)
// tiles at most, swept in LDS from a region with a ring of its own, as
// region_sweep does; then the second sweep runs on the same staging, whose
// tiles lie cx, cy sites further in.  Half the lattice traffic, launches and
// commits per sweep, for more attempts (1.5 instead of 1.16 per counted one
// at 32 x 8 tiles).  The first sweep's tiles are counted by the block that
// holds their corner site.
//
// Each launch changes buffers, so a pair of sweeps leaves the state in the
// buffer of the wrong parity and the next pair brings it back (flip): the
// host launches this kernel twice, for four sweeps that every surface makes.
//
// Host requirements as for region_sweep with the larger region (L at least
// its rows), 2 N D <= 96 for int8, N (RW + RH + 4) + 2 D^2 <= 32767.
// Bound by the latency of a launch's parts (start, loads, four dependent
// phases, commit, stores), which a pair pays once: L = 2048 23.2 -> 18.8 us
// per sweep, L = 4096 42.4 -> 36.4; in steps (8 x 8 tiles) L = 256 13.9 ->
// 11.3, L = 1024 17.1 -> 12.9.  Where every CU is full the attempts are
// the bound, and L = 16384 takes 406 -> 431 (32 x 16 blocks): not used there.
// Blocks are full power-of-two workgroups: 12 rows of tiles and 6 waves took
// 45 us at L = 4096, 16 x 16 tiles and 4.5 waves 60.
// ---------------------------------------------------------------------------
constexpr int kTwoMargin = 4;  // more tiles a side in the first sweep

// The tiles of the first sweep: W0 x H of frame tiles from (tx0, ty0), of
// which those of even tile + row + par go first, and the ones around them.
template <int W0>
struct FirstFrame {
    int tx0, ty0, H, par, half, p0;  // tiles of the second phase, of the first
    __device__ __forceinline__ FirstFrame(int x, int y, int h)
        : tx0(x), ty0(y), H(h), par((x + y) & 1), half(W0 / 2 * h), p0(half + W0 + h) {}

    __device__ __forceinline__ void tile(int k, uint32_t p, int &ltx, int &lty) const
    {
        lty = k / (W0 / 2);
        ltx = 2 * (k % (W0 / 2)) + ((lty + par + (int)p) & 1);
        if (p == 0 && k >= half) {
            const int g = k - half;
            if (g < W0 / 2) { lty = -1; ltx = 2 * g + ((par + 1) & 1); }
            else if (g < W0) { lty = H; ltx = 2 * (g - W0 / 2) + ((par + H) & 1); }
            else { lty = g - W0; ltx = ((par + lty) & 1) ? -1 : W0; }
        }
    }
    __device__ __forceinline__ uint32_t id(int ltx, int lty, int T) const
    {
        int gtx = tx0 + ltx, gty = ty0 + lty;
        gtx = gtx < 0 ? gtx + T : gtx;
        gty = gty < 0 ? gty + T : gty;
        gtx = gtx >= T ? gtx - T : gtx;
        gty = gty >= T ? gty - T : gty;
        gtx = gtx >= T ? gtx - T : gtx;  // a region that wraps twice
        return (uint32_t)(gty * T + gtx);
    }
};

// The four phases of two sweeps in steps (see BlockSteps, whose tile order
// the second sweep takes).
template <int D, int TX, int TY, int NT>
struct PairSteps {
    using TB = TileBits<D>;
    using R = StepList<D>;
    using G = BlockGeom<D, TX + kTwoMargin, TY + kTwoMargin>;
    using F = FirstFrame<TX + kTwoMargin>;
    using Second = BlockSteps<D, TX, TY, NT, G::RWL, G::RH>;
    static constexpr int P = G::RWL, RING = D + 1;
    // each phase's first tile in the lists, and first 16 tiles
    static constexpr int K1 = G::P0, K2 = K1 + G::HALF, K3 = K2 + Second::P0, ALL = K3 + Second::HALF;
    static constexpr int G1 = (K1 + 15) / 16, G2 = G1 + (G::HALF + 15) / 16, G3 = G2 + Second::G0,
                         GROUPS = G3 + (Second::HALF + 15) / 16;
    static constexpr int IDLE = Second::IDLE, LISTS = Second::LISTS;
    static constexpr int STEPS = LISTS + ALL * D * D * kLdsWin + 8;
    static constexpr int BYTES = 2 * STEPS + 4 * TB::NCALL * GROUPS;

    static __device__ __forceinline__ void clear(int16_t *lds, int N)
    {
        int *steps = (int *)(lds + STEPS);
        for (int i = threadIdx.x; i < TB::NCALL * GROUPS; i += NT) steps[i] = 0;
        if (threadIdx.x == 0) {
            int16_t *c = lds + IDLE + 1 + P;
            c[0] = 0;
            c[-1] = c[1] = c[-P] = c[P] = (int16_t)-N;
        }
    }
    static __device__ __forceinline__ uint16_t *list(int16_t *lds, int j, int k, int stride)
    {
        return (uint16_t *)(lds + LISTS) + (j * R::NPER * ALL + k * stride) * kLdsWin;
    }
    static __device__ __forceinline__ void lay_out(int16_t *lds, int off, const F &f, BlockPos bp, int cx, int cy, int T,
                                                   uint32_t s, uint32_t k0, uint32_t k1)
    {
        int *steps = (int *)(lds + STEPS);
        for (int i = threadIdx.x; i < ALL * TB::NCALL; i += NT) {
            const int j = i / ALL, k = i - j * ALL;
            int ltx, lty, base = off, group;
            uint32_t id, p;
            if (k < K2) {
                p = k >= K1;
                const int m = p ? k - K1 : k;
                if (m >= (p ? f.half : f.p0)) continue;  // one row of tiles less
                f.tile(m, p, ltx, lty);
                id = f.id(ltx, lty, T);
                group = (p ? G1 : 0) + m / 16;
            } else {
                p = k >= K3;
                Second::tile(k - K2, ltx, lty);
                int gtx = bp.tx + ltx, gty = bp.ty + lty;
                gtx = gtx < 0 ? gtx + T : (gtx >= T ? gtx - T : gtx);
                gty = gty < 0 ? gty + T : (gty >= T ? gty - T : gty);
                id = (uint32_t)(gty * T + gtx);
                base += cx + cy * P;
                group = p ? G3 + (k - K3) / 16 : G2 + (k - K2) / 16;
            }
            const int stride = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
            const int16_t *above = lds + (lty * D + RING - 1) * P + ltx * D + base;
            const int n = lay_out_steps<D, P, 0>(list(lds, j, k, stride), stride, above,
                                                 lds_address(lds + IDLE + 1) * 0x10001u, j, id, k < K2 ? s : s + 1u, p, k0, k1);
            atomicMax(&steps[j * GROUPS + group], n);
        }
    }
    // phase ph: n tiles from list entry k, groups from g; counted(i) says
    // whether the i-th counts
    template <typename C>
    static __device__ __forceinline__ void phase(int16_t *lds, int k, int g, int n, int N, int &acc, int &q, C counted)
    {
        const int *steps = (const int *)(lds + STEPS);
        for (int i = threadIdx.x / kLdsWin; i < n; i += NT / kLdsWin) {
            int a = 0, qq = 0;
#pragma unroll 1
            for (int j = 0; j < TB::NCALL; ++j) {
                const int m = __builtin_amdgcn_readfirstlane(steps[j * GROUPS + g + i / 16]);
                const int stride = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
                make_steps<P, 0>((const uint32_t *)(list(lds, j, k + i, stride) + (threadIdx.x & (kLdsWin - 1)) * stride), m, N, a, qq);
            }
            if (counted(i)) { acc += a; q += qq; }
        }
        __syncthreads();
    }
};

template <int D, int TX, int TY, int NT, typename E, bool STEPS, int U = 8>
__device__ __forceinline__ bool region_sweep2(E *lds, SurfDev &d, BlockPos bp, long long t, uint32_t flip, int ox0,
                                              int oy0, int ox1, int oy1, int *s_bad, long long (&inc)[4],
                                              bool commit_here, int b, int nblocks)
{
    constexpr int W0 = TX + kTwoMargin;
    using G = BlockGeom<D, W0, TY + kTwoMargin>;
    constexpr int RING = G::RING, PP = RowPitch<(int)sizeof(E), G::RWL, 0>::v, LOG2D = TileBits<D>::LOG2D;
    constexpr bool checked = sizeof(E) == 1;
    const uint32_t s = (uint32_t)t;
    const int L = d.L, N = d.N, T = d.T;
    const uint32_t k0 = d.key0, k1 = d.key1;
    const gint32 *__restrict__ hin = as_global(d.buf[(s + flip) & 1u]);
    gint32 *__restrict__ hout = as_global(d.buf[(s + flip + 1u) & 1u]);

    // the block's corner, and the first frame's tile that holds the site RING
    // up and left of it
    const int X1 = ox1 + D * bp.tx, Y1 = oy1 + D * bp.ty;
    const int tx0 = (X1 - RING - ox0) >> LOG2D, ty0 = (Y1 - RING - oy0) >> LOG2D;
    const int cx = X1 - ox0 - D * tx0, cy = Y1 - oy0 - D * ty0;   // RING .. RING + D - 1
    const int H0 = (cy + D * TY + RING + D - 1) >> LOG2D;          // TY + 3 or TY + 4
    int gx0 = X1 - cx - RING, gy0 = Y1 - cy - RING;
    gx0 = gx0 < 0 ? gx0 + L : gx0 >= L ? gx0 - L : gx0;
    gy0 = gy0 < 0 ? gy0 + L : gy0 >= L ? gy0 - L : gy0;
    const int cpad = gx0 & 3, gxa = gx0 - cpad;
    const int ref = hin[(size_t)gy0 * L + gx0];
    const int off = RING + cpad;  // LDS column of the first frame's column 0
    const FirstFrame<W0> f(tx0, ty0, H0);

    int vmin = 0x7FFFFFFF, vmax = -0x7FFFFFFF;
    {
        const int nch = G::CH * (D * H0 + 2 * RING);
        auto fetch = [&](int i) {
            const int r = i / G::CH, cc = i - r * G::CH;
            int gy = gy0 + r;
            if (gy >= L) gy -= L;
            int gx = gxa + 4 * cc;
            if (gx >= L) gx -= L;
            if (gx >= L) gx -= L;
            return load4(hin + (size_t)gy * L + gx);
        };
        auto stage = [&](int i, const int4 &v) {
            const int r = i / G::CH, cc = i - r * G::CH;
            lds_put4<E>(lds + r * PP + 4 * cc, v, ref);
            if (checked) {
                vmin = min(vmin, min(min(v.x, v.y), min(v.z, v.w)));
                vmax = max(vmax, max(max(v.x, v.y), max(v.z, v.w)));
            }
        };
        int i0 = threadIdx.x;
#pragma unroll 1
        for (; i0 - (int)threadIdx.x + NT * U <= nch; i0 += NT * U) {
            int4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = fetch(i0 + u * NT);
#pragma unroll
            for (int u = 0; u < U; ++u) stage(i0 + u * NT, v[u]);
        }
        int4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * NT < nch) v[u] = fetch(i0 + u * NT);
        // (no height is read: the loads are on their way meanwhile)
        if constexpr (STEPS) PairSteps<D, TX, TY, NT>::lay_out(lds, off, f, bp, cx, cy, T, s, k0, k1);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * NT < nch) stage(i0 + u * NT, v[u]);
    }
    // (see region_sweep: a sweep raises no site by more than N D)
    if (checked && (vmin - ref < -128 || (long long)vmax - ref + 2ll * N * D > 127)) *s_bad = 1;
    __syncthreads();
    if (checked && *(volatile int *)s_bad) return false;

    // the first sweep; a tile counts where its corner lies in the block
    const int xlo = D * max(bp.dupx, 0), ylo = D * max(bp.dupy, 0);
    auto mine = [&](int ltx, int lty) {
        const int dx = D * ltx - cx, dy = D * lty - cy;
        return dx >= xlo && dx < D * TX && dy >= ylo && dy < D * TY;
    };
    int acc = 0, q = 0;
    if constexpr (STEPS) {
        using S = PairSteps<D, TX, TY, NT>;
        auto counts = [&](int m, uint32_t p) {
            int ltx, lty;
            f.tile(m, p, ltx, lty);
            return (p || m < f.half) && mine(ltx, lty);
        };
        S::phase(lds, 0, 0, f.p0, N, acc, q, [&](int m) { return counts(m, 0u); });
        S::phase(lds, S::K1, S::G1, f.half, N, acc, q, [&](int m) { return counts(m, 1u); });
    } else {
        auto tile = [&](int m, uint32_t p) {
            int a = 0, qq = 0, ltx, lty;
            f.tile(m, p, ltx, lty);
            tile_attempts<D, PP, E, int>(lds, (lty * D + RING) * PP + ltx * D + off, f.id(ltx, lty, T), s, p, N, k0, k1, a, qq);
            if ((p || m < f.half) && mine(ltx, lty)) {
                acc += a;
                q += qq;
            }
        };
        for (int m = threadIdx.x; m < f.p0; m += NT) tile(m, 0u);
        __syncthreads();
        for (int m = threadIdx.x; m < f.half; m += NT) tile(m, 1u);
        __syncthreads();
    }
    inc[0] += acc;
    inc[1] += 2ll * (long long)q + (long long)acc + 2ll * (long long)ref * acc;
    // the second
    acc = q = 0;
    if constexpr (STEPS) {
        using S = PairSteps<D, TX, TY, NT>;
        auto counts = [&](int m, int k) {
            int ltx, lty;
            S::Second::tile(k, ltx, lty);
            return m < S::Second::HALF && bp.counts(ltx, lty);
        };
        S::phase(lds, S::K2, S::G2, S::Second::P0, N, acc, q, [&](int m) { return counts(m, m); });
        S::phase(lds, S::K3, S::G3, S::Second::HALF, N, acc, q, [&](int m) { return counts(m, S::Second::P0 + m); });
    } else {
        block_phases<D, TX, TY, NT, PP, E, int>(lds, off + cx + cy * PP, bp, T, s + 1u, N, k0, k1, acc, q);
    }
    inc[2] += acc;
    inc[3] += 2ll * (long long)q + (long long)acc + 2ll * (long long)ref * acc;
    bool last = false;
    unsigned long long before = 0;
    if (commit_here) before = commit_sweep<NT, 2>(d, b, inc);
    if (commit_here && !STEPS) {
        last = is_last(nblocks, before);
        __syncthreads();
    }
    store_block<D, TX, TY, NT, E, PP>(lds, off + cx, RING + cy, gxa + off + cx >= L ? gxa - L : gxa, gy0 + RING + cy, L,
                                      hout, ref);
    if (commit_here && STEPS) last = is_last(nblocks, before);
    if (last) finish_sweep<false, 2>(d, t, flip);
    return true;
}

// Two sweeps per launch for every active surface of the descriptor table (see
// block_sweep): int8 staging with int16 sub-blocks where a block does not fit,
// or attempts in steps on int16 staging.
template <int D, int TX, int TY, int NT, bool STEPS>
__global__ __launch_bounds__(NT) void block_sweep2(SurfDev *__restrict__ descs, int nsurf, const int *__restrict__ owner,
                                                   int xmode, int xnbx)
{
    using G = BlockGeom<D, TX + kTwoMargin, TY + kTwoMargin>;
    using GS = BlockGeom<D, TX / 2 + kTwoMargin, TY / 2 + kTwoMargin>;
    constexpr int NB = RowPitch<1, G::RWL, 0>::v * G::RH, WB = GS::RWL * GS::RH * 2;
    constexpr int BYTES = STEPS ? PairSteps<D, TX, TY, NT>::BYTES : NB > WB ? NB : WB;
    __shared__ __attribute__((aligned(16))) uint8_t lds_raw[BYTES];
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;

    const int lb = block_map(blockIdx.x, gridDim.x, xmode, xnbx);
    SurfDev &d = descs[find_surface<true>(descs, nsurf, owner, lb)];
    const long long t = d.t;
    const uint32_t flip = d.flip;
    const u32x4 org0 = philox4x32_10(0u, 0u, (uint32_t)t, 2u, d.key0, d.key1);
    const u32x4 org1 = philox4x32_10(0u, 0u, (uint32_t)t + 1u, 2u, d.key0, d.key1);
    const int ox0 = (int)(org0.v[0] % (2u * D)), oy0 = (int)(org0.v[1] % (2u * D));
    const int ox1 = (int)(org1.v[0] % (2u * D)), oy1 = (int)(org1.v[1] % (2u * D));
    const int b = lb - d.block_start2;
    const int nbx = xnbx ? xnbx : (d.T + TX - 1) / TX, nblocks = nbx * ((d.T + TY - 1) / TY);
    const BlockPos bp = block_pos<TX, TY>(b % nbx, b / nbx, d.T);
    long long inc[4] = {0, 0, 0, 0};
    if constexpr (STEPS) PairSteps<D, TX, TY, NT>::clear((int16_t *)lds_raw, d.N);
    __syncthreads();  // s_bad (and the counts of steps) cleared
    if constexpr (STEPS) {
        region_sweep2<D, TX, TY, NT, int16_t, true>((int16_t *)lds_raw, d, bp, t, flip, ox0, oy0, ox1, oy1, &s_bad, inc,
                                                    true, b, nblocks);
    } else if (__builtin_expect(!region_sweep2<D, TX, TY, NT, int8_t, false>((int8_t *)lds_raw, d, bp, t, flip, ox0, oy0,
                                                                            ox1, oy1, &s_bad, inc, true, b, nblocks), 0)) {
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const int sx = (i & 1) * (TX / 2), sy = (i >> 1) * (TY / 2);
            __syncthreads();  // the previous stores have read the LDS
            region_sweep2<D, TX / 2, TY / 2, NT, int16_t, false, 4>((int16_t *)lds_raw, d,
                                                                    BlockPos{bp.tx + sx, bp.ty + sy, bp.dupx - sx, bp.dupy - sy},
                                                                    t, flip, ox0, oy0, ox1, oy1, &s_bad, inc, i == 3, b, nblocks);
        }
    }
}

// ---------------------------------------------------------------------------
// 16-bit storage.  Heights live in HBM as residues mod 2^16.  On the torus
// the restriction bounds the spread max h - min h by N L (any two sites are
// joined by a path of at most L bonds), and the mean grows by at most one per
// sweep, so while N L <= 32766 every height of a sweep lies within 2^15 of
// m0 = floor(S1 / L^2) at the sweep's start: h = m0 + int16(r - m0 mod 2^16)
// recovers it from its residue r, and the difference of any two heights is
// the int16 difference of their residues.  The sweep's last block keeps m0
// in the accumulator area.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(1))) uint16_t gu16;
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) v4u gv4u;

// two 16-bit lanes per 32-bit word, each wrapping mod 2^16
__device__ __forceinline__ uint32_t pk_sub16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b));
}
__device__ __forceinline__ uint32_t pk_add16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b));
}
__device__ __forceinline__ uint32_t pk_max16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Staging from 16-bit residues.  uint8 staging holds u = h - (h_ref - 128),
// checked to lie in [0, 255 - N D] at load time (the same bound as the int8
// staging of int32 heights); int16 staging holds h - h_ref.
template <typename E> struct Stage16;
template <> struct Stage16<uint8_t> {
    static constexpr int bias = 128;
    typedef uint2 raw;
    // 8 lanes of u (two per word) -> 8 bytes; lane maximum into umax
    __device__ static void put(uint8_t *dst, const v4u w, uint32_t &umax)
    {
        umax = pk_max16(umax, pk_max16(pk_max16(w.x, w.y), pk_max16(w.z, w.w)));
        const uint32_t lo = __builtin_amdgcn_perm(w.y, w.x, 0x06040200u);
        const uint32_t hi = __builtin_amdgcn_perm(w.w, w.z, 0x06040200u);
        *reinterpret_cast<uint2 *>(dst) = make_uint2(lo, hi);
    }
    // 8 bytes -> 8 residues (bytes spread to the low halves of 16-bit lanes)
    __device__ static v4u get(const raw r, uint32_t basep)
    {
        v4u o;
        o.x = pk_add16(__builtin_amdgcn_perm(0u, r.x, 0x0C010C00u), basep);
        o.y = pk_add16(__builtin_amdgcn_perm(0u, r.x, 0x0C030C02u), basep);
        o.z = pk_add16(__builtin_amdgcn_perm(0u, r.y, 0x0C010C00u), basep);
        o.w = pk_add16(__builtin_amdgcn_perm(0u, r.y, 0x0C030C02u), basep);
        return o;
    }
};
template <> struct Stage16<int16_t> {
    static constexpr int bias = 0;
    typedef uint4 raw;
    __device__ static void put(int16_t *dst, const v4u w, uint32_t &)
    {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(w.x, w.y, w.z, w.w);
    }
    __device__ static v4u get(const raw r, uint32_t basep)
    {
        v4u o;
        o.x = pk_add16(r.x, basep);
        o.y = pk_add16(r.y, basep);
        o.z = pk_add16(r.z, basep);
        o.w = pk_add16(r.w, basep);
        return o;
    }
};

// region_sweep on 16-bit residues: E = uint8 (range-checked; returns false
// when the region does not fit) or int16.  Host requirements as for
// region_sweep, with chunks of 8 cells: L % 8 == 0, RWL <= L, N L <= 32766,
// N D <= 96, and N (RW + RH + 4) + D^2 <= 32767 for int16.
template <int D, int TX, int TY, int NT, typename E, int SCHED, int U = 8>
__device__ __forceinline__ bool region_sweep16(E *lds, SurfDev &d, BlockPos bp, long long t, int ox, int oy,
                                               int *s_bad, long long &ca, long long &cs2, bool commit_here, int b)
{
    const uint32_t s = (uint32_t)t;
    using G = BlockGeom<D, TX, TY, 8>;
    using S = Stage16<E>;
    constexpr int PP = RowPitch<(int)sizeof(E), G::RWL, SCHED>::v;
    constexpr bool checked = sizeof(E) == 1;
    const int L = d.L, N = d.N, T = d.T;
    const uint32_t k0 = d.key0, k1 = d.key1;
    const gu16 *__restrict__ hin = (const gu16 *)d.buf[s & 1u];
    gu16 *__restrict__ hout = (gu16 *)d.buf[(s + 1u) & 1u];

    int gx0 = ox + bp.tx * D - G::RING;
    int gy0 = oy + bp.ty * D - G::RING;
    if (gx0 < 0) gx0 += L;
    if (gy0 < 0) gy0 += L;
    const int cpad = gx0 & 7;
    const int gxa = gx0 - cpad;  // LDS column c holds global column gxa + c (mod L)
    const uint32_t ref_r = hin[(size_t)gy0 * L + gx0];
    const uint32_t base_r = (ref_r - S::bias) & 0xFFFFu;  // residue of staged value 0
    const uint32_t basep = base_r * 0x10001u;

    uint32_t umax = 0;
    {
        constexpr int NCH = G::CH * G::RH;
        constexpr int FULL = NCH / (NT * U);
        auto fetch = [&](int i) {
            const int r = i / G::CH, cc = i - r * G::CH;
            int gy = gy0 + r;
            if (gy >= L) gy -= L;
            int gx = gxa + 8 * cc;
            if (gx >= L) gx -= L;
            if (gx >= L) gx -= L;
            return *reinterpret_cast<const gv4u *>(hin + (size_t)gy * L + gx);
        };
        auto stage = [&](int i, const v4u &v) {
            const int r = i / G::CH, cc = i - r * G::CH;
            v4u w;
            w.x = pk_sub16(v.x, basep);
            w.y = pk_sub16(v.y, basep);
            w.z = pk_sub16(v.z, basep);
            w.w = pk_sub16(v.w, basep);
            S::put(lds + r * PP + 8 * cc, w, umax);
        };
#pragma unroll 1
        for (int g = 0; g < FULL; ++g) {
            const int i0 = g * NT * U + threadIdx.x;
            v4u v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = fetch(i0 + u * NT);
#pragma unroll
            for (int u = 0; u < U; ++u) stage(i0 + u * NT, v[u]);
        }
        {
            const int i0 = FULL * NT * U + threadIdx.x;
            v4u v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * NT < NCH) v[u] = fetch(i0 + u * NT);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * NT < NCH) stage(i0 + u * NT, v[u]);
        }
    }
    if (checked) {
        // u = h - h_ref + 128 must lie in [0, 255 - N D] (see region_sweep);
        // |h - h_ref| < 2^15, so an out-of-range u shows as a 16-bit lane
        // above 255 - N D
        if ((int)max(umax & 0xFFFFu, umax >> 16) > 255 - N * D) *s_bad = 1;
    }
    __syncthreads();
    if (checked && *(volatile int *)s_bad) return false;

    const int off = G::RING + cpad;
    int acc = 0;
    int q = 0;
    sweep_phases<SCHED, D, TX, TY, NT, PP, E, int>(lds, off, bp, T, s, N, k0, k1, acc, q);
    // the unsigned byte staging counts acceptances negatively
    if constexpr (std::is_same<E, uint8_t>::value) acc = -acc;
    {
        // true height of staged value 0: the reference site's height,
        // recovered from m0 of the sweep's start, less the staging bias
        // (read before the block is counted: the sweep's last block
        // rewrites m0)
        const long long m0 = *(const gi64 *)(d.acc + kMeanWord);
        const long long base = m0 + (long long)(int16_t)(uint16_t)(ref_r - (uint32_t)m0) - S::bias;
        ca += acc;
        cs2 += 2ll * (long long)q + (long long)acc + 2ll * base * acc;
    }
    bool last = false;
    if (commit_here) {
        long long inc[2] = {ca, cs2};
        last = is_last(d.nblocks, commit_sweep<NT>(d, b, inc));
    }

    // ---- store: 16-byte chunks of 8 residues; 16-bit stores in the partial
    // chunks at both ends of each row
    {
        constexpr int SPR = G::BW / 8;
        static_assert(NT % SPR == 0, "threads must tile whole block rows");
        constexpr int RPP = NT / SPR;
        const int m = off & 7;
        const int slot = threadIdx.x % SPR;
        const int kslot = (off >> 3) + slot;
        int gc = gxa + 8 * kslot;
        if (gc >= L) gc -= L;
        if (gc >= L) gc -= L;
        const bool partial = slot == 0 && m != 0;
        // byte offsets within the row; rows are 128-byte aligned when L % 64 == 0
        const int row_lo = 2 * (gxa + off), row_hi = row_lo + 2 * G::BW;
        const int line = (2 * (gxa + 8 * kslot)) & ~127;
        const bool whole_line = (L % 64 == 0) && line >= row_lo && line + 128 <= row_hi &&
                                gxa + off + G::BW <= L;
        if (whole_line) {
            for (int r = threadIdx.x / SPR; r < G::BH; r += RPP) {
                int gy = gy0 + G::RING + r;
                if (gy >= L) gy -= L;
                const E *src = lds + (G::RING + r) * PP + 8 * kslot;
                __builtin_nontemporal_store(S::get(*reinterpret_cast<const typename S::raw *>(src), basep),
                                            reinterpret_cast<gv4u *>(hout + (size_t)gy * L + gc));
            }
        } else {
            for (int r = threadIdx.x / SPR; r < G::BH; r += RPP) {
                int gy = gy0 + G::RING + r;
                if (gy >= L) gy -= L;
                gu16 *row = hout + (size_t)gy * L;
                const E *src = lds + (G::RING + r) * PP + 8 * kslot;
                if (!partial) {
                    *reinterpret_cast<gv4u *>(row + gc) = S::get(*reinterpret_cast<const typename S::raw *>(src), basep);
                } else {
#pragma unroll
                    for (int k = 1; k < 8; ++k)
                        if (k >= m) row[gc + k] = (uint16_t)(base_r + (uint32_t)(int)src[k]);
                }
            }
        }
        if (m != 0) {
            const int kt = (off >> 3) + SPR;
            int gct = gxa + 8 * kt;
            if (gct >= L) gct -= L;
            if (gct >= L) gct -= L;
            for (int r = threadIdx.x; r < G::BH; r += NT) {
                int gy = gy0 + G::RING + r;
                if (gy >= L) gy -= L;
                gu16 *row = hout + (size_t)gy * L;
                const E *src = lds + (G::RING + r) * PP + 8 * kt;
#pragma unroll
                for (int k = 0; k < 7; ++k)
                    if (k < m) row[gct + k] = (uint16_t)(base_r + (uint32_t)(int)src[k]);
            }
        }
    }
    if (last) finish_sweep<true>(d, t);
    return true;
}

// int16 sub-blocks of a 16-bit storage block (see wide_sweep).
template <int D, int TX, int TY, int NT, int SCHED, int SX, int SY>
__device__ __forceinline__ void wide_sweep16(int16_t *lds, SurfDev &d, BlockPos bp, long long t, int ox, int oy,
                                             int *s_bad, long long &ca, long long &cs2, int b)
{
#pragma unroll 1
    for (int j = 0; j < SY; ++j)
#pragma unroll 1
        for (int i = 0; i < SX; ++i) {
            __syncthreads();  // the previous stores have read the LDS
            region_sweep16<D, TX, TY, NT, int16_t, SCHED, 4>(lds, d, BlockPos{bp.tx + i * TX, bp.ty + j * TY, bp.dupx - i * TX, bp.dupy - j * TY}, t, ox, oy, s_bad, ca,
                                                             cs2, i == SX - 1 && j == SY - 1, b);
        }
}

// block_sweep on 16-bit residues: uint8 staging, int16 for the blocks that
// do not fit it.
template <int D, int TX, int TY, int NT, int SCHED = 0>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WideOcc<D, TX, TY, NT, 8, 1, 2, SCHED>::v))) void block_sweep16(SurfDev *__restrict__ descs, int nsurf,
                                                    const int *__restrict__ owner, int xmode, int xnbx)
{
    using W = WideSplit<D, TX, TY, NT, 8, 1, 2>;
    constexpr int NB = NarrowBytes<D, TX, TY, 8, 1, SCHED>::v;
    __shared__ __attribute__((aligned(16))) uint8_t lds_raw[NB > W::BYTES ? NB : W::BYTES];
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;

    const int lb = block_map(blockIdx.x, gridDim.x, xmode, xnbx);
    SurfDev &d = descs[find_surface(descs, nsurf, owner, lb)];
    const long long t = d.t;
    if (t >= d.t_end) return;
    const uint32_t s = (uint32_t)t;
    const u32x4 org = philox4x32_10(0u, 0u, s, 2u, d.key0, d.key1);
    const int ox = (int)(org.v[0] % (2u * D));
    const int oy = (int)(org.v[1] % (2u * D));
    const int b = lb - d.block_start;
    const BlockPos bp = block_pos<TX, TY>(b % d.nbx, b / d.nbx, d.T);
    long long ca = 0, cs2 = 0;
    __syncthreads();  // s_bad cleared
    // twelve 16-byte loads in flight per thread (the 32 x 8 region of 16-bit
    // residues in one round of 256 threads; measured 1% faster than eight,
    // within the same registers)
    constexpr int U16 = SCHED == 0 ? 12 : 8;
    if (__builtin_expect(!region_sweep16<D, TX, TY, NT, uint8_t, SCHED, U16>(lds_raw, d, bp, t, ox, oy, &s_bad, ca,
                                                                              cs2, true, b), 0))
        wide_sweep16<D, TX / W::SX, TY / W::SY, NT, SCHED, W::SX, W::SY>((int16_t *)lds_raw, d, bp, t, ox, oy,
                                                                     &s_bad, ca, cs2, b);
}

// Zeroes up to kFills ranges of whole 16-byte words (one per blockIdx.y), by
// one launch: a fill call each leaves the stream idle between the fills
// (24 jobs admitted and run: 3445 -> 3309 us).
constexpr int kFills = 32;
struct FillList {
    int4 *p[kFills];
    int n16[kFills];
};
__global__ void zero_ranges(FillList f)
{
    int4 *p = f.p[blockIdx.y];
    const int n = f.n16[blockIdx.y];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = make_int4(0, 0, 0, 0);
}

// The record (S1, S2, A) of every surface's current time: out[3 k] for row k
// of the descriptor table.
__global__ void gather_records(const SurfDev *__restrict__ descs, int n, long long *__restrict__ out)
{
    const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (k >= n) return;
    const SurfDev &d = descs[k];
    const long long *r = d.log + 3 * d.slot;
    for (int i = 0; i < 3; ++i) out[3 * k + i] = r[i];
}

// Conversions between int32 heights and 16-bit residues, eight sites (one
// 16-byte chunk of residues) per thread and turn; n % 8 == 0, residues
// 16-byte aligned.  The int32 side is the caller's and need not be: then its
// words move one by one.  Both are bound by memory.  A readout that the 256 MiB
// cache in front of HBM cannot hold (6 bytes a site) streams past it: with one
// residue at a time L = 16384 took 493 us, so 413, L = 8192 140 and 103; what
// fits goes through it (L = 6144: 48 us, streamed 62).
__global__ void pack16(const int32_t *__restrict__ src, uint16_t *__restrict__ dst, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n / 8; i += (long long)gridDim.x * blockDim.x) {
        v4u a, b;
        if (((uintptr_t)src & 15) == 0) {
            a = ((const gv4u *)src)[2 * i];
            b = ((const gv4u *)src)[2 * i + 1];
        } else {
            const gint32 *p = as_global(src) + 8 * i;
            for (int k = 0; k < 4; ++k) {
                a[k] = (uint32_t)p[k];
                b[k] = (uint32_t)p[k + 4];
            }
        }
        const v4u o = {__builtin_amdgcn_perm(a.y, a.x, 0x05040100u), __builtin_amdgcn_perm(a.w, a.z, 0x05040100u),
                       __builtin_amdgcn_perm(b.y, b.x, 0x05040100u), __builtin_amdgcn_perm(b.w, b.z, 0x05040100u)};
        ((gv4u *)dst)[i] = o;
    }
}

constexpr long long kStreamSites = (256ll << 20) / 6;  // more sites than these stream
template <bool STREAM>
__global__ void unpack16(const uint16_t *__restrict__ src, int32_t *__restrict__ dst, long long n,
                         const long long *__restrict__ mean_floor)
{
    const int m0 = (int)*mean_floor;  // heights fit int32
    const uint32_t r0 = ((uint32_t)m0 & 0xFFFFu) * 0x10001u;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n / 8; i += (long long)gridDim.x * blockDim.x) {
        v4u v;
        if constexpr (STREAM) v = __builtin_nontemporal_load((const gv4u *)src + i);
        else v = ((const gv4u *)src)[i];
        v4u o[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t d = pk_sub16(v[k], r0);  // h - m0 in each 16-bit lane
            o[k / 2][2 * (k % 2)] = (uint32_t)(m0 + (int)(int16_t)(uint16_t)d);
            o[k / 2][2 * (k % 2) + 1] = (uint32_t)(m0 + ((int)d >> 16));
        }
        if (((uintptr_t)dst & 15) == 0) {
            if constexpr (STREAM) {
                __builtin_nontemporal_store(o[0], (gv4u *)dst + 2 * i);
                __builtin_nontemporal_store(o[1], (gv4u *)dst + 2 * i + 1);
            } else {
                ((gv4u *)dst)[2 * i] = o[0];
                ((gv4u *)dst)[2 * i + 1] = o[1];
            }
        } else {
            for (int k = 0; k < 8; ++k) as_global(dst)[8 * i + k] = (int32_t)o[k / 4][k % 4];
        }
    }
}

// ---------------------------------------------------------------------------
// Surfaces small enough to live in LDS, one workgroup each, all their sweeps
// in one launch.  which[] lists descriptor indices.
//
// A small surface is bound by the chain of dependent attempts of a tile:
// with one lane per tile L = 64 keeps 32 lanes of a CU busy, 64 attempts
// after each other.  So the attempts are made in steps (four lanes per tile);
// for L <= 64 the waves that would idle lay the steps out, one sweep ahead.
// Steps of eight would be about 20 at twice the lanes, which L = 128 does not
// have idle.  Many surfaces are bound by how many are resident: the host then
// leaves the lists ahead out (AHEAD) or takes lds_run32 (lds_plan).
//
// Heights are staged as 16-bit offsets from a base that follows the surface
// (the restriction keeps the spread below N L, the mean rises by at most one
// per sweep; needs N L <= kLdsRunMaxNL).  The array covers [0, L + 2D) in x
// and y plus a frame of one site; sweep s works on the window of side L at
// its origin (ox, oy), so no tile wraps.  Between sweeps only the strips by
// which the window moved are copied over, and the frame around the window
// (the torus neighbours of its edge) is refreshed before every phase.
//
// L = 64, D = 8: 20.4 -> 6.8 us per sweep; 192 surfaces of L = 32, 64, 128
// (bound by L = 128): 25.9 -> 14.1 us per sweep.
// ---------------------------------------------------------------------------
constexpr int kLdsRunMaxNL = 8192;
constexpr int kLdsRebase = 4096;  // sweeps between moves of the base: 2 N L + kLdsRebase < 2^15
constexpr int kLdsMaxL = 128;
constexpr int kLdsThreads = 512;  // four lanes for each of the 128 tiles of a phase at L = 128, D = 8

template <int D, bool AHEAD = true>
struct LdsRun {
    using TB = TileBits<D>;
    // one row pitch for every L: the neighbours of a site are at constant
    // offsets; an odd number of words spreads the rows over the banks
    static constexpr int P = kLdsMaxL + 2 * D + 2;
    static_assert((P / 2) % 2 == 1, "odd words per row");
    static constexpr int SHIFT = D == 32 ? 1 : 0;  // of the lists' entries
    static constexpr int NPER = StepList<D>::NPER, NLAST = StepList<D>::NLAST;

    __host__ __device__ static int lattice_rows(int L) { return L + 2 * D + 2 + 3; }  // and 3 of the idle lanes' site
    __host__ __device__ static int lattice_bytes(int L) { return (lattice_rows(L) * P * 2 + 15) & ~15; }
    // Small lattices leave waves without an attempt to make: these lay out
    // the next sweep's steps (all phases) meanwhile, into a second set of
    // lists.  The others (all, without AHEAD) lay out one phase at a time, by
    // all waves.
    __host__ __device__ static bool ahead(int L, int phases)
    {
        return AHEAD && L <= 64 && L / D * (L / D) / phases * kLdsWin <= kLdsThreads / 2;
    }
    __host__ __device__ static int list_bytes(int L, int phases)  // of one set
    {
        return L * L / (ahead(L, phases) ? 1 : phases) * kLdsWin * 2 + 16;  // one pair is read beyond the last
    }
    __host__ __device__ static int bytes(int L, int phases)
    {
        return lattice_bytes(L) + list_bytes(L, phases) * (ahead(L, phases) ? 2 : 1);
    }
};

// AHEAD false: one phase's lists at a time for every L, less LDS.
template <int D, int NT, int SCHED = 0, bool AHEAD = true>
__global__ __launch_bounds__(NT) void lds_run(SurfDev *__restrict__ descs, const int *__restrict__ which)
{
    using R = LdsRun<D, AHEAD>;
    using TB = TileBits<D>;
    constexpr int PH = SCHED == 0 ? 2 : 4, P = R::P;
    constexpr int MAXT = kLdsMaxL / D;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_dyn[];
    __shared__ int s_sum[2][2];  // by sweep parity: accepted, sum of (h - base) over accepted
    // steps of the longest of 16 tiles (one wave's), by set of lists, call
    // and group of tiles
    constexpr int GROUPS = MAXT * MAXT / 16 + PH;  // every phase's last group may be part of one
    __shared__ int s_steps[2][TB::NCALL][GROUPS];

    SurfDev &d = descs[which[blockIdx.x]];
    long long t = d.t;
    const long long t_end = d.t_end;
    if (t >= t_end) return;
    const int L = d.L, N = d.N, T = d.T, tid = threadIdx.x;
    const uint32_t k0 = d.key0, k1 = d.key1;
    const bool ahead = R::ahead(L, PH);
    const int ntiles = T * T / PH, ngroups = (ntiles + 15) / 16;
    const int all = ahead ? T * T : ntiles;   // tiles of a set of lists
    // threads that lay out steps while the others make attempts
    const int makers = min(NT, (ntiles * kLdsWin + 63) & ~63);
    int16_t *h = (int16_t *)lds_dyn + P + 1;  // site (0, 0); the frame's at index -1
    uint16_t *const lists = (uint16_t *)(lds_dyn + R::lattice_bytes(L));
    const int set = R::list_bytes(L, PH) / 2;  // entries of a set
    // a site that no attempt changes, for lanes without one: N above all its
    // neighbours
    int16_t *const idle = h + (L + 2 * D + 2) * P;  // row L + 2 D + 3 of the array
    const uint32_t idle2 = (lds_address(idle - P) >> R::SHIFT) * 0x10001u;

    auto origin = [&](long long tau, int &x, int &y) {
        const u32x4 o = philox4x32_10(0u, 0u, (uint32_t)tau, 2u, k0, k1);
        x = (int)(o.v[0] % (2u * D));
        y = (int)(o.v[1] % (2u * D));
    };
    int ox, oy;
    origin(t, ox, oy);
    int base;
    {
        const int32_t *src = d.buf[t & 1];
        base = src[0];
        for (int i = tid; i < L * L; i += NT) {
            const int y = i / L, x = i - y * L;
            h[(y < oy ? y + L : y) * P + (x < ox ? x + L : x)] = (int16_t)(src[i] - base);
        }
        for (int i = tid; i < 2 * TB::NCALL * GROUPS; i += NT) (&s_steps[0][0][0])[i] = 0;
        if (tid < 4) s_sum[tid >> 1][tid & 1] = 0;
        if (tid == 0) {
            idle[0] = 0;
            idle[-1] = idle[1] = idle[-P] = idle[P] = (int16_t)-N;
        }
    }
    // thread 0 keeps the sums
    long long S1 = 0, S2 = 0, slot = d.slot;
    if (tid == 0) {
        const long long *rec = d.log + 3 * slot;
        S1 = rec[0];
        S2 = rec[1];
    }
    __syncthreads();

    const float r_half = 1.0f / (float)(T / 2), r_tiles = 1.0f / (float)ntiles, r_all = 1.0f / (float)all;
    // tile k of phase p: its place in the window, in tiles
    auto tile_of = [&](int k, int p, int &tx, int &ty) {
        const int q = div_by(k, r_half);
        ty = SCHED == 0 ? q : 2 * q + (p >> 1);
        tx = 2 * (k - q * (T / 2)) + (SCHED == 0 ? (ty + p) & 1 : p & 1);
    };
    // the torus neighbours of the window's edge (kLdsMaxL threads a side)
    auto frame = [&]() {
#pragma unroll
        for (int i = 0; i < 4 * kLdsMaxL; i += NT) {
            const int side = (i + tid) / kLdsMaxL, k = (i + tid) % kLdsMaxL;
            if (k >= L) continue;
            int16_t *row = h + (oy + k) * P + ox, *col = h + oy * P + ox + k;
            int16_t *to = side == 0 ? row - 1 : side == 1 ? row + L : side == 2 ? col - P : col + L * P;
            const int16_t *from = side == 0 ? row + L - 1 : side == 1 ? row : side == 2 ? col + (L - 1) * P : col;
            *to = *from;
        }
    };
    // lists of the phases from p on that a set holds, for the window at
    // (x, y), by threads `first` .. of the `nthr`
    auto lay_out = [&](uint32_t s, int p, int half, int x, int y, int first, int nthr) {
        for (int i = first; i < all * TB::NCALL; i += nthr) {
            // consecutive lanes take consecutive tiles
            const int j = div_by(i, r_all), i2 = i - j * all, g = ahead ? div_by(i2, r_tiles) : 0;
            const int k = i2 - g * ntiles;
            int tx, ty;
            tile_of(k, p + g, tx, ty);
            const int stride = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
            const int n = lay_out_steps<D, P, R::SHIFT>(lists + half * set + j * R::NPER * all * kLdsWin + i2 * kLdsWin * stride,
                                           stride, h + (y + ty * D - 1) * P + x + tx * D, idle2, j, (uint32_t)(ty * T + tx), s,
                                           (uint32_t)(SCHED == 0 ? p + g : 4 + p + g), k0, k1);
            atomicMax(&s_steps[half][j][g * ngroups + (k >> 4)], n);
        }
    };

    int half = 0;
    if (ahead) {
        lay_out((uint32_t)t, 0, 0, ox, oy, tid, NT);
    }
    for (int run = 0; t < t_end; ++t) {
        const uint32_t s = (uint32_t)t;
        int nx = ox, ny = oy;
        if (t + 1 < t_end) origin(t + 1, nx, ny);
        frame();
        int acc = 0, q = 0;
#pragma unroll 1
        for (int p = 0; p < PH; ++p) {
            if (!ahead) lay_out(s, p, 0, ox, oy, tid, NT);
            __syncthreads();
            if (ahead && tid >= makers && p == 0 && t + 1 < t_end)
                lay_out(s + 1u, 0, half ^ 1, nx, ny, tid - makers, NT - makers);
            for (int k = tid / kLdsWin; k < ntiles; k += NT / kLdsWin) {
                const int g = ahead ? p : 0;
                int *const nsteps = &s_steps[half][0][g * ngroups + (k >> 4)];
                const uint16_t *e0 = lists + half * set;
#pragma unroll 1
                for (int j = 0; j < TB::NCALL; ++j) {
                    const int n = __builtin_amdgcn_readfirstlane(nsteps[j * GROUPS]);
                    const int stride = j == TB::NCALL - 1 ? R::NLAST : R::NPER;
                    const uint32_t *e = (const uint32_t *)(e0 + j * R::NPER * all * kLdsWin +
                                               ((g * ntiles + k) * kLdsWin + (tid & (kLdsWin - 1))) * stride);
                    make_steps<P, R::SHIFT>(e, n, N, acc, q);
                    nsteps[j * GROUPS] = 0;
                }
            }
            __syncthreads();
            if (p + 1 < PH) frame();
        }
        half ^= ahead ? 1 : 0;
        acc = wave_sum63(acc);
        q = wave_sum63(q);
        if ((tid & 63) == 63 && acc) {
            atomicAdd(&s_sum[s & 1][0], acc);
            atomicAdd(&s_sum[s & 1][1], q);
        }
        // the next window: strips of columns, then of rows
        {
            const int wx = abs(nx - ox), wy = abs(ny - oy), x0 = min(nx, ox), y0 = min(ny, oy);
            if ((tid & (2 * D - 1)) < wx)
                for (int y = tid / (2 * D); y < L; y += NT / (2 * D)) {
                    int16_t *c = h + (oy + y) * P + x0 + (tid & (2 * D - 1));
                    if (nx > ox) c[L] = c[0];
                    else c[0] = c[L];
                }
            ox = nx;
            __syncthreads();
            if ((tid & (kLdsMaxL - 1)) < L)
                for (int y = tid / kLdsMaxL; y < wy; y += NT / kLdsMaxL) {
                    int16_t *c = h + (y0 + y) * P + ox + (tid & (kLdsMaxL - 1));
                    if (ny > oy) c[L * P] = c[0];
                    else c[0] = c[L * P];
                }
            oy = ny;
        }
        __syncthreads();
        if (tid == 0) {
            const int a = s_sum[s & 1][0];
            const long long c = (long long)s_sum[s & 1][1] + (long long)base * a;
            s_sum[s & 1][0] = s_sum[s & 1][1] = 0;
            S1 += a;
            S2 += 2 * c + a;  // a deposit on h raises h^2 by 2 h + 1
            slot = slot + 1 == d.log_cap ? 0 : slot + 1;
            long long *e = d.log + 3 * slot;
            e[0] = S1;
            e[1] = S2;
            e[2] = a;
        }
        if (++run == kLdsRebase) {
            run = 0;
            const int v0 = h[oy * P + ox];
            __syncthreads();
            for (int i = tid; i < L * L; i += NT) {
                const int y = i / L;
                h[(oy + y) * P + ox + i - y * L] -= (int16_t)v0;
            }
            base += v0;
            __syncthreads();
        }
    }
    {
        int32_t *dst = d.buf[t_end & 1];
        for (int i = tid; i < L * L; i += NT) {
            const int y = i / L, x = i - y * L;
            dst[i] = base + h[(y < oy ? y + L : y) * P + (x < ox ? x + L : x)];
        }
    }
    if (tid == 0) {
        d.t = t_end;
        d.slot = slot;
    }
}

// ---------------------------------------------------------------------------
// lds_run32: the same for restrictions with N L > kLdsRunMaxNL (up to none at
// all) and for small tiles that fill the lanes: int32 heights on the bare
// torus, one lane per tile, the LDS is L_max^2 int32.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ int tile_attempts_torus(int32_t *h, int L, int x0, int y0,
                                                   uint32_t tile_id, uint32_t s, uint32_t p, int N,
                                                   uint32_t k0, uint32_t k1)
{
    using TB = TileBits<D>;
    int acc = 0;
#pragma unroll 1
    for (int j = 0; j < TB::NCALL; ++j) {
        const u32x4 r = philox4x32_10((uint32_t)j, tile_id, s, p, k0, k1);
#pragma unroll
        for (int q = 0; q < TB::PER; ++q) {
            if (j * TB::PER + q < D * D) {
                const uint32_t f = (r.v[q / TB::F] >> ((q % TB::F) * TB::B)) & (uint32_t)(D * D - 1);
                int x = x0 + (int)(f & (D - 1));
                int y = y0 + (int)(f >> TB::LOG2D);
                if (x >= L) x -= L;
                if (y >= L) y -= L;
                const int xl = x == 0 ? L - 1 : x - 1, xr = x == L - 1 ? 0 : x + 1;
                const int yu = y == 0 ? L - 1 : y - 1, yd = y == L - 1 ? 0 : y + 1;
                const int c = h[y * L + x];
                const int m = min(min(h[y * L + xl], h[y * L + xr]), min(h[yu * L + x], h[yd * L + x]));
                const int ok = (c - m) < N;
                h[y * L + x] = c + ok;
                acc += ok;
            }
        }
    }
    return acc;
}

template <int D, int NT, int SCHED = 0>
__global__ __launch_bounds__(NT) void lds_run32(SurfDev *__restrict__ descs, const int *__restrict__ which)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_dyn[];
    int32_t *lat = (int32_t *)lds_dyn;
    SurfDev &d = descs[which[blockIdx.x]];
    long long t = d.t;
    const long long t_end = d.t_end;
    if (t >= t_end) return;
    const int L = d.L, N = d.N, T = d.T;
    const int n = L * L;
    const uint32_t k0 = d.key0, k1 = d.key1;
    {
        const int32_t *src = d.buf[t & 1];
        for (int i = threadIdx.x; i < n; i += NT) lat[i] = src[i];
    }
    __syncthreads();
    const int half = T * T / 2;
    for (; t < t_end; ++t) {
        const uint32_t s = (uint32_t)t;
        const u32x4 org = philox4x32_10(0u, 0u, s, 2u, k0, k1);
        const int ox = (int)(org.v[0] % (2u * D));
        const int oy = (int)(org.v[1] % (2u * D));
        long long acc = 0;
        if constexpr (SCHED == 0) {
            for (int p = 0; p < 2; ++p) {
                for (int k = threadIdx.x; k < half; k += NT) {
                    const int ty = k / (T / 2);
                    const int tx = 2 * (k % (T / 2)) + ((ty + p) & 1);
                    acc += tile_attempts_torus<D>(lat, L, ox + tx * D, oy + ty * D,
                                                  (uint32_t)(ty * T + tx), s, (uint32_t)p, N, k0, k1);
                }
                __syncthreads();
            }
        } else {
            // double tiling: set p = (sx mod 2) + 2 (sy mod 2), phase code 4 + p
            for (int p = 0; p < 4; ++p) {
                for (int k = threadIdx.x; k < half / 2; k += NT) {
                    const int sy = 2 * (k / (T / 2)) + (p >> 1);
                    const int sx = 2 * (k % (T / 2)) + (p & 1);
                    acc += tile_attempts_torus<D>(lat, L, ox + sx * D, oy + sy * D,
                                                  (uint32_t)(sy * T + sx), s, 4u + (uint32_t)p, N, k0, k1);
                }
                __syncthreads();
            }
        }
        long long s1 = 0, s2 = 0;
        for (int i = threadIdx.x; i < n; i += NT) {
            const long long v = lat[i];
            s1 += v;
            s2 += v * v;
        }
        block_reduce3<NT>(s1, s2, acc);
        if (threadIdx.x == 0) {
            long long *e = d.log + 3 * ((t + 1) % d.log_cap);
            e[0] = s1;
            e[1] = s2;
            e[2] = acc;
        }
        __syncthreads();
    }
    {
        int32_t *dst = d.buf[t_end & 1];
        for (int i = threadIdx.x; i < n; i += NT) dst[i] = lat[i];
    }
    if (threadIdx.x == 0) {
        d.t = t_end;
        d.slot = t_end % d.log_cap;
    }
}

}  // namespace rsosk
