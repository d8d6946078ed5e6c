// Exhaustive NCC block matching of 12-bit volumes on the gfx950 matrix cores.
//
// The cross term of the NCC equation (section 3), X(d) = sum_o T(o) F(o + d)
// over the block's voxels o, is one sliding correlation per block: a single
// template against its search window.  A single template is a matrix-vector
// product, which matrix cores cannot use; this kernel gives it a second
// matrix dimension by letting the 16 columns of a 16x16x32 fp16 MFMA be a
// 4x4 patch of (dx, dy) displacement offsets, so the block operand is the
// block T written out once per offset (a zero-padded Toeplitz matrix):
//
//   C[m][n] = sum_{x', y', s} F(p_m + (x', y', s)) * T(x' - a_n, y' - b_n, s)
//
// where row m is a window base position p_m = (bx, by, dz) and column n the
// offset (a_n, b_n); C[m][n] is the cross term of displacement
// (bx + a_n, by + b_n, dz).  K runs over the plane s of the block and the
// 4-column by 2-row groups of (x', y') that any column of the patch touches.
//
// Exactness and precision: 12-bit voxels centred on an integer c are exact in
// fp16 when |v - c| <= 2048.  The block and its window take a constant each,
// both starting at the block's rounded mean: c_T clamped into [max - 2048,
// min + 2048] over the block, c_F into the same interval over the window
// (neither is ever empty for 12-bit data), so every product is exact and only
// the FP32 accumulation rounds.  T - c_T sums to at most about N/2 in
// magnitude, so the terms that cancel in N X - S_T S_F stay small even where
// the window holds values far from the block's (a single constant clamped
// over both would leave T - c far from zero mean there, and FP32 partial sums
// N times the covariance's size); F - c_F is centred for the displacements
// that look like the block, where the ranking has to be accurate.  The
// ranking key follows the exact integer window statistics, and the winner's
// NCC is recomputed in exact integer arithmetic from the staged operands.
//
// Data flow of one workgroup (one selected block).  What bounds it is latency:
// 5508 blocks of the 256x256x124 workload (b = 7, W = 10) pass two at a time
// through each of 256 CUs, and a wavefront used to spend 72,000 cycles on a
// block, of which the products and their ranking were 18,600 (cycle stamps
// per phase).  So the phases are arranged to wait for memory once:
//  * every load of the block (its voxels, then the window's 16-byte row
//    chunks, at most KREG per thread) is issued at the start, into registers;
//  * while the window's loads return, the block's sums give its centre and
//    T - c goes to four zero-bordered fp16 tables (one per x offset, so that
//    the reads are aligned), from which each wavefront builds its Toeplitz B
//    operands once (they stay in registers for the whole block);
//  * the window's value range then gives its centre, and the window is written
//    to LDS once, as fp16 (v - c), over the tables, two rows interleaved so
//    that an A operand is one 16-byte read;
//  * each wavefront sweeps the window planes for a tile of 16 bases: the A
//    operand loaded for plane p feeds the accumulators of every displacement
//    plane dz = p - s that uses it (s = 0..b-1), a ring of b accumulator
//    tiles indexed at compile time; the tile whose last plane was just added
//    is ranked (key = N cov * rsqrt(N varF) from the statistics table) and
//    its slot reused;
//  * bases cover the valid (dx, dy) range in steps of 4; the displacement
//    planes are split into phases so that tiles = ceil(bases * phases / 16)
//    balance over the workgroup's wavefronts; a table in LDS, filled while the
//    loads are in flight, says which base and phase a tile's row is;
//  * argmax: largest key, smallest shift index among equal keys, reduced over
//    lanes (by DPP moves), wavefronts and the workgroup.
//
// One 256-thread workgroup per selected block, two co-resident per CU up to
// b = 7: the latencies of one are hidden behind the matrix work of the other.
// Measured against the earlier form (window staged raw in two rounds, centred
// in place, operands from one table by 2-byte reads, 64-bit record addresses,
// shuffle reductions): the search takes 0.160 ms instead of 0.356 on
// 256x256x124 (b = 7, W = 10, 5508 blocks), 30.8 instead of 57.1 ms on 512x512x256
// (b = 9, W = 12, 357,035 blocks); the keys and the winners are the same bits.
// Of the 0.160 ms, 0.08 are the phases around the sweep (a variant without it),
// 0.05 the matrix instructions; at b = 9 (one wavefront per SIMD) the sweep's
// products and ranking add up.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <type_traits>
#include <utility>

#include "nrr_internal.h"
#include "record_planes.h"
#include "wave64.h"

namespace nrr {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));  // volume rows
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));

constexpr int OFF = 3;  // zero border of the T table (offsets 0..3)

// Compile-time sizes of the K layout for block edge B, and of the block
// tables the B operands are read from: four copies of T - c (offset a's
// values moved right by a columns, so that every operand half is an aligned
// 8-byte read), each with OFF zero rows above.
template <int B>
struct KGeo {
    static constexpr int GX = (B + 3 + 3) / 4;   // x' groups of 4 (x' extent B + 3)
    static constexpr int GYP = (B + 3 + 1) / 2;  // y' row pairs (y' extent B + 3)
    static constexpr int NG = GX * GYP;          // k-groups of 8 per block plane
    static constexpr int NQ = (NG + 3) / 4;      // 32-wide K chunks per block plane
    static constexpr int TXW = 4 * GX;           // T table row width (halves)
    static constexpr int TYW = 2 * GYP + OFF;    // T table rows per plane
    static constexpr int TCOPY = B * TYW * TXW;  // halves per copy
    static constexpr int T_BYTES = (4 * TCOPY * 2 + 15) & ~15;
};

struct MfParams {
    const uint16_t *ref;
    const uint16_t *flt;
    int nx, ny, nz;
    const int32_t *centers;
    int64_t first;  // first block of this launch
    int w;
    const StatU16 *stats;
    int64_t nstat;  // records of the table
    int ox, oy;
    int rp2;       // LDS pitch of a pair of window rows (halves)
    int tab_off;   // LDS byte offset of the tile-row table
    int tz[2];     // phase length of an unclipped window, x parity shift 0 / 1
    int32_t *disp;
    float *ncc;
    float *conf;
    // optional [n][2w+1]^3 ranking NCC of every valid displacement (the
    // diagnostic instantiation only)
    float *surface;
};

__device__ inline int64_t xcd_order(int64_t wg, int64_t n) {
    const int64_t q = n / 8, r = n % 8, k = wg % 8, j = wg / 8;
    return k * q + (k < r ? k : r) + j;
}

__device__ inline void keep_best(float &bk, int &bi, float k, int i) {
    const bool take = (k > bk) | ((k == bk) & (i < bi));  // no short-circuit branches
    bk = take ? k : bk;
    bi = take ? i : bi;
}

__device__ inline void put(const MfParams &p, int64_t blk, int dx, int dy, int dz, float v) {
    p.disp[3 * blk] = dx;
    p.disp[3 * blk + 1] = dy;
    p.disp[3 * blk + 2] = dz;
    p.ncc[blk] = v;
    p.conf[blk] = v > 0.0f ? v : 0.0f;
}

// Of the wavefront (valid in lane 63).
__device__ inline int wave_sum(int v) {  // 32-bit sums, wrapping
    dpp_steps([&](auto move) { v += (int)move(0u, (uint32_t)v); });
    return v;
}
__device__ inline u16x2 wave_min(u16x2 v) {
    dpp_steps([&](auto move) {
        const uint32_t o = move(0xffffffffu, __builtin_bit_cast(uint32_t, v));
        v = __builtin_elementwise_min(v, __builtin_bit_cast(u16x2, o));
    });
    return v;
}

constexpr int MAX_NW = 4;  // wavefronts per workgroup
struct MfSmall {
    int sum[MAX_NW][3];
    uint32_t mm[MAX_NW];  // block value range: min | (4095 - max) << 16
    uint32_t wm[MAX_NW];  // window value range, the same
    float key[MAX_NW];
    int idx[MAX_NW];
};

// Fewest wavefront rounds of (MFMAs of a tile + per-step overhead): phase
// length tz (a multiple of b) for bases nxy and dzn displacement planes.
__host__ __device__ inline int best_phase(int nxy, int dzn, int b, int nq, int nw) {
    int best = b;
    float bc = 3.0e38f;
    for (int tz = b; tz < dzn + b; tz += b) {
        const int ph = (dzn + tz - 1) / tz;
        const int tiles = (nxy * ph + 15) / 16;
        const int rounds = (tiles + nw - 1) / nw;
        const float c = rounds * ((float)tz * b * nq + 3.0f * (tz + b - 1));
        if (c < bc) {
            bc = c;
            best = tz;
        }
    }
    return best;
}

// Search geometry of one block: valid displacement range per axis (the
// displaced block inside the volume), the window origin, and the staged
// region.  Rows are staged from the even element at or before the window's
// first column (volumes with an even row length), so window column x sits at
// LDS column x + px; the tiles' x bases are LDS columns 4i.
//
// Tile decomposition of the displacements: bases every 4 voxels in x and y
// (nbx x nby of them); the displacement planes in `nph` phases of `tz` planes
// each, tz a multiple of the block edge so the sweep's ramps fall on whole
// unrolled blocks of steps (planes past the valid range are computed and
// masked).  A tile is 16 rows (base, phase).
//
// LDS layout of the window: rows two by two (the two window rows a K group
// of 8 reads are always an even row and the next), 4 columns of the upper
// row then the same 4 of the lower, so an A operand is one aligned 16-byte
// read.
struct BGeo {
    int cx, cy, cz;
    bool inside;
    int lox, loy, loz, dxn, dyn, dzn;
    int wx0, wy0, wz0, ex, ey, ez, px;
    int nbx, nby, cpr;  // bases per axis, 8-column chunks per staged row
    int eyp;            // staged rows per plane (even; a row past the window repeats the last)
    int rp2, pl;        // LDS pitch of a row pair and of a plane (halves)
    int tz, nph, nrows, ntiles;
};

template <int B>
__device__ inline BGeo block_geo(const MfParams &p, int64_t blk) {
    using G = KGeo<B>;
    constexpr int H = (B - 1) / 2;
    BGeo g;
    g.cx = p.centers[3 * blk];
    g.cy = p.centers[3 * blk + 1];
    g.cz = p.centers[3 * blk + 2];
    g.inside = g.cx - H >= 0 && g.cy - H >= 0 && g.cz - H >= 0 && g.cx + H <= p.nx - 1 &&
               g.cy + H <= p.ny - 1 && g.cz + H <= p.nz - 1;
    g.lox = max(-p.w, H - g.cx);
    g.loy = max(-p.w, H - g.cy);
    g.loz = max(-p.w, H - g.cz);
    g.dxn = min(p.w, p.nx - 1 - H - g.cx) - g.lox + 1;
    g.dyn = min(p.w, p.ny - 1 - H - g.cy) - g.loy + 1;
    g.dzn = min(p.w, p.nz - 1 - H - g.cz) - g.loz + 1;
    g.wx0 = g.cx - H + g.lox;
    g.wy0 = g.cy - H + g.loy;
    g.wz0 = g.cz - H + g.loz;
    g.ex = g.dxn + B - 1;
    g.ey = g.dyn + B - 1;
    g.ez = g.dzn + B - 1;
    g.px = (p.nx & 1) == 0 ? (g.wx0 & 1) : 0;
    g.nbx = (g.dxn + g.px + 3) / 4;
    g.nby = (g.dyn + 3) / 4;
    g.cpr = (4 * (g.nbx - 1) + 4 * G::GX + 7) / 8;
    g.eyp = (g.ey + 1) & ~1;
    g.rp2 = p.rp2;
    g.pl = (g.eyp / 2) * g.rp2;
    return g;
}

template <int B, int NW>
__device__ inline void block_tiles(const MfParams &p, BGeo &g) {
    const int d = 2 * p.w + 1, nxy = g.nbx * g.nby;
    g.tz = g.dxn == d && g.dyn == d && g.dzn == d ? p.tz[g.px]
                                                  : best_phase(nxy, g.dzn, B, KGeo<B>::NQ, NW);
    g.nph = (g.dzn + g.tz - 1) / g.tz;
    g.nrows = nxy * g.nph;
    g.ntiles = (g.nrows + 15) / 16;
}

// Tile rows as packed table entries: x base index, y base index, phase, and
// whether the row exists (rows past the last repeat row 0, masked).
__device__ inline uint32_t row_entry(const BGeo &g, int r) {
    const bool real = r < g.nrows;
    const int rr = real ? r : 0, nxy = g.nbx * g.nby;
    const int ph = quotient(rr, nxy), xy = rr - ph * nxy;
    const int yi = quotient(xy, g.nbx), xi = xy - yi * g.nbx;
    return (uint32_t)xi | (uint32_t)yi << 8 | (uint32_t)ph << 16 | (real ? 1u << 24 : 0u);
}

// The chunk 8 columns wide that starts `sh` voxels after the 16 bytes v, the
// volume's last: voxels past the end repeat the last pair.
__device__ inline u32x4 shift_chunk(u32x4 v, int sh) {
    const uint32_t h[4] = {v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16,
                           v[2] >> 16 | v[3] << 16, v[3] >> 16 | (v[3] & 0xffff0000u)};
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = sh & 1 ? h[j] : v[j];
    v = sh & 2 ? u32x4{v[1], v[2], v[3], v[3]} : v;
    return sh & 4 ? u32x4{v[2], v[3], v[3], v[3]} : v;
}

// One unrolled block of B sweep steps t0 .. t0 + B - 1 (t0 a multiple of B):
// MODE 0 is the first block (plane s of the block only reaches displacement
// planes tau = t - s >= 0), MODE 1 a full block, MODE 2 the last one (B - 1
// steps, tau = t - s < tz).  The accumulator of tau is slot tau mod B; after
// step t, plane tau = t - B + 1 is complete and `rank` takes it.
template <int B, int NQ, int MODE, typename LoadA, typename Rank>
__device__ __attribute__((always_inline)) inline void sweep_block(
    int t0, float4v (&acc)[B], const half8 (&bop)[B][NQ], half8 (&aop)[NQ], LoadA load_a,
    Rank rank) {
    constexpr int STEPS = MODE == 2 ? B - 1 : B;
    static_for<STEPS>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        const int t = t0 + u;
        // consecutive products feed different accumulators, and the plane
        // completed by this step (block plane B - 1) is fed first in each
        // chunk, so its sums are ready when the ranking reads them
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const int s = B - 1 - k;
                if (MODE == 0 && s > u) continue;
                if (MODE == 2 && s <= u) continue;
                const int slot = (u - s + B) % B;
                acc[slot] =
                    __builtin_amdgcn_mfma_f32_16x16x32_f16(aop[q], bop[s][q], acc[slot], 0, 0, 0);
            }
        // the next plane's operand replaces this one (its reads are issued
        // behind the products above and complete while the ranking runs)
        load_a(t + 1, aop);
        constexpr int fs = (u + 1) % B;
        if (MODE != 0 || u == B - 1) rank(acc[fs], t - (B - 1), std::integral_constant<int, fs>());
        acc[fs] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    });
}

// Toeplitz B operands of this lane for every block plane and K chunk, from
// the zero-bordered copies of T - c: column (oa, ob) reads copy oa, ob rows
// up.
template <int B>
__device__ __attribute__((always_inline)) inline void build_bop(
    const _Float16 *tt, int lane, half8 (&bop)[B][KGeo<B>::NQ]) {
    using G = KGeo<B>;
    const int grp = lane >> 4, oa = lane & 3, ob = (lane >> 2) & 3;
#pragma unroll
    for (int q = 0; q < G::NQ; ++q) {
        const int g = 4 * q + grp;
        const bool real = g < G::NG;
        // groups past the last read two of the zero rows
        const int gx = g % G::GX, gy = g / G::GX;
        const _Float16 *tr =
            tt + oa * G::TCOPY + (real ? (2 * gy - ob + OFF) * G::TXW + 4 * gx : 0);
#pragma unroll
        for (int s = 0; s < B; ++s) {
            const half4 lo = *reinterpret_cast<const half4 *>(tr + s * G::TYW * G::TXW);
            const half4 hi = *reinterpret_cast<const half4 *>(tr + (s * G::TYW + 1) * G::TXW);
            bop[s][q] = half8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    }
}

// This wavefront's tiles of the block's search over the centred window
// `win`: keeps the lane's best (key, shift index).  key = (N C - S_T S_F) *
// rsqrt(N varF), with S_T = sum (T - c_T) and S_F = sum (F - c_F) = s + N
// (2048 - c_F) (the table's s sums F - 2048): S_T S_F = S_T s + S_T N (2048 -
// c_F), both terms in FP32 from exact integers (relative error 2^-24 of
// terms at most |S_T| N 2048).
//
// WIDE: volumes whose window spans more than 2 GiB of records; the records
// are read through 64-bit addresses, clamped into the valid range.  Else
// through a buffer descriptor of the table from the step's plane on
// (record_planes.h): one 32-bit offset per row, the plane added to the
// descriptor's base, and reads past the table's end (planes that are masked)
// return 0 by its range check.
template <int B, int NW, bool SURF, bool WIDE>
__device__ __attribute__((always_inline)) inline void sweep_tiles(
    const MfParams &p, const BGeo &g, int64_t blk, const _Float16 *win, const uint32_t *rowtab,
    const half8 (&bop)[B][KGeo<B>::NQ], long long sTc, float inv_vt, int cf, int wave, int lane,
    float &bk, int &bi) {
    using G = KGeo<B>;
    constexpr int N = B * B * B, NQ = G::NQ;
    const int n16 = lane & 15, grp = lane >> 4;
    const int oa = n16 & 3, ob = n16 >> 2;
    const float fN = (float)N, fST = (float)sTc;
    const float fshift = (float)(sTc * (long long)N * (2048 - cf));
    const int side = 2 * p.w + 1, side2 = side * side;
    const int plane_rec = p.oy * p.ox;
    const int64_t corner = ((int64_t)g.wz0 * p.oy + g.wy0) * p.ox + g.wx0;
    const StatU16 *srec = p.stats + corner;
    int kq[NQ];  // this lane's K group of each chunk, from its row's base
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int gg = 4 * q + grp < G::NG ? 4 * q + grp : 0;
        kq[q] = (gg / G::GX) * g.rp2 + (gg % G::GX) * 8;
    }
    for (int tile = wave; tile < g.ntiles; tile += NW) {
        // the lane's A row (base of row n16): window halves at abase + kq,
        // plane aph + t, which advances while t < alim
        int abase, alim;
        {
            const uint32_t e = rowtab[16 * tile + n16];
            const int aph = (int)(e >> 16 & 0xff) * g.tz;
            abase = min(aph, g.ez - 1) * g.pl + (int)(e >> 8 & 0xff) * 2 * g.rp2 +
                    (int)(e & 0xff) * 8;
            alim = g.ez - 1 - aph;
        }
        // the lane's four output rows: displacement (odx, ody) relative to the
        // valid range's corner, plane offset oph.  Plane tau is ranked while
        // tau < lim (lim = -1 for rows outside the valid range), shift index
        // oidx + tau side^2; its record is at roff + tau planes (WIDE: at
        // rcur, which advances by a plane while tau < lim3 = dzn - 1 - oph)
        int lim[4], lim3[4], oidx[4];
        uint32_t roff[4];
        int64_t rcur[4];
        const uint4 ent = *reinterpret_cast<const uint4 *>(rowtab + 16 * tile + 4 * grp);
        const uint32_t ents[4] = {ent.x, ent.y, ent.z, ent.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t e = ents[i];
            const int odx = 4 * (int)(e & 0xff) + oa - g.px;
            const int ody = 4 * (int)(e >> 8 & 0xff) + ob;
            const int oph = (int)(e >> 16 & 0xff) * g.tz;
            const bool orow = (e >> 24) && odx >= 0 && odx < g.dxn && ody < g.dyn;
            const int cell = min(ody, g.dyn - 1) * p.ox + min(max(odx, 0), g.dxn - 1);
            if constexpr (WIDE)
                rcur[i] = (int64_t)cell + (int64_t)min(oph, g.dzn - 1) * plane_rec;
            else
                roff[i] = (uint32_t)(cell + min(oph, g.dzn - 1) * plane_rec) *
                          (uint32_t)sizeof(StatU16);
            lim[i] = orow ? g.dzn - oph : -1;
            lim3[i] = g.dzn - 1 - oph;
            oidx[i] = (g.loz + oph + p.w) * side2 + (g.loy + ody + p.w) * side +
                      (g.lox + odx + p.w);
        }
        float4v acc[B];
#pragma unroll
        for (int k = 0; k < B; ++k) acc[k] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
        // A operand of plane t + phase (clamped: planes past the window feed
        // only displacements that are masked out)
        auto read_a = [&](half8 (&aop)[NQ]) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                aop[q] = *reinterpret_cast<const half8 *>(win + abase + kq[q]);
        };
        auto load_a = [&](int t, half8 (&aop)[NQ]) {
            abase += t <= alim ? g.pl : 0;
            read_a(aop);
        };
        // statistics records of the four output rows, loaded AHEAD displacement
        // planes before their ranking, in a ring indexed like the accumulators
        // (AHEAD of its B slots are live)
        // (a record's round trip is longer than a step: one plane ahead left the
        // ramps waiting, 42.4 against 32.6 ms on the dense workload; at b = 7 the
        // registers allow three)
        constexpr int AHEAD = B == 7 ? 3 : B;
        StatU16 rec[B][4];
        RecordPlanes at;
        at.start(p.stats, p.nstat, corner, sizeof(StatU16));
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char *>(at.base), 0, (int)at.bytes, 0x00020000);
        // of the plane fetched next (planes in order), added to the lanes' offsets
        // load by load: a descriptor per plane cost the steps' scalar issue (b = 7 208
        // us against 204, dense b = 9 31.3 ms against 31.0), sums kept ahead by the
        // compiler registers (13 spilled at b = 7: 213 us)
        uint32_t plane_off = 0;
        auto fetch = [&](int tau, StatU16 (&rec)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (WIDE) {
                    rec[i] = srec[rcur[i]];
                    rcur[i] += tau < lim3[i] ? plane_rec : 0;
                } else {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(
                        rsrc, (int)(roff[i] + plane_off), 0, 0);
                    rec[i].s = (int)v[0];
                    rec[i].r = __uint_as_float(v[1]);
                }
            }
            plane_off += (uint32_t)plane_rec * (uint32_t)sizeof(StatU16);
            asm volatile("" : "+s"(plane_off));
        };
        // best key of each output row in this tile and its plane (-1: none).
        // Along a row the shift index grows with tau, so a strict comparison
        // keeps the smallest index among equal keys; rows are merged with the
        // full rule after the tile.
        float rk[4];
        int rt[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rk[i] = -INFINITY;
            rt[i] = -1;
        }
        // ranking of displacement plane tau, then the records of tau + AHEAD
        auto rank = [&](const float4v &c4, int tau, auto slot) __attribute__((always_inline)) {
            constexpr int S = decltype(slot)::value;
            const StatU16(&rec0)[4] = rec[S];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float sts = __builtin_fmaf(fST, (float)rec0[i].s, fshift);
                const float cov = __builtin_fmaf(fN, c4[i], -sts);
                const float key = cov * rec0[i].r;
                const bool take = (tau < lim[i]) & (key > rk[i]);
                rk[i] = take ? key : rk[i];
                rt[i] = take ? tau : rt[i];
                if constexpr (SURF)  // NCC = key / sqrt(N varT)
                    if (tau < lim[i]) p.surface[blk * side2 * side + oidx[i] + tau * side2] =
                        key * inv_vt;
            }
            fetch(tau + AHEAD, rec[(S + AHEAD) % B]);
        };
        static_for<AHEAD>([&](auto k) { fetch(decltype(k)::value, rec[decltype(k)::value]); });
        half8 aop[NQ];
        read_a(aop);
        sweep_block<B, NQ, 0>(0, acc, bop, aop, load_a, rank);
        for (int t0 = B; t0 < g.tz; t0 += B) sweep_block<B, NQ, 1>(t0, acc, bop, aop, load_a, rank);
        sweep_block<B, NQ, 2>(g.tz, acc, bop, aop, load_a, rank);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (rt[i] >= 0) keep_best(bk, bi, rk[i], oidx[i] + rt[i] * side2);
    }
}

// A centre: the block's rounded mean, clamped so every |v - c| <= 2048 over
// the values of range [vmin, vmax] (12-bit values: the interval is never
// empty).
template <int N>
__device__ inline int centre(uint32_t st, int vmin, int vmax) {
    static_assert(N % 2 == 1, "an odd count: the mean is never half way between integers");
    return min(max((int)((2 * st + N) / (2 * N)), vmax - 2048), vmin + 2048);
}

// 16 bytes of raw 12-bit voxels -> fp16 (v - c), exact for |v - c| <= 2048.
__device__ inline u32x4 centre_chunk(u32x4 v, i16x2 c2) {
    i16x2 d[4];
    half2v h[4];
    __builtin_memcpy(d, &v, 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = __builtin_convertvector(d[j] - c2, half2v);
    __builtin_memcpy(&v, h, 16);
    return v;
}

// ------------------------------------------------------------------ kernel
// One 256-thread workgroup per selected block.  Two wavefronts per SIMD up
// to 7^3 blocks; the 9^3 block's B operands (180 registers) take the whole
// register file of one.
constexpr int PB_NW = 4;

template <int B, bool SURF, bool WIDE>
__global__ __launch_bounds__(64 * PB_NW, B == 3 ? 4 : B == 5 ? 3 : B == 7 ? 2 : 1) void k_match_mfma(MfParams p) {
    using G = KGeo<B>;
    constexpr int H = (B - 1) / 2, N = B * B * B, NQ = G::NQ, NT = 64 * PB_NW;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ MfSmall sm;
    _Float16 *tt = reinterpret_cast<_Float16 *>(lds);  // [4][B][TYW][TXW], until the operands are built
    _Float16 *win = reinterpret_cast<_Float16 *>(lds);  // the window, after that
    uint32_t *rowtab = reinterpret_cast<uint32_t *>(lds + p.tab_off);

    const int64_t blk = p.first + xcd_order(blockIdx.x, gridDim.x);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    BGeo g = block_geo<B>(p, blk);
    if (!g.inside) {
        if (tid == 0) put(p, blk, 0, 0, 0, NAN);
        return;
    }

    // ---- loads of the block's voxels (at most 3 per thread for edges up to
    // 9) and of the window's rows, all in flight together; the block tables
    // and operands are built while the window's loads return
    constexpr int TPT = (N + NT - 1) / NT;  // block voxels per thread
    int tv[TPT];
    {
        const uint16_t *rb =
            p.ref + ((int64_t)(g.cz - H) * p.ny + (g.cy - H)) * p.nx + (g.cx - H);
        const int64_t rplane = (int64_t)p.ny * p.nx;
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
            const int o = min(tid + k * NT, N - 1);
            const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
            tv[k] = rb[oz * rplane + (int64_t)oy * p.nx + ox];
        }
    }
    // Thread t copies chunk column xc of every R-th row of the window (rows
    // (z, y) in order, R even: an LDS row pair per two rows), so its addresses
    // advance by additions.  Threads and steps past the last row repeat it.
    // Steps beyond KREG (half windows above 12 or so) are read again when
    // their centre is known.
    constexpr int KREG = B == 3 ? 8 : B == 5 ? 16 : B == 7 ? 20 : 32;
    using Off = typename std::conditional<WIDE, int64_t, uint32_t>::type;
    const bool odd = (p.nx & 1) != 0;
    const int R = (NT / g.cpr) & ~1, rows = g.ez * g.eyp;
    const int kn = (rows + R - 1) / R;
    const int rz = R / g.eyp, ry = R - rz * g.eyp;
    const int xc = tid - quotient(tid, g.cpr) * g.cpr;
    const Off nx_ = (Off)p.nx, nxy_ = (Off)p.nx * (Off)p.ny;
    const Off inc = (Off)rz * nxy_ + (Off)ry * nx_, wrap = nxy_ - (Off)g.eyp * nx_;
    const Off last = (Off)(g.ez - 1) * nxy_ + (Off)(g.ey - 1) * nx_ + (Off)(8 * xc);
    const uint16_t *wb = p.flt + ((int64_t)g.wz0 * p.ny + g.wy0) * p.nx + g.wx0 - g.px;
    // A chunk that would run past the volume's last voxel is read 8 voxels
    // before the end and moved into place when it is used (`edge`, uniform:
    // the window has such chunks).
    const int64_t end = (int64_t)p.nx * p.ny * p.nz - 8 - (wb - p.flt);
    const bool edge =
        ((int64_t)(g.ez - 1) * p.ny + (g.ey - 1)) * p.nx + 8 * (g.cpr - 1) > end;
    const Off tail = edge ? (Off)end : std::numeric_limits<Off>::max();
    struct Walk {
        int r, y;  // row, and its row in its plane
        Off e;     // its chunk's first voxel, from wb
    };
    auto walk_start = [&]() {
        Walk a;
        a.r = quotient(tid, g.cpr);
        if (a.r >= R) a.r = rows;  // idle thread: repeats the last row
        const int z = quotient(a.r, g.eyp);
        a.y = a.r - z * g.eyp;
        a.e = (Off)z * nxy_ + (Off)a.y * nx_ + (Off)(8 * xc);
        return a;
    };
    auto walk_next = [&](Walk &a) {
        a.r += R;
        a.y += ry;
        const bool over = a.y >= g.eyp;
        a.y -= over ? g.eyp : 0;
        a.e += inc + (over ? wrap : (Off)0);
    };
    auto walk_elem = [&](const Walk &a) {
        const Off e = a.e - (a.y >= g.ey ? nx_ : (Off)0);  // the padding row repeats the last
        return a.r < rows ? e : last;
    };
    auto walk_load = [&](const Walk &a) {
        return __builtin_bit_cast(
            u32x4, *reinterpret_cast<const u32x4u *>(wb + min(walk_elem(a), tail)));
    };
    auto walk_fix = [&](u32x4 v, const Walk &a) {  // the chunk of an `edge` window
        const int64_t sh = (int64_t)walk_elem(a) - end;
        return sh > 0 ? shift_chunk(v, (int)min(sh, (int64_t)(odd ? 7 : 6))) : v;
    };
    u32x4 w[KREG];
    Walk at = walk_start();
#pragma unroll
    for (int k2 = 0; k2 < KREG; k2 += 2)
        if (k2 < kn) {
#pragma unroll
            for (int k = k2; k < k2 + 2; ++k) {
                w[k] = walk_load(at);
                walk_next(at);
            }
        }

    // ---- tile rows, zeroed block tables
    block_tiles<B, PB_NW>(p, g);
    // row r of a tile takes base 4 (r mod 4) + r / 4 of its 16: a lane group's
    // i-th output rows are then four x-neighbouring bases, whose records are
    // 128 contiguous bytes per y
    for (int r = tid; r < 16 * g.ntiles; r += NT)
        rowtab[r] = row_entry(g, (r & ~15) | (r & 3) << 2 | (r >> 2 & 3));
    for (int i = tid; i < G::T_BYTES / 16; i += NT)
        *reinterpret_cast<u32x4 *>(lds + 16 * i) = u32x4{0, 0, 0, 0};

    // ---- block sums and value range (per wavefront at most 192 values: the
    // squares sum below 2^32), then c_T
    uint32_t ws = 0, wss = 0;
    u16x2 mm = {4095, 4095};
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const bool real = tid + k * NT < N;
        const uint32_t v = real ? (uint32_t)tv[k] : 0u;
        ws += v;
        wss += v * v;
        const u16x2 m = {(uint16_t)tv[k], (uint16_t)(4095 - tv[k])};
        if (real) mm = __builtin_elementwise_min(mm, m);
    }
    ws = (uint32_t)wave_sum((int)ws);
    wss = (uint32_t)wave_sum((int)wss);
    mm = wave_min(mm);
    if (lane == 63) {
        sm.sum[wave][0] = (int)ws;
        sm.sum[wave][1] = (int)wss;
        sm.mm[wave] = __builtin_bit_cast(uint32_t, mm);
    }
    __syncthreads();  // sums; the zeroed tables
    long long st = 0, stt = 0;
    mm = u16x2{4095, 4095};
#pragma unroll
    for (int i = 0; i < PB_NW; ++i) {
        st += (uint32_t)sm.sum[i][0];
        stt += (uint32_t)sm.sum[i][1];
        mm = __builtin_elementwise_min(mm, __builtin_bit_cast(u16x2, sm.mm[i]));
    }
    if ((long long)N * stt - st * st == 0) {  // flat block: every NCC is 0
        if (tid == 0) put(p, blk, g.lox, g.loy, g.loz, 0.0f);
        return;
    }
    const int c = centre<N>((uint32_t)st, mm[0], 4095 - mm[1]);  // c_T
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int o = tid + k * NT;
        if (o >= N) continue;
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        const _Float16 v = (_Float16)(float)(tv[k] - c);
        _Float16 *d = tt + (oz * G::TYW + oy + OFF) * G::TXW + ox;
#pragma unroll
        for (int a = 0; a < 4; ++a) d[a * G::TCOPY + a] = v;
    }
    __syncthreads();
    half8 bop[B][NQ];
    build_bop<B>(tt, lane, bop);

    // ---- value range of the staged voxels, then c_F.  The range covers the
    // window and, for even row lengths, the few neighbouring voxels its
    // padded rows pick up (odd row lengths: only the window's own columns).
    u16x2 mn2 = {0xffff, 0xffff}, mx2 = {0, 0};
    const Walk rest = at;
    if (edge) {
        Walk s = walk_start();
#pragma unroll
        for (int k = 0; k < KREG; ++k, walk_next(s))
            if (k < kn) w[k] = walk_fix(w[k], s);
    }
    auto reload = [&]() {
        u32x4 v = walk_load(at);
        if (edge) v = walk_fix(v, at);
        return v;
    };
    auto ranges = [&](auto &&use) {
#pragma unroll
        for (int k = 0; k < KREG; ++k)
            if (k < kn) use(w[k]);
        for (int k = KREG; k < kn; ++k, walk_next(at)) use(reload());
    };
    if (odd) {
        const int nv = g.ex - 8 * xc;  // this thread's columns inside the window
        uint32_t keep[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            keep[j] = (2 * j < nv ? 0xffffu : 0u) | (2 * j + 1 < nv ? 0xffff0000u : 0u);
        ranges([&](const u32x4 &v) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mn2 = __builtin_elementwise_min(mn2, __builtin_bit_cast(u16x2, v[j] | ~keep[j]));
                mx2 = __builtin_elementwise_max(mx2, __builtin_bit_cast(u16x2, v[j] & keep[j]));
            }
        });
    } else {
        ranges([&](const u32x4 &v) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t x = v[j];  // a bit cast of the element itself reads element 0
                mn2 = __builtin_elementwise_min(mn2, __builtin_bit_cast(u16x2, x));
                mx2 = __builtin_elementwise_max(mx2, __builtin_bit_cast(u16x2, x));
            }
        });
    }
    const int vmn = min((int)mn2[0], (int)mn2[1]), vmx = max((int)mx2[0], (int)mx2[1]);
    mm = wave_min(u16x2{(uint16_t)min(vmn, 4095), (uint16_t)(4095 - vmx)});
    if (lane == 63) sm.wm[wave] = __builtin_bit_cast(uint32_t, mm);
    __syncthreads();  // every wavefront's operands are built: the window takes the tables' place
    mm = u16x2{4095, 4095};
#pragma unroll
    for (int i = 0; i < PB_NW; ++i)
        mm = __builtin_elementwise_min(mm, __builtin_bit_cast(u16x2, sm.wm[i]));
    const int cf = centre<N>((uint32_t)st, mm[0], 4095 - mm[1]);  // c_F

    // ---- the window as fp16 (v - c_F); a pair of rows past the last plane,
    // which the lowest bases read against zeros, is cleared
    {
        const i16x2 c2 = {(short)cf, (short)cf};
        auto store = [&](const u32x4 &v, int r, int d) {
            const u32x4 h = centre_chunk(v, c2);
            _Float16 *q = win + (r < rows ? d : (rows / 2 - 1) * g.rp2 + 4 + 16 * xc);
            *reinterpret_cast<u32x2 *>(q) = u32x2{h[0], h[1]};
            *reinterpret_cast<u32x2 *>(q + 8) = u32x2{h[2], h[3]};
        };
        const int step = (R >> 1) * g.rp2;
        int r = quotient(tid, g.cpr);
        int d = (r >> 1) * g.rp2 + (r & 1) * 4 + 16 * xc;
        if (r >= R) r = rows;
#pragma unroll
        for (int k = 0; k < KREG; ++k, r += R, d += step)
            if (k < kn) store(w[k], r, d);
        at = rest;
        for (int k = KREG; k < kn; ++k, walk_next(at), d += step) store(reload(), at.r, d);
        for (int i = tid; i < g.rp2 / 8; i += NT)
            *reinterpret_cast<u32x4 *>(win + g.ez * g.pl + 8 * i) = u32x4{0, 0, 0, 0};
    }
    __syncthreads();

    float bk = -INFINITY;
    int bi = INT_MAX;
    const long long sTc = st - (long long)N * c;                      // sum (T - c)
    const long long tc2 = stt - 2ll * c * st + (long long)N * c * c;  // sum (T - c)^2
    const long long vt = (long long)N * tc2 - sTc * sTc;
    float inv_vt = 0.0f;
    if constexpr (SURF) inv_vt = (float)(1.0 / sqrt((double)vt));
    sweep_tiles<B, PB_NW, SURF, WIDE>(p, g, blk, win, rowtab, bop, sTc, inv_vt, cf, wave, lane, bk,
                                      bi);

    // ---- workgroup argmax, then the exact NCC at the winner from the staged
    // integers (F - c_F in the window, T - c_T from the registers; the NCC
    // does not depend on either constant), written by thread 0
    wave_best(bk, bi);
    if (lane == 63) {
        sm.key[wave] = bk;
        sm.idx[wave] = bi;
    }
    __syncthreads();
    bk = sm.key[0];
    bi = sm.idx[0];
#pragma unroll
    for (int i = 1; i < PB_NW; ++i) keep_best(bk, bi, sm.key[i], sm.idx[i]);
    if (bi == INT_MAX) {  // no finite key (cannot happen for 12-bit data)
        if (tid == 0) put(p, blk, 0, 0, 0, NAN);
        return;
    }
    const int side = 2 * p.w + 1;
    const int ddx = bi % side - p.w, ddy = (bi / side) % side - p.w, ddz = bi / (side * side) - p.w;
    const int rx = ddx - g.lox + g.px, ryo = ddy - g.loy, rzo = ddz - g.loz;
    // 32-bit sums per wavefront: at most 192 values of magnitude up to 2^22
    int sf = 0, sff = 0, stf = 0;
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int o = tid + k * NT;
        if (o >= N) continue;
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        const int y = ryo + oy, x = rx + ox;
        const int f = (int)(float)win[(rzo + oz) * g.pl + (y >> 1) * g.rp2 + (x >> 2) * 8 +
                                      (y & 1) * 4 + (x & 3)];
        sf += f;
        sff += f * f;
        stf += (tv[k] - c) * f;
    }
    sf = wave_sum(sf);
    sff = wave_sum(sff);
    stf = wave_sum(stf);
    if (lane == 63) {
        sm.sum[wave][0] = sf;
        sm.sum[wave][1] = sff;
        sm.sum[wave][2] = stf;
    }
    __syncthreads();
    if (tid == 0) {
        long long tf = 0, tff = 0, ttf = 0;
#pragma unroll
        for (int i = 0; i < PB_NW; ++i) {
            tf += sm.sum[i][0];
            tff += sm.sum[i][1];
            ttf += sm.sum[i][2];
        }
        const long long vf = (long long)N * tff - tf * tf;
        const long long cv = (long long)N * ttf - sTc * tf;
        const double v = (vt > 0 && vf > 0) ? (double)cv / sqrt((double)vt * (double)vf) : 0.0;
        put(p, blk, ddx, ddy, ddz, (float)v);
    }
}

// ------------------------------------------------------------------- host
typedef void (*mf_kernel_t)(MfParams);

struct MfVariant {
    int b;
    mf_kernel_t fn, wide, surf;
    int nq, t_bytes;
};

#define MFV(B)                                                                                  \
    {B, k_match_mfma<B, false, false>, k_match_mfma<B, false, true>, k_match_mfma<B, true, true>, \
     KGeo<B>::NQ, KGeo<B>::T_BYTES}
const MfVariant kMfVariants[] = {MFV(3), MFV(5), MFV(7), MFV(9)};
#undef MFV

const MfVariant *mf_variant(int b) {
    for (const MfVariant &v : kMfVariants)
        if (v.b == b) return &v;
    return nullptr;
}

// LDS sizes for the unclipped window of (b, w): the window (or, before it,
// the block tables) and the tile-row table; clipped windows need no more.
struct MfPlan {
    int rp2;      // pitch of a pair of rows (halves)
    int tab_off;  // byte offset of the tile-row table
    size_t lds;
};

bool mf_plan(int b, int w, size_t limit, MfPlan *out) {
    const MfVariant *v = mf_variant(b);
    if (!v) return false;
    const int d = 2 * w + 1;
    const int nbx = (d + 1 + 3) / 4, nby = (d + 3) / 4;  // x: one column of parity shift
    const int gx = (b + 6) / 4;
    const int cols = (4 * (nbx - 1) + 4 * gx + 7) / 8 * 8;  // whole 8-column chunks
    int rp2 = 2 * cols;
    const int planes = d + b - 1;  // also the window's rows per plane, odd
    if (planes >= 255) return false;  // tile rows keep base and phase numbers in bytes
    const size_t win = (size_t)(planes * (planes + 1) / 2 + 1) * rp2 * 2;
    const size_t tab = win > (size_t)v->t_bytes ? win : (size_t)v->t_bytes;
    const size_t nrows = (size_t)nbx * nby * ((d + b - 1) / b);
    const size_t lds = tab + (nrows + 15) / 16 * 16 * 4;
    if (lds + sizeof(MfSmall) > limit) return false;
    out->rp2 = rp2;
    out->tab_off = (int)tab;
    out->lds = lds;
    return true;
}

}  // namespace

bool mfma_supported(nrr_dtype dtype, int32_t block, int32_t window) {
    if (dtype != NRR_U16) return false;
    MfPlan pl;
    return mf_plan(block, window, device_lds_limit(), &pl);
}

bool mfma_fits(const MatchArgs &a) {
    // record indices are 32-bit
    return (int64_t)a.ox * a.oy * (a.nz - a.block + 1) < (1ll << 31);
}

hipError_t launch_match_mfma(const MatchArgs &a, hipStream_t stream, float *surface) {
    MfPlan pl;
    if (!mf_plan(a.block, a.window, device_lds_limit(), &pl) || !mfma_fits(a))
        return hipErrorInvalidValue;
    const MfVariant *v = mf_variant(a.block);
    MfParams p;
    p.ref = static_cast<const uint16_t *>(a.ref);
    p.flt = static_cast<const uint16_t *>(a.flt);
    p.nx = a.nx;
    p.ny = a.ny;
    p.nz = a.nz;
    p.centers = a.centers;
    p.first = 0;
    p.w = a.window;
    p.stats = static_cast<const StatU16 *>(a.stats);
    p.nstat = (int64_t)a.ox * a.oy * (a.nz - a.block + 1);
    p.ox = a.ox;
    p.oy = a.oy;
    p.rp2 = pl.rp2;
    p.tab_off = pl.tab_off;
    const int d = 2 * a.window + 1;
    for (int px = 0; px < 2; ++px)
        p.tz[px] = best_phase((d + px + 3) / 4 * ((d + 3) / 4), d, a.block, v->nq, PB_NW);
    p.disp = a.disp;
    p.ncc = a.ncc;
    p.conf = a.conf;
    p.surface = surface;
    // 32-bit record offsets reach the window's planes (and the masked ones
    // past it) unless the volume's planes are very large
    const bool wide = (int64_t)a.nx * a.ny * 8 * (2 * d + 3 * a.block) >= (1ll << 31);
    const mf_kernel_t fn = surface ? v->surf : wide ? v->wide : v->fn;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);
    if (e != hipSuccess) return e;
    const int64_t chunk = 1ll << 30;
    for (int64_t first = 0; first < a.n; first += chunk) {
        p.first = first;
        const int64_t cnt = a.n - first < chunk ? a.n - first : chunk;
        hipLaunchKernelGGL(fn, dim3((unsigned)cnt), dim3(64 * PB_NW), pl.lds, stream, p);
    }
    return hipGetLastError();
}

}  // namespace nrr
