// Matrix-core filter in front of the FP32 searches.
//
// The FP32 searches (float volumes, and blocks with per-axis sizes) rank every
// displacement by FMA chains on the vector units.  The filter finds the same
// winner, bit for bit, from matrix instructions: it computes every cross term
// in fp16 products with FP32 accumulation (the formulation of the 12-bit
// matrix-core search: a 4x4 patch of (dx, dy) offsets per instruction, the
// block as a Toeplitz operand in registers), bounds for every displacement
// how far the FP32 search's key can lie from it, and re-ranks only the
// displacements that can win, in the FP32 search's own order of operations.
//
// The bound.  With T^ the search's centred block, F' = fl(F - c) its staged
// window, Fmax the largest |F'| of the staged window and key = N X r (X = sum
// T^ F', r = 1 / sqrt(N varF) >= 0; the search's other term, sum T^ times the
// window's mean, is at most 2^-24 of the bound's scale), the distance of N X r
// from its fp16 value is at most EPS N |T^| |F'| r (Cauchy-Schwarz), and |F'|
// <= sqrt(N) Fmax.  EPS collects
//   the fp16 operands, T^ and F' scaled by powers of two so that their largest
//   magnitudes lie in [2^14, 2^15), rounded to nearest: 2^-10 + 2^-22;
//   the accumulation of at most 1440 products in FP32, whatever its order and
//   rounding: 1440 2^-23;
//   the FP32 search's own chain, at most 729 + 9 roundings: 738 2^-24;
//   operands below fp16's normal range (2^-14 absolute, whether or not they
//   are flushed), 2^-28 of Fmax;
// which sum to 1.20e-3; 1.3e-3 is used.  So key sT sF / N lies in (C -+ ea) r
// with C the accumulated sum and ea = EPS sqrt(N) |T^| sT Fmax sF.  A
// displacement whose upper end lies below the largest lower end cannot win.
// (|F'| of each displacement bounds it more tightly, from the record's sum; in
// the sweep it would cost 16-byte records and a third of the registers, so only
// listed displacements get it.)
//
// Broad peaks.  EPS separates displacements by about 0.003 in NCC: on tissue with
// noise most blocks keep one, on smooth volumes hundreds lie that close.  Those
// cost the FP32 chain of each, one displacement per thread, where the FP32 search
// reads eight from the same registers; so the cubic search sweeps the tiles that
// still matter a second time against the bound found (fewer whole rows), the
// voxels around the peak are staged once for all candidates, and the per-axis
// search leaves the block early.  64^3 blobs with noise of 0.02, 32 sets in one
// batch: 0.94 ms with all candidates' windows staged one by one, 0.67 now (1.20
// in the FP32 form).
// Blocks whose values do not scale (not finite, or magnitudes outside 2^-60 ..
// 2^58: above, the FP32 search's sums may overflow), flat ones, and those that
// keep more candidates than is worth ranking are left to the FP32 search itself.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "nrr_internal.h"
#include "record_planes.h"
#include "wave64.h"

namespace nrr {
namespace filt {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));

constexpr int NT = 256, NW = 4;  // threads and wavefronts of a workgroup
constexpr int OFF = 3;           // zero rows above a plane of the T tables
constexpr float EPS = 1.3e-3f;
constexpr int LIST = 896;   // list of displacements and rows that may win: at least,
constexpr int LIST_MAX = 4096;  // and at most, where a CU's LDS has room beside its workgroups
constexpr int SPREAD = 512;  // candidates re-ranked one by one, wherever they lie
constexpr int TILES = 64;   // 16-row tiles of a window at most
constexpr int MAXN = 729;   // block voxels served (the bound's terms above)

// Floats as integers of the same order (never 0 for a finite float).  The zeros
// are one value, as in a comparison of floats: bounds of a record with r = 0 are
// zeros of either sign, and their keys tie.
__device__ inline uint32_t ordered(float f) {
    const uint32_t b = __float_as_uint(f + 0.0f);
    return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ inline float unordered(uint32_t u) {
    return __uint_as_float(u & 0x80000000u ? u & 0x7fffffffu : ~u);
}

// Power of two that brings magnitude `bits` (of a positive float) into
// [2^14, 2^15); false where the magnitude is outside 2^-60 .. 2^58, zero or
// not finite.  (729 products of two magnitudes below 2^58 sum below 2^126.)
__device__ inline bool scale_of(uint32_t bits, float &scale) {
    const int e = (int)(bits >> 23);
    if (e < 127 - 60 || e > 127 + 57) return false;
    scale = __uint_as_float((uint32_t)(127 + 14 - (e - 127)) << 23);
    return true;
}

// Host and device sizes of one (block, window): the K layout (groups of 4
// columns by 2 rows that any offset of the patch touches) and LDS offsets.
using Sizes = FiltSizes;

__host__ __device__ inline int best_phase(int nxy, int dzn, int bz, int nq) {
    int best = bz;
    float bc = 3.0e38f;
    for (int tz = bz; tz < dzn + bz; tz += bz) {
        const int ph = (dzn + tz - 1) / tz;
        const int tiles = (nxy * ph + 15) / 16;
        const int rounds = (tiles + NW - 1) / NW;
        const float c = rounds * ((float)tz * bz * nq + 6.0f * (tz + bz - 1));
        if (c < bc) {
            bc = c;
            best = tz;
        }
    }
    return best;
}

// False where the filter does not serve the sizes (block edges 3-9 along z
// and up to 9 along x and y, the window in `limit` bytes of LDS).
inline bool plan(const int32_t b[3], const int32_t w[3], size_t limit, Sizes *s) {
    for (int a = 0; a < 3; ++a)
        if (b[a] > 9) return false;
    if (b[2] < 3 || b[0] * b[1] * b[2] > MAXN || b[0] * b[1] * b[2] < 27) return false;
    s->gx = (b[0] + 6) / 4;
    s->gyp = (b[1] + 4) / 2;
    s->nq = (s->gx * s->gyp + 3) / 4;
    s->txw = 4 * s->gx;
    s->tyw = 2 * s->gyp + OFF;
    s->tcopy = b[2] * s->tyw * s->txw;
    const int dx = 2 * w[0] + 1, dy = 2 * w[1] + 1, dz = 2 * w[2] + 1;
    const int nbx = (dx + 3) / 4, nby = (dy + 3) / 4;
    const int cols = (4 * (nbx - 1) + 4 * s->gx + 7) / 8 * 8;
    const int eyp = (dy + b[1] - 1 + 1) & ~1, ez = dz + b[2] - 1;
    if (ez >= 255 || nbx >= 255 || nby >= 255) return false;
    s->rp2 = 2 * cols;
    const size_t win = (size_t)(ez * eyp / 2 + 3) * s->rp2 * 2;
    const size_t tables = (size_t)4 * s->tcopy * 2;
    const size_t t_off = ((win > tables ? win : tables) + 15) & ~(size_t)15;
    const size_t tab_off = (t_off + (size_t)b[0] * b[1] * b[2] * 4 + 15) & ~(size_t)15;
    const size_t nrows = (size_t)nbx * nby * ((dz + b[2] - 1) / b[2]);
    if (nrows > 16 * TILES) return false;
    const size_t l_off = tab_off + (nrows + 15) / 16 * 16 * 4;
    if (l_off + LIST * 8 > limit) return false;
    // the list takes what is left of the CU's LDS by the workgroups that share it
    // (at most three: registers)
    const size_t shared = limit / (l_off + LIST * 8), groups = shared < 3 ? shared : 3;
    size_t room = (limit / groups - (groups > 1 ? 2048 : 0)) / 8 * 8;
    room = room < l_off + LIST * 8 ? l_off + LIST * 8 : room;
    const size_t list = (room - l_off) / 8 < LIST_MAX ? (room - l_off) / 8 : LIST_MAX;
    const size_t lds = l_off + list * 8;
    s->list = (int)list;
    s->t_off = (int)t_off;
    s->tab_off = (int)tab_off;
    s->l_off = (int)l_off;
    s->lds = (int)lds;
    s->tz = best_phase(nbx * nby, dz, b[2], s->nq);
    return true;
}

struct Small {
    uint32_t wmax[NW];  // largest |F'| bits per wavefront
    uint32_t tmin[NW], tmax[NW];  // smallest and largest block voxel (ordered) per wavefront
    uint32_t low;       // largest lower bound (ordered)
    uint32_t top[TILES];  // largest upper bound of each tile
    int nlist, ncand, rows;
    uint32_t box[6];    // of the candidates: largest x, y, z, and complements of the smallest
    double key[NW];
    int idx[NW];
};

// The block's scale from its extremes and mean; false where it does not scale.
// Uniform.
__device__ inline bool block_scale(const Small &sm, double mean, float &sT) {
    const uint32_t mn = min(min(sm.tmin[0], sm.tmin[1]), min(sm.tmin[2], sm.tmin[3]));
    const uint32_t mx = max(max(sm.tmax[0], sm.tmax[1]), max(sm.tmax[2], sm.tmax[3]));
    const float lo = (float)((double)unordered(mn) - mean), hi = (float)((double)unordered(mx) - mean);
    const uint32_t top =
        max(__float_as_uint(lo) & 0x7fffffffu, __float_as_uint(hi) & 0x7fffffffu);
    return scale_of((uint32_t)__builtin_amdgcn_readfirstlane((int)top), sT);
}

// One block's search: geometry (uniform), then the steps below in order.
struct Args {
    Sizes z;
    int b[3], w[3];
    int nx, ny, nz, ox, oy;
    const void *flt, *stats;
    int64_t nstat;  // records of the table
};

struct Geo {
    int lox, loy, loz, dxn, dyn, dzn;
    int ox0, oy0, oz0;  // the window's corner (= the origin of the first displacement)
    int ex, ey, ez, eyp, nbx, nby, cpr, pl;
    int tz, nrows, ntiles;
};

template <typename Vox>
struct Chunk;  // one 16-byte load of a window row
template <>
struct Chunk<float> {
    static constexpr int C = 4;
};
template <>
struct Chunk<uint16_t> {
    static constexpr int C = 8;
};

template <typename Vox>
__device__ inline Geo geometry(const Args &p, int cx, int cy, int cz) {
    Geo g;
    const int hx = (p.b[0] - 1) / 2, hy = (p.b[1] - 1) / 2, hz = (p.b[2] - 1) / 2;
    g.lox = max(-p.w[0], hx - cx);
    g.loy = max(-p.w[1], hy - cy);
    g.loz = max(-p.w[2], hz - cz);
    g.dxn = min(p.w[0], p.nx - 1 - hx - cx) - g.lox + 1;
    g.dyn = min(p.w[1], p.ny - 1 - hy - cy) - g.loy + 1;
    g.dzn = min(p.w[2], p.nz - 1 - hz - cz) - g.loz + 1;
    g.ox0 = cx - hx + g.lox;
    g.oy0 = cy - hy + g.loy;
    g.oz0 = cz - hz + g.loz;
    g.ex = g.dxn + p.b[0] - 1;
    g.ey = g.dyn + p.b[1] - 1;
    g.ez = g.dzn + p.b[2] - 1;
    g.eyp = (g.ey + 1) & ~1;
    g.nbx = (g.dxn + 3) / 4;
    g.nby = (g.dyn + 3) / 4;
    g.cpr = (4 * (g.nbx - 1) + 4 * p.z.gx + Chunk<Vox>::C - 1) / Chunk<Vox>::C;
    g.pl = (g.eyp / 2) * p.z.rp2;
    return g;
}

// Tile rows (base x, base y, phase, real) in LDS; row r of a tile takes base
// 4 (r mod 4) + r / 4 of its 16, so that a lane group's i-th output rows are
// four x-neighbouring bases.  Also clears the T tables and the counters.
__device__ __attribute__((always_inline)) inline void open_block(const Args &p, Geo &g,
                                                                 unsigned char *lds, Small &sm) {
    const int tid = threadIdx.x, nxy = g.nbx * g.nby;
    g.tz = g.dxn == 2 * p.w[0] + 1 && g.dyn == 2 * p.w[1] + 1 && g.dzn == 2 * p.w[2] + 1
               ? p.z.tz
               : best_phase(nxy, g.dzn, p.b[2], p.z.nq);
    g.nrows = nxy * ((g.dzn + g.tz - 1) / g.tz);
    g.ntiles = (g.nrows + 15) / 16;
    uint32_t *rowtab = reinterpret_cast<uint32_t *>(lds + p.z.tab_off);
    for (int i = tid; i < 16 * g.ntiles; i += NT) {
        const int r = (i & ~15) | (i & 3) << 2 | (i >> 2 & 3);
        const bool real = r < g.nrows;
        const int rr = real ? r : 0;
        const int ph = quotient(rr, nxy), xy = rr - ph * nxy;
        const int yi = quotient(xy, g.nbx), xi = xy - yi * g.nbx;
        rowtab[i] = (uint32_t)xi | (uint32_t)yi << 8 | (uint32_t)ph << 16 | (real ? 1u << 24 : 0u);
    }
    for (int i = tid; i < (4 * p.z.tcopy + 7) / 8; i += NT)
        *reinterpret_cast<u32x4 *>(lds + 16 * i) = u32x4{0, 0, 0, 0};
    if (tid == 0) {
        sm.low = 0;
        sm.nlist = sm.ncand = sm.rows = 0;
        for (int i = 0; i < 6; ++i) sm.box[i] = 0;
    }
}

// The window's 16-byte chunks: thread t copies chunk column xc of every R-th
// row (rows (z, y) in order; a padding row past the window repeats its last
// row, as do threads and steps past the last row).
template <typename Vox>
struct Walk {
    static constexpr int C = Chunk<Vox>::C;
    int R, rows, kn, ry, xc;
    uint32_t inc, wrap, last;
    const Vox *wb;
    bool edge;    // some chunk would run past the volume's last voxel
    int64_t end;  // the last voxel, from wb
    int r, y;
    uint32_t e;

    __device__ inline void start(const Args &p, const Geo &g) {
        const int tid = threadIdx.x;
        R = (NT / g.cpr) & ~1;
        rows = g.ez * g.eyp;
        kn = (rows + R - 1) / R;
        const int rz = R / g.eyp;
        ry = R - rz * g.eyp;
        const uint32_t nx = (uint32_t)p.nx, nxy = nx * (uint32_t)p.ny;
        inc = (uint32_t)rz * nxy + (uint32_t)ry * nx;
        wrap = nxy - (uint32_t)g.eyp * nx;
        wb = static_cast<const Vox *>(p.flt) +
             (((int64_t)g.oz0 * p.ny + g.oy0) * p.nx + g.ox0);
        end = (int64_t)p.nx * p.ny * p.nz - 1 - (wb - static_cast<const Vox *>(p.flt));
        edge = ((int64_t)(g.ez - 1) * p.ny + (g.ey - 1)) * p.nx + C * g.cpr - 1 > end;
        r = quotient(tid, g.cpr);
        xc = tid - r * g.cpr;
        last = (uint32_t)(g.ez - 1) * nxy + (uint32_t)(g.ey - 1) * nx + (uint32_t)(C * xc);
        if (r >= R) r = rows;
        const int z = quotient(r, g.eyp);
        y = r - z * g.eyp;
        e = (uint32_t)z * nxy + (uint32_t)y * nx + (uint32_t)(C * xc);
    }
    __device__ inline void next(const Geo &g) {
        r += R;
        y += ry;
        const bool over = y >= g.eyp;
        y -= over ? g.eyp : 0;
        e += inc + (over ? wrap : 0u);
    }
    __device__ inline u32x4 load(const Args &p, const Geo &g) const {
        const uint32_t at = r < rows ? e - (y >= g.ey ? (uint32_t)p.nx : 0u) : last;
        if (edge) {  // voxel by voxel, clamped to the volume's last
            u32x4 v = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const int64_t i = min((int64_t)at + j, end);
                if constexpr (C == 4)
                    v[j] = __float_as_uint(((const float *)wb)[i]);
                else
                    v[j / 2] |= (uint32_t)((const uint16_t *)wb)[i] << (16 * (j & 1));
            }
            return v;
        }
        if constexpr (C == 4)
            return __builtin_bit_cast(u32x4, *reinterpret_cast<const float4u *>(wb + at));
        else
            return __builtin_bit_cast(u32x4, *reinterpret_cast<const u32x4u *>(wb + at));
    }
};

// The C voxels of a chunk as floats less c.
template <typename Vox>
__device__ inline void centred(const u32x4 &v, float c, float (&f)[Chunk<Vox>::C]) {
#pragma unroll
    for (int j = 0; j < Chunk<Vox>::C; ++j) {
        if constexpr (sizeof(Vox) == 4) {
            const uint32_t x = v[j];
            f[j] = __uint_as_float(x) - c;
        } else {
            const uint32_t x = v[j / 2];
            f[j] = (float)(j & 1 ? x >> 16 : x & 0xffffu) - c;
        }
    }
}

// T^ of block voxel (ox, oy, oz): the float, and its four fp16 copies scaled by
// sT (copy a moved right by a columns).
__device__ inline void put_voxel(const Args &p, unsigned char *lds, int ox, int oy, int oz,
                                 float v, float sT) {
    reinterpret_cast<float *>(lds + p.z.t_off)[(oz * p.b[1] + oy) * p.b[0] + ox] = v;
    _Float16 *d = reinterpret_cast<_Float16 *>(lds) + (oz * p.z.tyw + oy + OFF) * p.z.txw + ox;
    const _Float16 h = (_Float16)(v * sT);
#pragma unroll
    for (int a = 0; a < 4; ++a) d[a * p.z.tcopy + a] = h;
}

template <int BZ, int NQ>
__device__ __attribute__((always_inline)) inline void build_operands(
    const Args &p, const unsigned char *lds, int lane, half8 (&bop)[BZ][NQ]) {
    const _Float16 *tt = reinterpret_cast<const _Float16 *>(lds);
    const int grp = lane >> 4, oa = lane & 3, ob = (lane >> 2) & 3;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int g = 4 * q + grp;
        const int gy = quotient(g, p.z.gx), gx = g - gy * p.z.gx;
        // groups past the last read two of the zero rows
        const _Float16 *tr = tt + oa * p.z.tcopy +
                             (gy < p.z.gyp ? (2 * gy - ob + OFF) * p.z.txw + 4 * gx : 0);
#pragma unroll
        for (int s = 0; s < BZ; ++s) {
            const half4 lo = *reinterpret_cast<const half4 *>(tr + s * p.z.tyw * p.z.txw);
            const half4 hi = *reinterpret_cast<const half4 *>(tr + (s * p.z.tyw + 1) * p.z.txw);
            bop[s][q] = half8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    }
}

// One unrolled block of BZ sweep steps (see the 12-bit matrix-core search):
// MODE 0 the first, 1 a full one, 2 the last.
template <int BZ, int NQ, int MODE, typename LoadA, typename Rank>
__device__ __attribute__((always_inline)) inline void sweep_block(
    int t0, float4v (&acc)[BZ], const half8 (&bop)[BZ][NQ], half8 (&aop)[NQ], LoadA load_a,
    Rank rank) {
    constexpr int STEPS = MODE == 2 ? BZ - 1 : BZ;
    static_for<STEPS>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        const int t = t0 + u;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int k = 0; k < BZ; ++k) {
                const int s = BZ - 1 - k;
                if (MODE == 0 && s > u) continue;
                if (MODE == 2 && s <= u) continue;
                const int slot = (u - s + BZ) % BZ;
                acc[slot] =
                    __builtin_amdgcn_mfma_f32_16x16x32_f16(aop[q], bop[s][q], acc[slot], 0, 0, 0);
            }
        load_a(t + 1, aop);
        constexpr int fs = (u + 1) % BZ;
        if (MODE != 0 || u == BZ - 1)
            rank(acc[fs], t - (BZ - 1), std::integral_constant<int, fs>());
        acc[fs] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
        // a step's work stays in it: hoisting the next steps' loads and
        // conversions into it costs more registers than there are
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The candidates' shift indices (candidate k at [-k], down from the list's end),
// and room for SPREAD keys (at its start).
__device__ inline int *candidates(const Args &p, unsigned char *lds) {
    return reinterpret_cast<int *>(lds + p.z.l_off + 8 * p.z.list) - 1;
}
template <typename Key>
__device__ inline Key *candidate_keys(const Args &p, unsigned char *lds) {
    return reinterpret_cast<Key *>(lds + p.z.l_off);
}

template <typename Vox>
struct Record;
template <>
struct Record<float> {
    using Type = StatF32;
};
template <>
struct Record<uint16_t> {
    using Type = StatU16;
};

// One tile's sweep: take(i, tau, hi, lo) with the upper and lower end of the
// key of output row i of the lane in plane tau of the row's phase (valid where tau
// < lim[i]; lim and ents: the valid planes and table entries of the four rows).
template <typename Rec, int BZ, int NQ, int AHEAD, typename Take>
__device__ __attribute__((always_inline)) inline void sweep_tile(
    const Args &p, const Geo &g, const _Float16 *win, const uint32_t *rowtab,
    const half8 (&bop)[BZ][NQ], const int (&kq)[NQ], int64_t corner, float ea, int tile, int lane,
    int (&lim)[4], uint32_t (&ents)[4], Take take) {
    const int n16 = lane & 15, grp = lane >> 4;
    const int oa = n16 & 3, ob = n16 >> 2;
    const int plane_rec = p.oy * p.ox;
    int abase, alim;
    {
        const uint32_t e = rowtab[16 * tile + n16];
        const int aph = (int)(e >> 16 & 0xff) * g.tz;
        abase = min(aph, g.ez - 1) * g.pl + (int)(e >> 8 & 0xff) * 2 * p.z.rp2 +
                (int)(e & 0xff) * 8;
        alim = g.ez - 1 - aph;
    }
    uint32_t roff[4];
    const uint4 ent = *reinterpret_cast<const uint4 *>(rowtab + 16 * tile + 4 * grp);
    ents[0] = ent.x, ents[1] = ent.y, ents[2] = ent.z, ents[3] = ent.w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t e = ents[i];
        const int odx = 4 * (int)(e & 0xff) + oa, ody = 4 * (int)(e >> 8 & 0xff) + ob;
        const int oph = (int)(e >> 16 & 0xff) * g.tz;
        roff[i] = (uint32_t)(min(ody, g.dyn - 1) * p.ox + min(odx, g.dxn - 1) +
                             min(oph, g.dzn - 1) * plane_rec) *
                      (uint32_t)sizeof(Rec) +
                  (uint32_t)(sizeof(Rec) - 4);  // r, or its high word
        lim[i] = (e >> 24) && odx < g.dxn && ody < g.dyn ? g.dzn - oph : -1;
    }
    float4v acc[BZ];
#pragma unroll
    for (int k = 0; k < BZ; ++k) acc[k] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    auto read_a = [&](half8 (&aop)[NQ]) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            aop[q] = *reinterpret_cast<const half8 *>(win + abase + kq[q]);
    };
    auto load_a = [&](int t, half8 (&aop)[NQ]) {
        abase += t <= alim ? g.pl : 0;
        read_a(aop);
    };
    // r of each output row's record, AHEAD planes early: of a double the high
    // word (2^-20 of its value below it)
    uint32_t rec[BZ][4];
    RecordPlanes at_rec;  // of the plane fetched next (planes in order)
    at_rec.start(p.stats, p.nstat, corner, sizeof(Rec));
    auto fetch = [&](uint32_t (&rc)[4]) __attribute__((always_inline)) {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char *>(at_rec.base), 0, (int)at_rec.bytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            rc[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)roff[i], 0, 0);
        at_rec.next((uint32_t)plane_rec * (uint32_t)sizeof(Rec));
    };
    auto rank = [&](const float4v &c4, int tau, auto slot) __attribute__((always_inline)) {
        constexpr int S = decltype(slot)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // (the clamp keeps the ends finite: beyond 2^86 the distance between
            // them exceeds any key)
            float r = sizeof(Rec) == 16 ? (float)__hiloint2double((int)rec[S][i], 0)
                                        : __uint_as_float(rec[S][i]);
            r = r > 0x1p86f ? 0x1p86f : r;
            const float hi = (c4[i] + ea) * r, lo = (c4[i] - ea) * r;
            take(i, tau, hi, lo);
        }
        fetch(rec[(S + AHEAD) % BZ]);
    };
    static_for<AHEAD>([&](auto k) { fetch(rec[decltype(k)::value]); });
    half8 aop[NQ];
    read_a(aop);
    sweep_block<BZ, NQ, 0>(0, acc, bop, aop, load_a, rank);
    for (int t0 = BZ; t0 < g.tz; t0 += BZ)
        sweep_block<BZ, NQ, 1>(t0, acc, bop, aop, load_a, rank);
    sweep_block<BZ, NQ, 2>(g.tz, acc, bop, aop, load_a, rank);
}

// Everything after the caller's T^ (put_voxel, after open_block's clears, and
// published by a barrier): w[] holds the first KREG chunks
// of `walk0`'s walk, and `at` the walk behind them.  Returns the number of
// displacements that can win (shift indices in candidates(), with repeats), or
// 0 where the block is left to the FP32 search.  `few`: with AGAIN the candidates
// above which broad peaks are swept a second time; without, the list's entries
// above which the block is left.  Uniform; the window in LDS is
// free for reuse, and the list published, on return.
template <typename Vox, int BZ, int NQ, int KREG, int AHEAD, bool AGAIN>
__device__ __attribute__((always_inline)) inline int search(
    const Args &p, const Geo &g, unsigned char *lds, Small &sm, u32x4 (&w)[KREG],
    const Walk<Vox> &walk0, Walk<Vox> at, float c, float tnorm, float sT, int few) {
    using Rec = typename Record<Vox>::Type;
    constexpr int C = Chunk<Vox>::C;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = p.b[0] * p.b[1] * p.b[2];
    float sF;
    half8 bop[BZ][NQ];
    build_operands<BZ, NQ>(p, lds, lane, bop);

    // ---- largest |F'| of the staged voxels, then its scale
    uint32_t fmax = 0;
    auto range = [&](const u32x4 &v) {
        float f[C];
        centred<Vox>(v, c, f);
#pragma unroll
        for (int j = 0; j < C; ++j) fmax = max(fmax, __float_as_uint(f[j]) & 0x7fffffffu);
    };
#pragma unroll
    for (int k = 0; k < KREG; ++k)
        if (k < walk0.kn) range(w[k]);
    {
        Walk<Vox> a = at;
        for (int k = KREG; k < walk0.kn; ++k, a.next(g)) range(a.load(p, g));
    }
    fmax = wave_max(fmax);
    if (lane == 63) sm.wmax[wave] = fmax;
    __syncthreads();  // every wavefront's operands are built: the window takes their place
    fmax = max(max(sm.wmax[0], sm.wmax[1]), max(sm.wmax[2], sm.wmax[3]));
    fmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)fmax);
    if (!scale_of(fmax, sF)) return 0;  // uniform

    // ---- the window as fp16 F' sF: rows two by two, 4 columns of the upper
    // row then the same 4 of the lower; three row pairs past the last plane are
    // cleared (read by the lowest bases against zeros)
    _Float16 *win = reinterpret_cast<_Float16 *>(lds);
    {
        const int step = (walk0.R >> 1) * p.z.rp2;
        int r = quotient(tid, g.cpr);
        if (r >= walk0.R) r = walk0.rows;
        const int dlast = (walk0.rows / 2 - 1) * p.z.rp2 + 4 + 2 * C * walk0.xc;
        int d = (r >> 1) * p.z.rp2 + (r & 1) * 4 + 2 * C * walk0.xc;
        auto store = [&](const u32x4 &v) {
            float f[C];
            centred<Vox>(v, c, f);
            _Float16 *q = win + (r < walk0.rows ? d : dlast);
#pragma unroll
            for (int h = 0; h < C / 4; ++h) {
                half4 o;
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = (_Float16)(f[4 * h + j] * sF);
                *reinterpret_cast<half4 *>(q + 8 * h) = o;
            }
            r += walk0.R;
            d += step;
        };
#pragma unroll
        for (int k = 0; k < KREG; ++k)
            if (k < walk0.kn) store(w[k]);
        for (int k = KREG; k < walk0.kn; ++k, at.next(g)) store(at.load(p, g));
        for (int i = tid; i < 3 * p.z.rp2 / 8; i += NT)
            *reinterpret_cast<u32x4 *>(win + g.ez * g.pl + 8 * i) = u32x4{0, 0, 0, 0};
    }
    __syncthreads();

    // ---- sweep: bounds of every displacement.  Of each row of displacements
    // along z the one with the largest upper end goes to the list if it may win,
    // and the row itself if its second largest may.
    const uint32_t *rowtab = reinterpret_cast<const uint32_t *>(lds + p.z.tab_off);
    u32x2 *list = reinterpret_cast<u32x2 *>(lds + p.z.l_off);
    const int sx = 2 * p.w[0] + 1, sxy = sx * (2 * p.w[1] + 1);
    const float ea = uniform(EPS * sqrtf((float)N) * (tnorm * sT) * (__uint_as_float(fmax) * sF));
    const int64_t corner = ((int64_t)g.oz0 * p.oy + g.oy0) * p.ox + g.ox0;
    int kq[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int gg = 4 * q + (lane >> 4), gy = quotient(gg, p.z.gx);
        kq[q] = gy < p.z.gyp ? gy * p.z.rp2 + (gg - gy * p.z.gx) * 8 : 0;
    }
    int lim[4];
    uint32_t ents[4];
    // shift index of plane 0 of the lane's row i
    auto row_index = [&](int i) {
        const uint32_t e = ents[i];
        const int odx = 4 * (int)(e & 0xff) + (lane & 3);
        const int ody = 4 * (int)(e >> 8 & 0xff) + (lane >> 2 & 3);
        return (g.loz + (int)(e >> 16 & 0xff) * g.tz + p.w[2]) * sxy + (g.loy + ody + p.w[1]) * sx +
               (g.lox + odx + p.w[0]);
    };
    auto push = [&](uint32_t key, uint32_t what) {
        const int k = atomicAdd(&sm.nlist, 1);
        if (k < p.z.list) list[k] = u32x2{key, what};
    };
    float low = -INFINITY;
    for (int tile = wave; tile < g.ntiles; tile += NW) {
        // largest upper bound of each row, its plane, and the second largest
        float top[4], second[4];
        int tp[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            top[i] = second[i] = -INFINITY;
            tp[i] = 0;
        }
        sweep_tile<Rec, BZ, NQ, AHEAD>(
            p, g, win, rowtab, bop, kq, corner, ea, tile, lane, lim, ents,
            [&](int i, int tau, float hi, float lo) __attribute__((always_inline)) {
                const bool in = tau < lim[i];
                const float up = in ? hi : -INFINITY;
                low = in & (lo > low) ? lo : low;
                second[i] = __builtin_amdgcn_fmed3f(up, top[i], second[i]);
                const bool take = up > top[i];
                tp[i] = take ? tau : tp[i];
                top[i] = take ? up : top[i];
            });
        // the workgroup's largest lower bound so far, then this tile's rows
        const uint32_t wl = wave_max(ordered(low));
        if (lane == 63) atomicMax(&sm.low, wl);
        if constexpr (AGAIN) {
            const uint32_t wt =
                wave_max(ordered(fmaxf(fmaxf(top[0], top[1]), fmaxf(top[2], top[3]))));
            if (lane == 63) sm.top[tile] = wt;
        }
        // (this wavefront's own maximum is among them: LDS operations of a
        // wavefront complete in order)
        const uint32_t all = *(volatile uint32_t *)&sm.low;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (lim[i] > 0 && ordered(top[i]) >= all) {
                const int idx = row_index(i);
                push(ordered(top[i]), (uint32_t)(idx + tp[i] * sxy));
                if (ordered(second[i]) >= all)
                    push(ordered(second[i]), (uint32_t)idx | (uint32_t)min(lim[i], g.tz) << 24);
            }
    }
    __syncthreads();

    // ---- the listed displacements get their own bound, with |F'| from their
    // record: sqrt(N) |F'| r = sqrt(1 + m^2), m = (sum F - N c) r, and 2^-17 of
    // the window's bound (2^-28 of Fmax for operands below fp16's range).  It is a
    // third to a twentieth of the window's: most blocks keep one displacement.
    auto own_bounds = [&](int n) {
        for (int k = tid; k < n; k += NT) {
            const u32x2 e = list[k];
            const uint32_t top = e[0];
            const int idx = (int)e[1];
            if (e[1] >> 24 || top < *(volatile uint32_t *)&sm.low) continue;
            const int iz = quotient(idx, sxy), ir = idx - iz * sxy, iy = quotient(ir, sx);
            const int64_t at_rec = ((int64_t)(g.oz0 + iz - p.w[2] - g.loz) * p.oy +
                                    (g.oy0 + iy - p.w[1] - g.loy)) * p.ox +
                                   (g.ox0 + ir - iy * sx - p.w[0] - g.lox);
            const Rec rec = static_cast<const Rec *>(p.stats)[at_rec];
            float m;
            if constexpr (sizeof(Rec) == 16)
                m = (float)((rec.s - (double)N * (double)c) * rec.r);
            else  // sums of F - 2048
                m = ((float)rec.s + (float)N * (2048.0f - c)) * rec.r;
            const float r = (float)rec.r;
            const float t = unordered(top) - ea * r;  // C r, to 2^-20 of its size and of ea r
            const float own = EPS * (tnorm * sT) * sF * rsqrtf((float)N) * (1.0f + fabsf(m)) +
                              0x1p-17f * (ea * r) + 0x1p-19f * fabsf(t);
            if (r < 0x1p86f && own < ea * r) {  // (also not taken where a term is not a number)
                atomicMax(&sm.low, ordered(t - own));
                list[k][0] = ordered(t + own);
            }
        }
    };
    // the listed displacements that reach the largest lower end, and the rows with
    // all their planes, behind the n entries of the list; false where they do not fit
    int *cand = candidates(p, lds);
    auto collect = [&](int n) {
        const uint32_t all = sm.low;
        const int room = 2 * (p.z.list - n);
        for (int k = tid; k < n; k += NT) {
            const u32x2 e = list[k];
            if (e[0] < all) continue;
            const int m = max((int)(e[1] >> 24), 1), idx = (int)(e[1] & 0xffffffu);
            const int at = atomicAdd(&sm.ncand, m);
            if (m > 1) sm.rows = 1;
            for (int j = 0; j < m; ++j)
                if (at + j < room) cand[-(at + j)] = idx + j * sxy;
        }
        __syncthreads();
        return sm.ncand <= room;
    };
    int nlist = sm.nlist;
    if (!AGAIN && nlist > few) return 0;  // uniform
    own_bounds(min(nlist, p.z.list));
    __syncthreads();
    bool fits = collect(min(nlist, p.z.list));

    // ---- broad peaks: where whole rows make more than `few` candidates, or the
    // list overflowed, the tiles that may hold the winner are swept again against
    // the bound that stands now, and every displacement that reaches it is listed
    // and bounded by itself
    if (!AGAIN) {
        if (nlist > few) return 0;  // uniform
    } else if (nlist > p.z.list || !fits || (sm.ncand > few && sm.rows)) {  // uniform
        const uint32_t all = sm.low;
        const uint64_t again = __ballot(lane < g.ntiles && sm.top[lane] >= all);
        const float cut = unordered(all);
        __syncthreads();
        if (tid == 0) sm.nlist = sm.ncand = 0;
        __syncthreads();
        int turn = 0;
        for (uint64_t left = again; left; left &= left - 1) {
            if ((turn++ & (NW - 1)) != wave) continue;
            const int tile = __ffsll((unsigned long long)left) - 1;
            sweep_tile<Rec, BZ, NQ, AHEAD>(
                p, g, win, rowtab, bop, kq, corner, ea, tile, lane, lim, ents,
                [&](int i, int tau, float hi, float) __attribute__((always_inline)) {
                    if (tau < lim[i] && hi >= cut)
                        push(ordered(hi), (uint32_t)(row_index(i) + tau * sxy));
                });
        }
        __syncthreads();
        nlist = sm.nlist;
        if (nlist > p.z.list) return 0;  // uniform
        own_bounds(nlist);
        __syncthreads();
        fits = collect(nlist);
    }
    return fits ? __builtin_amdgcn_readfirstlane(sm.ncand) : 0;
}

// The best of candidates that lie close together (a broad peak): the voxels of
// their common box are staged as F' in the window's place and every thread runs
// the FP32 search's chain for a candidate of its own.  chain(f, pitch, plane, idx)
// is the key of the displacement whose block starts at f.  Returns the shift index
// of the largest key (the smallest among equal ones; INT_MAX where every key is a
// NaN), or -1 where the box does not fit.  Uniform.
template <typename Vox, typename Key, typename Chain>
__device__ __attribute__((always_inline)) inline int pick_in_box(const Args &p, const Geo &g,
                                                                 unsigned char *lds, Small &sm,
                                                                 int ncand, float c, Chain chain) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int *cand = candidates(p, lds);
    const int sx = 2 * p.w[0] + 1, sxy = sx * (2 * p.w[1] + 1);
    auto split = [&](int idx, int (&i)[3]) {
        i[2] = quotient(idx, sxy);
        const int r = idx - i[2] * sxy;
        i[1] = quotient(r, sx);
        i[0] = r - i[1] * sx;
    };
    uint32_t top[6] = {0, 0, 0, 0, 0, 0};
    for (int k = tid; k < ncand; k += NT) {
        int i[3];
        split(cand[-k], i);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            top[a] = max(top[a], (uint32_t)i[a]);
            top[3 + a] = max(top[3 + a], 0xffffu - (uint32_t)i[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        top[a] = wave_max(top[a]);
        if (lane == 63) atomicMax(&sm.box[a], top[a]);
    }
    __syncthreads();
    int lo[3], e[3];  // the box: first displacement, voxels per axis
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = (int)(0xffffu - sm.box[3 + a]);
        e[a] = (int)sm.box[a] - lo[a] + p.b[a];
    }
    const int pitch = e[0] | 1, plane = e[1] * pitch, rows = e[1] * e[2];
    if (plane * e[2] * 4 > p.z.t_off) return -1;  // uniform
    float *box = reinterpret_cast<float *>(lds);
    const int64_t sy = p.nx, sz = (int64_t)p.nx * p.ny;
    const Vox *src = static_cast<const Vox *>(p.flt) + (g.oz0 + lo[2] - p.w[2] - g.loz) * sz +
                     (g.oy0 + lo[1] - p.w[1] - g.loy) * sy + (g.ox0 + lo[0] - p.w[0] - g.lox);
    const int n = rows * e[0];
    for (int i0 = tid; i0 < n; i0 += 4 * NT) {
        float v[4];
        int at[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u * NT, n - 1), r = quotient(i, e[0]), x = i - r * e[0];
            const int z = quotient(r, e[1]), y = r - z * e[1];
            at[u] = r * pitch + x;
            v[u] = (float)src[z * sz + y * sy + x] - c;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) box[at[u]] = v[u];
    }
    __syncthreads();
    Key bk = -INFINITY;
    int bi = INT_MAX;
    for (int k = tid; k < ncand; k += NT) {
        const int idx = cand[-k];
        int i[3];
        split(idx, i);
        const Key key = chain(box + (i[2] - lo[2]) * plane + (i[1] - lo[1]) * pitch + (i[0] - lo[0]),
                              pitch, plane, i);
        if (key > bk || (key == bk && idx < bi)) {
            bk = key;
            bi = idx;
        }
    }
    wave_best(bk, bi);
    if (lane == 63) {
        sm.key[tid >> 6] = (double)bk;
        sm.idx[tid >> 6] = bi;
    }
    __syncthreads();
    double best = sm.key[0];
    bi = sm.idx[0];
#pragma unroll
    for (int w = 1; w < NW; ++w)
        if (sm.key[w] > best || (sm.key[w] == best && sm.idx[w] < bi)) {
            best = sm.key[w];
            bi = sm.idx[w];
        }
    return __builtin_amdgcn_readfirstlane(bi);
}

// The best of the re-ranked candidates (keys in LDS beside them, published):
// largest key, smallest shift index; INT_MAX where every key is a NaN.
template <typename Key>
__device__ inline int pick(const int *cand, const Key *keys, int ncand) {
    Key bk = -INFINITY;
    int bi = INT_MAX;
    for (int k = threadIdx.x & 63; k < ncand; k += 64) {
        const Key key = keys[k];
        const int i = cand[-k];
        if (key > bk || (key == bk && i < bi)) {
            bk = key;
            bi = i;
        }
    }
    wave_best(bk, bi);
    return __builtin_amdgcn_readlane(bi, 63);
}

}  // namespace filt
}  // namespace nrr
