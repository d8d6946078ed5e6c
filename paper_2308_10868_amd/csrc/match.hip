// Exhaustive NCC block matching on gfx950.
//
// The paper's GPU algorithm (GPU section) maps one image block to one thread
// block, spreads the loop over the candidate displacements of the search
// window across the threads, and then takes the maximum similarity and its
// displacement.  This kernel keeps that outer mapping (one workgroup per
// selected block) and re-designs the inner part for CDNA:
//
//  * the block's search window of `flt` is staged in LDS, a run of CZ
//    displacement planes at a time (z-chunks, so any window size fits), and
//    the pre-operative block T is staged beside it; every staged voxel is
//    then reused by all displacements that touch it;
//  * each thread owns an RX x RY tile of (dx, dy) displacements at one dz and
//    keeps RX*RY accumulators in registers; a window row read from LDS is
//    reused by every (tile displacement, block column) pair that needs it;
//    LDS is read as single aligned dwords (4 bytes per staged element);
//  * two arithmetic forms of the cross term sum_o T(o) F(o+d):
//      DOT2 (12-bit data, exact): T' = T-2048 and F' = F-2048 as int16
//        pairs of planes (z, z+1), multiplied and accumulated exactly in int32
//        by v_dot2_i32_i16; the block's planes are grouped so no int32 partial
//        sum can overflow (|T'|, |F'| <= 2048);
//      FMA (any data): T^ = T - mean(T) in FP32 against F - c (c = the
//        block mean, rounded to an integer for 12-bit data) with v_fmac_f32,
//        summed in FP32 per block plane, then across planes (FP64 for 12-bit
//        data);
//  * the window statistics (sum F and 1/sqrt of its spread) come from a
//    per-voxel table computed once per call (stats.hip), so the epilogue per
//    displacement is a handful of operations;
//  * displacements are ranked by key = cov * rsqrt(varF), proportional to the
//    NCC (the block's own spread is a constant factor); the argmax keeps the
//    smallest shift index among equal keys and is reduced across the
//    workgroup with wavefront shuffles;
//  * the NCC reported for the winning displacement is recomputed exactly
//    (integer sums for 12-bit data, two-pass FP64 for float data) from the
//    volumes, so it does not inherit the ranking arithmetic's rounding.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "mfma_filter.h"
#include "nrr_internal.h"

namespace nrr {
namespace {

typedef short short2v __attribute__((ext_vector_type(2)));
// LDS dword read one at a time: the volatile qualifier keeps the compiler from
// merging neighbouring window reads into wider, misaligned LDS accesses, and
// the LDS address space keeps them ds_read_b32 with immediate offsets.
typedef __attribute__((address_space(3))) const volatile uint32_t lds_word;

constexpr int MAX_B = 15;  // largest block edge served
constexpr int ZPAD = 1;    // padding dwords after each staged window plane
enum Arith { DOT2 = 0, FMA = 1 };

struct Params {
    const void *ref;
    const void *flt;
    int nx, ny, nz;
    const int32_t *centers;
    int64_t n;
    int64_t first;  // first block of this launch
    int w;
    int cz;  // displacement planes per z-chunk
    const void *stats;  // StatU16 / StatF32 records over block origins
    const uint32_t *pv;  // plane-pair volume of flt (12-bit data)
    int ox, oy;
    int32_t *disp;
    float *ncc;
    float *conf;
    float *surface;  // optional ranking NCC per displacement (diagnostic instantiations)
};

// Workgroup index -> block index such that consecutive blocks (overlapping
// windows) land on the same XCD, which round-robins workgroups by index.
__device__ inline int64_t xcd_block(int64_t wg, int64_t n) {
    const int64_t q = n / 8, r = n % 8, k = wg % 8, j = wg / 8;
    return k * q + (k < r ? k : r) + j;
}

// Per-block search geometry: valid displacement range per axis (displaced
// block fully inside the volume) and the window origin in `flt`.
struct Geom {
    int cx, cy, cz;
    int lox, loy, loz;
    int dx, dy, dz;     // number of valid displacements per axis
    int wx0, wy0, wz0;  // window origin = c - h + lo
    bool inside;
};

// UNIFORM: in scalar registers (the filtered search, short of vector ones).
template <bool UNIFORM = false>
__device__ inline Geom make_geom(const Params &p, int64_t blk, int h) {
    auto coord = [&](int i) {
        const int v = p.centers[3 * blk + i];
        return UNIFORM ? __builtin_amdgcn_readfirstlane(v) : v;
    };
    Geom g;
    g.cx = coord(0);
    g.cy = coord(1);
    g.cz = coord(2);
    g.inside = g.cx - h >= 0 && g.cy - h >= 0 && g.cz - h >= 0 && g.cx + h <= p.nx - 1 &&
               g.cy + h <= p.ny - 1 && g.cz + h <= p.nz - 1;
    g.lox = max(-p.w, h - g.cx);
    g.loy = max(-p.w, h - g.cy);
    g.loz = max(-p.w, h - g.cz);
    g.dx = min(p.w, p.nx - 1 - h - g.cx) - g.lox + 1;
    g.dy = min(p.w, p.ny - 1 - h - g.cy) - g.loy + 1;
    g.dz = min(p.w, p.nz - 1 - h - g.cz) - g.loz + 1;
    g.wx0 = g.cx - h + g.lox;
    g.wy0 = g.cy - h + g.loy;
    g.wz0 = g.cz - h + g.loz;
    return g;
}

template <typename K>
__device__ inline void better(K &bk, int &bi, K k, int i) {
    if (k > bk || (k == bk && i < bi)) {
        bk = k;
        bi = i;
    }
}

// Workgroup argmax of (key, shift index): largest key, smallest index on ties.
template <int NT, typename K>
__device__ inline void wg_argmax(K &key, int &idx, K *s_key, int *s_idx) {
    for (int off = 32; off > 0; off >>= 1) {
        K ok = __shfl_xor(key, off);
        int oi = __shfl_xor(idx, off);
        better(key, idx, ok, oi);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_key[w] = key;
        s_idx[w] = idx;
    }
    __syncthreads();
    key = s_key[0];
    idx = s_idx[0];
    for (int i = 1; i < NT / 64; ++i) better(key, idx, s_key[i], s_idx[i]);
    __syncthreads();
}

template <int NT, typename T, int NV>
__device__ inline void wg_sum(T (&v)[NV], T *s_red) {
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_xor_sum(v[k]);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) s_red[w * NV + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        T s = 0;
        for (int i = 0; i < NT / 64; ++i) s += s_red[i * NV + k];
        v[k] = s;
    }
    __syncthreads();
}

__device__ inline void write_result(const Params &p, int64_t blk, int dx, int dy, int dz,
                                    float v) {
    p.disp[3 * blk] = dx;
    p.disp[3 * blk + 1] = dy;
    p.disp[3 * blk + 2] = dz;
    p.ncc[blk] = v;
    p.conf[blk] = v > 0.0f ? v : 0.0f;
}

// Stage planes [z0, z0 + pz) of the window into LDS as 4-byte elements at
// z*plane + y*pitch + x (plane >= py*pitch); element (z, y, x) = make(a, b, nb)
// where a = src(z0+z, y0+y, x0+x) and, with PAIR, b = the same voxel of the
// next plane (nb = false and b = 0 past plane `ez`), for y < ey and x < ex;
// 0 elsewhere (tile padding).  Each lane moves chunks of 4 consecutive x;
// UNR chunks per lane are loaded before any is written so several global
// loads are in flight, and the chunk coordinates advance incrementally (no
// integer division in the loop).
template <int NT, bool PAIR, int UNR, typename Src, typename Make>
__device__ inline void stage_planes(const Src *__restrict__ src, int nx, int ny, int x0, int y0,
                                    int z0, int ex, int ey, int ez, uint32_t *__restrict__ dst,
                                    int pitch, int plane, int py, int pz, Make make) {
    const int cpr = (pitch + 3) >> 2;  // chunks per row
    const int total = pz * py * cpr;
    const int drow = NT / cpr, dxc = NT - drow * cpr;
    int row = (int)threadIdx.x / cpr;
    int xc = (int)threadIdx.x - row * cpr;
    int z = row / py, y = row - z * py;
    for (int c0 = 0; c0 < total; c0 += NT * UNR) {
        Src a[UNR][4], b[UNR][4];
        int base[UNR], xs[UNR];
        bool rin[UNR], nin[UNR], live[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            live[u] = c0 + u * NT + (int)threadIdx.x < total;
            xs[u] = 4 * xc;
            base[u] = z * plane + y * pitch + 4 * xc;
            rin[u] = live[u] && y < ey && z < ez;
            nin[u] = PAIR && rin[u] && z + 1 < ez;
            const Src *s = src + ((int64_t)(z0 + z) * ny + (y0 + y)) * nx + (x0 + 4 * xc);
            const Src *s1 = s + (int64_t)ny * nx;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = 4 * xc + e < ex;
                a[u][e] = (rin[u] && in) ? s[e] : Src(0);
                b[u][e] = (PAIR && nin[u] && in) ? s1[e] : Src(0);
            }
            xc += dxc;
            y += drow;
            if (xc >= cpr) {
                xc -= cpr;
                ++y;
            }
            while (y >= py) {
                y -= py;
                ++z;
            }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            if (!live[u]) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int x = xs[u] + e;
                if (x < pitch) {
                    const bool in = rin[u] && x < ex;
                    dst[base[u] + e] = in ? make(a[u][e], b[u][e], nin[u]) : 0u;
                }
            }
        }
    }
}

// Stage planes [z0, z0 + pz) of the window from the plane-pair volume as
// plain copies into LDS at z*plane + y*pitch + x, with `pitch` and `plane`
// multiples of CW words.  Each lane moves whole CW-word row chunks (one
// global and one LDS access each); rows at or past `ey` re-read row ey-1 and
// columns past the window's own width read whatever follows in the volume
// row (the pair volume carries slack at its end), so no load needs a
// predicate.  Those extra words only feed displacements that are masked out.
template <int CW>
struct Chunk {
    typedef uint32_t type __attribute__((ext_vector_type(CW), aligned(4)));
};
constexpr int CW = 4;  // row chunk width of the DOT2 window (16-byte copies)

template <int NT, int UNR>
__device__ inline void stage_rows(const uint32_t *__restrict__ src, int nx, int ny, int x0, int y0,
                                  int z0, int ey, uint32_t *__restrict__ dst, int pitch,
                                  int plane, int py, int pz) {
    using V = typename Chunk<CW>::type;
    const int cpr = pitch / CW;  // chunks per row
    const int total = pz * py * cpr;
    const int drow = NT / cpr, dxc = NT - drow * cpr;
    int row = (int)threadIdx.x / cpr;
    int xc = (int)threadIdx.x - row * cpr;
    int z = row / py, y = row - z * py;
    for (int c0 = 0; c0 < total; c0 += NT * UNR) {
        V v[UNR];
        int off[UNR];
        bool live[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            live[u] = c0 + u * NT + (int)threadIdx.x < total;
            const int zz = live[u] ? z : 0, yy = min(y, ey - 1);
            const uint32_t *s = src + ((int64_t)(z0 + zz) * ny + (y0 + yy)) * nx + (x0 + CW * xc);
            v[u] = *reinterpret_cast<const V *>(s);
            off[u] = z * plane + y * pitch + CW * xc;
            xc += dxc;
            y += drow;
            if (xc >= cpr) {
                xc -= cpr;
                ++y;
            }
            while (y >= py) {
                y -= py;
                ++z;
            }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            if (live[u]) *reinterpret_cast<V *>(dst + off[u]) = v[u];
    }
}

// The same row-chunk staging for float volumes, storing F - c: a chunk that
// would run past the end of a volume row (the window's right edge at the
// volume border) reads its elements one by one, clamped into the row (the
// extra values only feed masked displacements).
template <int NT, int UNR>
__device__ inline void stage_rows_f32(const float *__restrict__ src, int nx, int ny, int x0, int y0,
                                      int z0, int ey, uint32_t *__restrict__ dst, int pitch,
                                      int plane, int py, int pz, float c) {
    using V = typename Chunk<CW>::type;
    const int cpr = pitch / CW;
    const int total = pz * py * cpr;
    const int drow = NT / cpr, dxc = NT - drow * cpr;
    int row = (int)threadIdx.x / cpr;
    int xc = (int)threadIdx.x - row * cpr;
    int z = row / py, y = row - z * py;
    for (int c0 = 0; c0 < total; c0 += NT * UNR) {
        float v[UNR][CW];
        int off[UNR];
        bool live[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            live[u] = c0 + u * NT + (int)threadIdx.x < total;
            const int zz = live[u] ? z : 0, yy = min(y, ey - 1), xs = x0 + CW * xc;
            const float *r = src + ((int64_t)(z0 + zz) * ny + (y0 + yy)) * nx;
            if (xs + CW <= nx) {
                const V w = *reinterpret_cast<const V *>(r + xs);
#pragma unroll
                for (int e = 0; e < CW; ++e) v[u][e] = __uint_as_float(w[e]);
            } else {
#pragma unroll
                for (int e = 0; e < CW; ++e) v[u][e] = r[min(xs + e, nx - 1)];
            }
            off[u] = z * plane + y * pitch + CW * xc;
            xc += dxc;
            y += drow;
            if (xc >= cpr) {
                xc -= cpr;
                ++y;
            }
            while (y >= py) {
                y -= py;
                ++z;
            }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            if (live[u]) {
                // word writes: rows start at any word (odd plane stride)
#pragma unroll
                for (int e = 0; e < CW; ++e) dst[off[u] + e] = __float_as_uint(v[u][e] - c);
            }
    }
}

// Exact int32 grouping for DOT2: a plane contributes at most B*B*2048*2048.
template <int B>
struct Groups {
    static constexpr int P = (B + 1) / 2;  // plane pairs of the block
    static constexpr long long PLANE_MAX = (long long)B * B * 2048 * 2048;
    static constexpr int GPAIRS = (int)(2147483647LL / PLANE_MAX) / 2;  // pairs per group
    static constexpr int NG = (P + GPAIRS - 1) / GPAIRS;
    static_assert(GPAIRS >= 1, "block edge too large for exact int32 groups");
};

// DOT2 cross terms X(d) = sum_o T'(o) F'(o + d) of an RX x RY tile of
// displacements at one dz: `tp` is the block's pair table [P][B][BP], `base`
// the tile's first window row and column, and the window plane of pair m is
// in ring slot (slot + 2m) mod R.  Exact: int32 groups of plane pairs that
// cannot overflow, combined in FP64 when a block needs more than one.
template <int B, int RX, int RY, typename XT>
__device__ __attribute__((always_inline)) inline void dot2_cross(
    const uint32_t *tp, const uint32_t *base, int slot, int R, int plane, int pitch,
    XT (&xacc)[RX][RY]) {
    constexpr int P = Groups<B>::P, GP = Groups<B>::GPAIRS, NG = Groups<B>::NG;
    constexpr int BP = (B + 3) & ~3;
    int acc[RX][RY], acc0[RX][RY];
    double dacc[NG > 2 ? RX : 1][NG > 2 ? RY : 1];
#pragma unroll
    for (int i = 0; i < RX; ++i)
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            acc[i][j] = 0;
            acc0[i][j] = 0;
            if constexpr (NG > 2) dacc[i][j] = 0.0;
        }
    for (int m = 0; m < P; ++m) {
        int tq[B][B];
        const uint32_t *tpm = tp + m * B * BP;
#pragma unroll
        for (int oy = 0; oy < B; ++oy)
#pragma unroll
            for (int ox = 0; ox < B; ++ox)  // uniform: kept in scalar registers
                tq[oy][ox] = __builtin_amdgcn_readfirstlane((int)tpm[oy * BP + ox]);
        const lds_word *wm = (const lds_word *)(base + slot * plane);
        slot += 2;
        if (slot >= R) slot -= R;
        // rows are software-pipelined: row yw+1 is read while row yw
        // is multiplied
        int fr[2][RX + B - 1];
#pragma unroll
        for (int xw = 0; xw < RX + B - 1; ++xw) fr[0][xw] = (int)wm[xw];
#pragma unroll
        for (int yw = 0; yw < RY + B - 1; ++yw) {
            if (yw + 1 < RY + B - 1) {
#pragma unroll
                for (int xw = 0; xw < RX + B - 1; ++xw)
                    fr[(yw + 1) & 1][xw] = (int)wm[(yw + 1) * pitch + xw];
            }
            const int *f = fr[yw & 1];
#pragma unroll
            for (int j = 0; j < RY; ++j) {
                const int oy = yw - j;
                if (oy < 0 || oy >= B) continue;
#pragma unroll
                for (int i = 0; i < RX; ++i)
#pragma unroll
                    for (int ox = 0; ox < B; ++ox)
                        acc[i][j] = __builtin_amdgcn_sdot2(
                            __builtin_bit_cast(short2v, f[i + ox]),
                            __builtin_bit_cast(short2v, tq[oy][ox]), acc[i][j],
                            false);
            }
        }
        if constexpr (NG == 2) {
            if (m == GP - 1) {
#pragma unroll
                for (int i = 0; i < RX; ++i)
#pragma unroll
                    for (int j = 0; j < RY; ++j) {
                        acc0[i][j] = acc[i][j];
                        acc[i][j] = 0;
                    }
            }
        } else if constexpr (NG > 2) {
            if ((m + 1) % GP == 0) {
#pragma unroll
                for (int i = 0; i < RX; ++i)
#pragma unroll
                    for (int j = 0; j < RY; ++j) {
                        dacc[i][j] += (double)acc[i][j];
                        acc[i][j] = 0;
                    }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RX; ++i)
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            if constexpr (NG == 1)
                xacc[i][j] = acc[i][j];
            else if constexpr (NG == 2)
                xacc[i][j] = (double)acc0[i][j] + (double)acc[i][j];
            else
                xacc[i][j] = dacc[i][j] + (double)acc[i][j];
        }
}

// Ranking key of float data from a cross term and its record.
__device__ inline double key_f32_of(double dN, float x, double tsum, const StatF32 &rec, float c) {
    const double cov = dN * (double)x - tsum * (rec.s - dN * (double)c);
    return cov * rec.r;
}

// Ranking of a tile: key = N*cov * rsqrt(N*varF), proportional to the NCC for
// the block at hand; keeps the largest key and, among equal keys, the
// smallest shift index (irow + j*side + i).  Displacements past the valid
// extents (nvx, nvy) are masked without a branch.  For 12-bit data the staged
// F sums are offset by `fshift` from the table's.
template <bool U16, bool SHIFT, int RX, int RY, typename Rec, typename XT, typename KeyT,
          bool SURF = false>
__device__ __attribute__((always_inline)) inline void rank_tile(
    const Rec (&rec)[RX][RY], const XT (&xacc)[RX][RY], double dN, double tsum, double fshift,
    float c, int nvx, int nvy, int irow, int side, KeyT &tk, int &ti, float *surf = nullptr,
    double inv_vt = 0.0) {
#pragma unroll
    for (int j = 0; j < RY; ++j)
#pragma unroll
        for (int i = 0; i < RX; ++i) {  // increasing shift index
            const bool valid = i < nvx && j < nvy;
            KeyT key;
            if constexpr (U16) {
                const double cov =
                    __builtin_fma(dN, (double)xacc[i][j],
                                  -tsum * (SHIFT ? (double)rec[i][j].s + fshift : (double)rec[i][j].s));
                key = (float)cov * rec[i][j].r;
            } else {
                key = key_f32_of(dN, xacc[i][j], tsum, rec[i][j], c);
            }
            const bool take = valid && key > tk;  // ties keep the smaller index
            tk = take ? key : tk;
            ti = take ? irow + j * side + i : ti;
            if constexpr (SURF)  // NCC = key / sqrt(N varT)
                if (valid) surf[irow + j * side + i] = (float)((double)key * inv_vt);
        }
}

// Workgroup scratch of the reductions (any NT <= 1024).
struct Small {
    double key[16];
    int idx[16];
    long long red[16 * 5];
    double redd[16 * 3];
};

// Search of one block `blk` (its window staged in `lds`); the body shared by
// the per-block kernel and the batched kernel.  Every thread of the NT-wide
// workgroup calls it; it ends with all LDS reads done by the thread itself,
// so a caller that reuses LDS for another block synchronises first.
template <typename Vox, int ARITH, int B, int RX, int RY, int NT, bool PF, bool SURF = false>
__device__ __attribute__((always_inline)) inline void match_one(const Params &p, int64_t blk,
                                                                unsigned char *lds, Small &sm,
                                                                int tid) {
    constexpr bool U16 = sizeof(Vox) == 2;
    static_assert(ARITH == FMA || U16, "DOT2 needs 12-bit data");
    constexpr int H = (B - 1) / 2, N = B * B * B, BP = (B + 3) & ~3;
    constexpr int P = Groups<B>::P, GP = Groups<B>::GPAIRS, NG = Groups<B>::NG;
    constexpr int TPL = ARITH == DOT2 ? P : B;  // block planes (pairs) in the T table
    constexpr int TP_WORDS = TPL * B * BP;
    using KeyT = typename std::conditional<U16, float, double>::type;
    uint32_t *tp = reinterpret_cast<uint32_t *>(lds);                  // [TPL][B][BP]
    uint32_t *win = reinterpret_cast<uint32_t *>(lds + TP_WORDS * 4);  // [cz+B-1][PY][PX]
    KeyT *s_key = reinterpret_cast<KeyT *>(sm.key);
    int *s_idx = sm.idx;
    long long *s_red = sm.red;
    double *s_redd = sm.redd;
    static_assert(NT <= 1024, "reduction scratch is sized for 16 wavefronts");

    const Geom g = make_geom(p, blk, H);
    if (!g.inside) {
        if (tid == 0) write_result(p, blk, 0, 0, 0, NAN);
        return;
    }
    const Vox *ref = static_cast<const Vox *>(p.ref);
    const Vox *flt = static_cast<const Vox *>(p.flt);
    const int txn = (g.dx + RX - 1) / RX, tyn = (g.dy + RY - 1) / RY;
    const int PX = txn * RX + B - 1, PY = tyn * RY + B - 1;
    // LDS row pitch: DOT2 and float windows are staged in whole CW-word chunks
    constexpr bool ROWS = ARITH == DOT2 || !U16;
    const int pitch = ROWS ? (PX + CW - 1) / CW * CW : PX;
    const int ex = g.dx + B - 1, ey = g.dy + B - 1;
    auto tval = [&](int o) {
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        return ref[((int64_t)(g.cz - H + oz) * p.ny + (g.cy - H + oy)) * p.nx + (g.cx - H + ox)];
    };

    // ---- block statistics and the staged T table
    // Plane stride: lanes of a wavefront take consecutive dz, so the stride
    // spreads their reads over the LDS banks: odd (one pad dword) for the
    // element-staged and the float windows, 4 x odd for the 12-bit
    // chunk-staged windows (whole 16-byte chunks: 16 consecutive planes still
    // hit distinct banks).
    // (float windows: an odd plane stride in words, since their products
    // read single words with consecutive lanes on consecutive dz planes; a
    // stride of 4 x odd words put 64 lanes on 8 banks)
    const int plane = ROWS ? (U16 ? PY * pitch + (((PY * pitch / CW) & 1) ? 0 : CW)
                                  : PY * pitch + 1)
                           : PY * pitch + ZPAD;
    auto stage_chunk = [&](int zc0, int ezc, float c) {
        if constexpr (ARITH == DOT2)  // plain copies of the precomputed pair words
            stage_rows<NT, 8>(p.pv, p.nx, p.ny, g.wx0, g.wy0, g.wz0 + zc0, ey, win, pitch,
                                  plane, PY, ezc);
        else if constexpr (!U16)
            stage_rows_f32<NT, 4>(reinterpret_cast<const float *>(flt), p.nx, p.ny, g.wx0, g.wy0,
                                  g.wz0 + zc0, ey, win, pitch, plane, PY, ezc, c);
        else
            stage_planes<NT, false, 4>(
                flt, p.nx, p.ny, g.wx0, g.wy0, g.wz0 + zc0, ex, ey, ezc, win, PX, plane, PY, ezc,
                [c](Vox a, Vox, bool) { return __float_as_uint((float)a - c); });
    };
    long long st[2] = {0, 0};  // 12-bit: exact sums of T and T^2
    double tmean;
    double vtn = 0.0;  // N sum T^2 - (sum T)^2 of the T actually used (surface output)
    long long sT = 0;   // DOT2: sum (T - 2048)
    double sTc = 0.0;   // FMA: sum of the centred float T^ actually used
    float c = 0.0f;     // FMA: F is staged as F - c
    if constexpr (ARITH == DOT2) {
        // one pass: each T voxel is read once, into its plane-pair word, and
        // counted into the exact sums; the first window chunk's loads are
        // issued before the reduction's barrier so both latencies overlap
        for (int i = tid; i < TP_WORDS; i += NT) {
            const int pl = i / (B * BP), oy = (i / BP) % B, ox = i % BP;
            uint32_t w = 0;
            if (ox < B) {
                const int z0 = 2 * pl, z1 = 2 * pl + 1;
                const int lo = (int)tval((z0 * B + oy) * B + ox);
                const int hi = z1 < B ? (int)tval((z1 * B + oy) * B + ox) : 2048;
                st[0] += lo + (z1 < B ? hi : 0);
                st[1] += (long long)lo * lo + (z1 < B ? (long long)hi * hi : 0);
                w = (uint32_t)(uint16_t)(lo - 2048) | ((uint32_t)(uint16_t)(hi - 2048) << 16);
            }
            tp[i] = w;
        }
        stage_chunk(0, min(p.cz, g.dz) + B - 1, 0.0f);
        wg_sum<NT, long long, 2>(st, s_red);  // its barrier also publishes tp and the window
        if ((long long)N * st[1] - st[0] * st[0] == 0) {  // flat block: all NCC are 0
            if (tid == 0) write_result(p, blk, g.lox, g.loy, g.loz, 0.0f);
            return;
        }
        tmean = (double)st[0] / (double)N;
        sT = st[0] - 2048ll * N;
        vtn = (double)((long long)N * st[1] - st[0] * st[0]);
    } else {
        double sd[1] = {0.0};
        for (int o = tid; o < N; o += NT) {
            const Vox v = tval(o);
            if constexpr (U16) {
                st[0] += v;
                st[1] += (long long)v * v;
            }
            sd[0] += (double)v;
        }
        wg_sum<NT, double, 1>(sd, s_redd);
        tmean = sd[0] / (double)N;
        if constexpr (U16) wg_sum<NT, long long, 2>(st, s_red);
        // 12-bit data keep c an integer (exact floats)
        c = U16 ? (float)llrint(tmean) : (float)tmean;
        double ctr[2] = {0.0, 0.0};  // sum T^, sum T^^2 of the float values used
        for (int i = tid; i < TP_WORDS; i += NT) {
            const int pl = i / (B * BP), oy = (i / BP) % B, ox = i % BP;
            uint32_t w = 0;
            if (ox < B) {
                const float v = (float)((double)tval((pl * B + oy) * B + ox) - tmean);
                ctr[0] += (double)v;
                ctr[1] += (double)v * (double)v;
                w = __float_as_uint(v);
            }
            tp[i] = w;
        }
        stage_chunk(0, min(p.cz, g.dz) + B - 1, c);
        wg_sum<NT, double, 2>(ctr, s_redd);  // barrier publishes tp and the window
        sTc = ctr[0];
        vtn = (double)N * ctr[1] - ctr[0] * ctr[0];
        if (!(ctr[1] > 0.0)) {  // flat block
            if (tid == 0) write_result(p, blk, g.lox, g.loy, g.loz, 0.0f);
            return;
        }
    }

    // ---- exhaustive search, one z-chunk of displacement planes at a time
    const double dN = (double)N;
    const int side = 2 * p.w + 1;
    KeyT bk = -INFINITY;
    int bi = INT_MAX;
    // DOT2 keeps the staged planes in a ring of R plane slots (window plane q
    // in slot q mod R), so a later chunk stages only the planes it adds
    const int R = min(p.cz, g.dz) + B - 1;
    int staged = R;  // window planes [0, staged) staged so far (chunk 0 above)
    for (int zc0 = 0; zc0 < g.dz; zc0 += p.cz) {
        const int czn = min(p.cz, g.dz - zc0);  // displacement planes in this chunk
        const int ezc = czn + B - 1;            // window planes in this chunk
        if (zc0 > 0) {                          // the first chunk was staged above
            __syncthreads();                    // previous chunk fully consumed
            if constexpr (ARITH == DOT2) {
                // new planes [staged, zc0 + ezc) replace planes below zc0
                for (int q = staged; q < zc0 + ezc;) {
                    const int slot = q % R, n = min(zc0 + ezc - q, R - slot);
                    stage_rows<NT, 8>(p.pv, p.nx, p.ny, g.wx0, g.wy0, g.wz0 + q, ey,
                                          win + slot * plane, pitch, plane, PY, n);
                    q += n;
                }
                staged = zc0 + ezc;
            } else {
                stage_chunk(zc0, ezc, c);
            }
            __syncthreads();
        }
        const int ntiles = txn * tyn * czn;
        for (int t = tid; t < ntiles; t += NT) {
            // consecutive lanes take consecutive dz (then x, then y tiles): with
            // the plane padding this spreads a wavefront's reads over the banks
            const int dzl = t % czn, tx = (t / czn) % txn, ty = t / (czn * txn);
            const int dz = zc0 + dzl;
            const uint32_t *base =
                win + (ARITH == DOT2 ? 0 : dzl * plane) + ty * RY * pitch + tx * RX;
            // the tile's table records: all loaded at once (coordinates clamped
            // into the valid range, so every load is in bounds), either before
            // the multiply loop (PF: their latency hides behind it) or after
            using Rec = typename std::conditional<U16, StatU16, StatF32>::type;
            const Rec *table = static_cast<const Rec *>(p.stats);
            Rec rec[RX][RY];
            // records of displacements past the valid range read neighbouring
            // origins (or the table's slack past its end); they are masked out
            const Rec *rb = table + ((int64_t)(g.wz0 + dz) * p.oy + (g.wy0 + ty * RY)) * p.ox +
                            (g.wx0 + tx * RX);
            auto load_recs = [&]() {
#pragma unroll
                for (int j = 0; j < RY; ++j)
#pragma unroll
                    for (int i = 0; i < RX; ++i) rec[i][j] = rb[j * p.ox + i];
            };
            if constexpr (PF) load_recs();
            // cross term of each displacement of the tile, kept in the narrowest
            // exact type (converted to FP64 per displacement in the ranking)
            // FMA (B >= 5): FP32 sums of one block plane at a time, carried
            // across planes in FP64 for 12-bit data and in a second FP32 sum
            // for float data, so no running sum takes more than B^2 roundings
            // at its own size: where a window's local level lies far from the
            // block's (F - c large, varF small) a whole-block FP32 sum ranks
            // with about 4x the error
            constexpr bool FLUSH = ARITH == FMA && B >= 5;
            using XT = typename std::conditional<
                ARITH == DOT2, typename std::conditional<NG == 1, int, double>::type,
                typename std::conditional<FLUSH && U16, double, float>::type>::type;
            XT xacc[RX][RY];
            if constexpr (ARITH == DOT2) {
                dot2_cross<B, RX, RY>(tp, base, (zc0 + dzl) % R, R, plane, pitch, xacc);
            } else {
                float acc[RX][RY];
#pragma unroll
                for (int i = 0; i < RX; ++i)
#pragma unroll
                    for (int j = 0; j < RY; ++j) {
                        acc[i][j] = 0.0f;
                        xacc[i][j] = 0;
                    }
                for (int oz = 0; oz < B; ++oz) {
                    float tq[B][B];
                    const uint32_t *tpz = tp + oz * B * BP;
#pragma unroll
                    for (int oy = 0; oy < B; ++oy)
#pragma unroll
                        for (int ox = 0; ox < B; ++ox)
                            tq[oy][ox] = __uint_as_float(tpz[oy * BP + ox]);
                    const lds_word *wz = (const lds_word *)(base + oz * plane);
                    float fr[2][RX + B - 1];
#pragma unroll
                    for (int xw = 0; xw < RX + B - 1; ++xw) fr[0][xw] = __uint_as_float(wz[xw]);
#pragma unroll
                    for (int yw = 0; yw < RY + B - 1; ++yw) {
                        if (yw + 1 < RY + B - 1) {
#pragma unroll
                            for (int xw = 0; xw < RX + B - 1; ++xw)
                                fr[(yw + 1) & 1][xw] = __uint_as_float(wz[(yw + 1) * pitch + xw]);
                        }
                        const float *f = fr[yw & 1];
#pragma unroll
                        for (int j = 0; j < RY; ++j) {
                            const int oy = yw - j;
                            if (oy < 0 || oy >= B) continue;
#pragma unroll
                            for (int i = 0; i < RX; ++i)
#pragma unroll
                                for (int ox = 0; ox < B; ++ox)
                                    acc[i][j] = __builtin_fmaf(f[i + ox], tq[oy][ox], acc[i][j]);
                        }
                    }
                    if constexpr (FLUSH) {
#pragma unroll
                        for (int i = 0; i < RX; ++i)
#pragma unroll
                            for (int j = 0; j < RY; ++j) {
                                xacc[i][j] += (XT)acc[i][j];
                                acc[i][j] = 0.0f;
                            }
                    }
                }
                if constexpr (!FLUSH) {
#pragma unroll
                    for (int i = 0; i < RX; ++i)
#pragma unroll
                        for (int j = 0; j < RY; ++j) xacc[i][j] = acc[i][j];
                }
            }
            // ---- rank the tile's displacements: key = N*cov * rsqrt(N*varF);
            // invalid displacements are masked, no branch per displacement
            if constexpr (!PF) load_recs();
            const int irow = ((g.loz + dz + p.w) * side + (g.loy + ty * RY + p.w)) * side +
                             (g.lox + tx * RX + p.w);
            // sum of the staged F: DOT2 F-2048 (= the table's s), FMA F-c
            const double fshift = ARITH == DOT2 ? 0.0 : dN * (2048.0 - (double)c);
            const double tsum = ARITH == DOT2 ? (double)sT : sTc;  // sum of the staged T
            KeyT tk = -INFINITY;
            int ti = INT_MAX;
            if constexpr (SURF)
                rank_tile<U16, ARITH != DOT2, RX, RY, Rec, XT, KeyT, true>(
                    rec, xacc, dN, tsum, fshift, c, g.dx - tx * RX, g.dy - ty * RY, irow, side, tk,
                    ti, p.surface + blk * side * side * side, 1.0 / sqrt(vtn));
            else
                rank_tile<U16, ARITH != DOT2>(rec, xacc, dN, tsum, fshift, c, g.dx - tx * RX,
                                              g.dy - ty * RY, irow, side, tk, ti);
            better(bk, bi, tk, ti);
        }
    }
    wg_argmax<NT>(bk, bi, s_key, s_idx);
    if (bi == INT_MAX) {  // every key NaN (non-finite input): report, never index
        if (tid == 0) write_result(p, blk, 0, 0, 0, NAN);
        return;
    }

    // ---- exact NCC at the winning displacement, from the volumes
    const int ddx = bi % side - p.w, ddy = (bi / side) % side - p.w, ddz = bi / (side * side) - p.w;
    auto fval = [&](int o) {
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        return flt[((int64_t)(g.cz - H + ddz + oz) * p.ny + (g.cy - H + ddy + oy)) * p.nx +
                   (g.cx - H + ddx + ox)];
    };
    if constexpr (U16) {
        // the exact sums of T and T^2 are already known (st); F and TF here.
        // Sums of shifted values (F - 2048, T - 2048) give the same covariance
        // and spreads as the raw values, and st is shift-free.
        long long sums[3] = {0, 0, 0};  // F, F^2, TF
        long long tS = st[0];             // sum of T in the same offset frame
        if constexpr (ARITH == DOT2) {
            // pair words of the winning window: from the LDS ring when its planes
            // are still staged, else from the plane-pair volume; the block's own
            // words are in the T table.  Values are int16, offset by -2048.
            tS = st[0] - 2048ll * N;
            const int zr = ddz - g.loz, yr = ddy - g.loy, xr = ddx - g.lox;
            const bool in_lds = zr >= staged - R;
            for (int i = tid; i < P * B * B; i += NT) {
                const int m = i / (B * B), oy = (i / B) % B, ox = i % B;
                const uint32_t tw = tp[(m * B + oy) * BP + ox];
                const int q = zr + 2 * m;
                const uint32_t fw =
                    in_lds ? win[(q % R) * plane + (yr + oy) * pitch + (xr + ox)]
                           : p.pv[((int64_t)(g.wz0 + q) * p.ny + (g.wy0 + yr + oy)) * p.nx +
                                  (g.wx0 + xr + ox)];
                const long long tlo = (short)(tw & 0xffff), thi = (short)(tw >> 16);
                const long long flo = (short)(fw & 0xffff);
                const long long fhi = 2 * m + 1 < B ? (long long)(short)(fw >> 16) : 0;
                sums[0] += flo + fhi;
                sums[1] += flo * flo + fhi * fhi;
                sums[2] += tlo * flo + thi * fhi;
            }
        } else {
            for (int o = tid; o < N; o += NT) {
                const long long tv = tval(o), fv = fval(o);
                sums[0] += fv;
                sums[1] += fv * fv;
                sums[2] += tv * fv;
            }
        }
        wg_sum<NT, long long, 3>(sums, s_red);
        if (tid == 0) {
            const long long vt = (long long)N * st[1] - st[0] * st[0];
            const long long vf = (long long)N * sums[1] - sums[0] * sums[0];
            const long long cv = (long long)N * sums[2] - tS * sums[0];
            const double v = (vt > 0 && vf > 0) ? (double)cv / sqrt((double)vt * (double)vf) : 0.0;
            write_result(p, blk, ddx, ddy, ddz, (float)v);
        }
    } else {
        double m2[1] = {0.0};
        for (int o = tid; o < N; o += NT) m2[0] += (double)fval(o);
        wg_sum<NT, double, 1>(m2, s_redd);
        const double fmean = m2[0] / (double)N;
        double q[3] = {0.0, 0.0, 0.0};  // A, B, X of the two-pass Pearson form
        for (int o = tid; o < N; o += NT) {
            const double a = (double)tval(o) - tmean, b = (double)fval(o) - fmean;
            q[0] += a * a;
            q[1] += b * b;
            q[2] += a * b;
        }
        wg_sum<NT, double, 3>(q, s_redd);
        if (tid == 0) {
            const double ab = q[0] * q[1];
            const double v = ab > 0.0 ? q[2] / sqrt(ab) : 0.0;
            write_result(p, blk, ddx, ddy, ddz, (float)v);
        }
    }
}


template <typename Vox, int ARITH, int B, int RX, int RY, int NT, bool PF>
__global__ __launch_bounds__(NT) void k_match(Params p) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Small sm;
    match_one<Vox, ARITH, B, RX, RY, NT, PF>(p, p.first + xcd_block(blockIdx.x, gridDim.x), lds,
                                             sm, threadIdx.x);
}

// The same search also writing the ranking NCC of every valid displacement
// to p.surface (a diagnostic of the ranking arithmetic's error).
template <typename Vox, int ARITH, int B, int RX, int RY, int NT, bool PF>
__global__ __launch_bounds__(NT) void k_match_surf(Params p) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Small sm;
    match_one<Vox, ARITH, B, RX, RY, NT, PF, true>(
        p, p.first + xcd_block(blockIdx.x, gridDim.x), lds, sm, threadIdx.x);
}


// The float search behind the matrix-core filter (mfma_filter.h): the same
// winner, bit for bit, as match_one's FMA form, which it calls for the blocks
// the filter leaves.  Every thread of the 256-thread workgroup calls it.
// What bounds the FMA form is its vector issue (30% of the FP32 peak at
// b = 7, W = 10); the filter moves the products to fp16 matrix instructions
// and leaves the vector units one bound per displacement.  5508 blocks of
// 256x256x124 float voxels, b = 7, W = 10: 0.29 ms against 0.66.  It waits for
// memory about as the 12-bit matrix-core search does, once per block.
template <int B>
struct FiltShape {
    static constexpr int NQ = ((B + 6) / 4 * ((B + 4) / 2) + 3) / 4;
    static constexpr int KREG = B == 5 ? 20 : B == 7 ? 24 : 40;  // window chunks held per thread
    static constexpr int AHEAD = B == 7 ? 3 : B == 5 ? 5 : 5;    // planes between a record's load and its use
    static constexpr int WAVES = B == 9 ? 1 : 2;   // wavefronts per SIMD the registers allow
    // candidates above which sweeping broad peaks again costs less than ranking all
    static constexpr int FEW = B == 5 ? 256 : 128;
};

template <int B>
__device__ __attribute__((always_inline)) inline void match_one_filtered(
    const Params &p, const filt::Args &fa, int64_t blk, unsigned char *lds, Small &sm,
    filt::Small &fs) {
    using S = FiltShape<B>;
    constexpr int H = (B - 1) / 2, N = B * B * B, BP = (B + 3) & ~3, NT = 256;
    constexpr int TP_WORDS = B * B * BP;
    constexpr int TPT = (N + NT - 1) / NT, TPI = (TP_WORDS + NT - 1) / NT;
    const Geom g = make_geom<true>(p, blk, H);
    const int tid = threadIdx.x;
    if (!g.inside) {
        if (tid == 0) write_result(p, blk, 0, 0, 0, NAN);
        return;
    }
    const float *ref = static_cast<const float *>(p.ref);
    const float *flt = static_cast<const float *>(p.flt);
    const int64_t nxy = (int64_t)p.nx * p.ny;
    const int64_t rbase = (int64_t)(g.cz - H) * nxy + (int64_t)(g.cy - H) * p.nx + (g.cx - H);
    // the block's voxels in the order of the FMA form's two sums over them,
    // then the window, all in flight together
    float tv[TPT], tw[TPI];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int o = min(tid + k * NT, N - 1);
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        tv[k] = ref[rbase + oz * nxy + (int64_t)oy * p.nx + ox];
    }
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
        const int i = tid + k * NT;
        const int oz = min(i / (B * BP), B - 1), oy = (i / BP) % B, ox = min(i % BP, B - 1);
        tw[k] = ref[rbase + oz * nxy + (int64_t)oy * p.nx + ox];
    }
    filt::Geo fg = filt::geometry<float>(fa, g.cx, g.cy, g.cz);
    filt::Walk<float> walk0;
    walk0.start(fa, fg);
    filt::Walk<float> at = walk0;
    filt::u32x4 w[S::KREG];
#pragma unroll
    for (int k2 = 0; k2 < S::KREG; k2 += 2)
        if (k2 < walk0.kn) {
#pragma unroll
            for (int k = k2; k < k2 + 2; ++k) {
                w[k] = at.load(fa, fg);
                at.next(fg);
            }
        }
    filt::open_block(fa, fg, lds, fs);

    // T^ = T - mean as floats, its sums: the FMA form's operations.  The largest
    // |T^| follows from the smallest and largest voxel (the same operations,
    // monotone; a NaN among them makes the mean one).
    double sd[1] = {0.0};
    uint32_t tmn = 0xffffffffu, tmx = 0;
#pragma unroll
    for (int k = 0; k < TPT; ++k)
        if (tid + k * NT < N) {
            sd[0] += (double)tv[k];
            tmn = min(tmn, filt::ordered(tv[k]));
            tmx = max(tmx, filt::ordered(tv[k]));
        }
    tmn = ~wave_max(~tmn);
    tmx = wave_max(tmx);
    if ((tid & 63) == 63) {
        fs.tmin[tid >> 6] = tmn;
        fs.tmax[tid >> 6] = tmx;
    }
    wg_sum<NT, double, 1>(sd, sm.redd);  // its barrier publishes the extremes too
    const double tmean = uniform(sd[0] / (double)N);
    const float c = uniform((float)tmean);
    float sT = 0.0f;
    bool scales = filt::block_scale(fs, tmean, sT);
    double ctr[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
        const int i = tid + k * NT;
        const int oz = i / (B * BP), oy = (i / BP) % B, ox = i % BP;
        if (i >= TP_WORDS || ox >= B) continue;
        const float v = (float)((double)tw[k] - tmean);
        ctr[0] += (double)v;
        ctr[1] += (double)v * (double)v;
        filt::put_voxel(fa, lds, ox, oy, oz, v, sT);
    }
    wg_sum<NT, double, 2>(ctr, sm.redd);  // its barriers publish T^
    if (!(ctr[1] > 0.0)) {  // flat block
        if (tid == 0) write_result(p, blk, g.lox, g.loy, g.loz, 0.0f);
        return;
    }
    const float *tf = reinterpret_cast<const float *>(lds + fa.z.t_off);
    const double dN = (double)N, tsum = uniform(ctr[0]);
    const int side = 2 * p.w + 1;
    const StatF32 *table = static_cast<const StatF32 *>(p.stats);
    int ncand = scales ? filt::search<float, B, S::NQ, S::KREG, S::AHEAD, true>(
                             fa, fg, lds, fs, w, walk0, at, c, uniform((float)sqrt(ctr[1])), sT,
                             S::FEW)
                       : 0;
    const int *cand = filt::candidates(fa, lds);
    int best = cand[0];
    constexpr int PER = 64 / B;  // candidates per wavefront step
    int picked = -1;
    if (ncand > 2 * filt::NW * PER)  // two turns of the loop below
        picked = filt::pick_in_box<float, double>(
            fa, fg, lds, fs, ncand, c,
            [&](const float *f, int pitch, int plane, const int (&i)[3]) {
                // the FMA form's key: plane sums, added in order
                float x = 0.0f;
#pragma unroll 1  // (a plane's T^ in registers, not the block's)
                for (int oz = 0; oz < B; ++oz) {
                    float acc = 0.0f;
#pragma unroll
                    for (int oy = 0; oy < B; ++oy)
#pragma unroll
                        for (int ox = 0; ox < B; ++ox)
                            acc = __builtin_fmaf(f[oz * plane + oy * pitch + ox],
                                                 tf[(oz * B + oy) * B + ox], acc);
                    x += acc;
                }
                const int64_t x0 = g.cx - H + i[0] - p.w, y0 = g.cy - H + i[1] - p.w,
                              z0 = g.cz - H + i[2] - p.w;
                return key_f32_of(dN, x, tsum, table[(z0 * p.oy + y0) * p.ox + x0], c);
            });
    if (picked >= 0) {
        best = picked;
    } else if (ncand > filt::SPREAD) {
        ncand = 0;
    } else if (ncand > 1) {
        // the FMA form's key of each candidate: lane oz sums block plane oz, the
        // plane sums are added in order
        double *keys = filt::candidate_keys<double>(fa, lds);
        const int lane = tid & 63, sub = lane / B, oz = lane - sub * B;
        for (int k0 = (tid >> 6) * PER; k0 < ncand; k0 += filt::NW * PER) {
            const int k = k0 + sub;
            const bool on = sub < PER && k < ncand;
            const int id = on ? cand[-k] : 0;
            const int iz = id / (side * side), ir = id - iz * side * side, iy = ir / side,
                      ix = ir - iy * side;
            const int x0 = g.cx - H + ix - p.w, y0 = g.cy - H + iy - p.w, z0 = g.cz - H + iz - p.w;
            float acc = 0.0f;
            if (on) {
                const float *f = flt + (int64_t)(z0 + oz) * nxy + (int64_t)y0 * p.nx + x0;
                const float *t = tf + oz * B * B;
#pragma unroll
                for (int oy = 0; oy < B; ++oy)
#pragma unroll
                    for (int ox = 0; ox < B; ++ox)
                        acc = __builtin_fmaf(f[(int64_t)oy * p.nx + ox] - c, t[oy * B + ox], acc);
            }
            float x = 0.0f;
#pragma unroll
            for (int j = 0; j < B; ++j) x += __shfl(acc, (lane - oz + j) & 63);
            if (on && oz == 0)
                keys[k] = key_f32_of(dN, x, tsum,
                                     table[((int64_t)z0 * p.oy + y0) * p.ox + x0], c);
        }
        __syncthreads();
        best = filt::pick(cand, keys, ncand);
    }
    if (best == INT_MAX) ncand = 0;
    // an opaque copy of the thread index: what follows recomputes its
    // addresses instead of holding them in registers through the sweep
    int t2 = tid;
    asm volatile("" : "+v"(t2));
    if (ncand == 0) {  // uniform
        __syncthreads();
        match_one<float, FMA, B, 4, 4, NT, false>(p, blk, lds, sm, t2);
        return;
    }
    const int ddx = best % side - p.w, ddy = (best / side) % side - p.w,
              ddz = best / (side * side) - p.w;
    const int64_t fbase = rbase + ddz * nxy + (int64_t)ddy * p.nx + ddx;
    float fv[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int o = min(t2 + k * NT, N - 1);
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        fv[k] = flt[fbase + oz * nxy + (int64_t)oy * p.nx + ox];
    }
    double m2[1] = {0.0};
#pragma unroll
    for (int k = 0; k < TPT; ++k)
        if (t2 + k * NT < N) m2[0] += (double)fv[k];
    wg_sum<NT, double, 1>(m2, sm.redd);
    const double fmean = m2[0] / (double)N;
    double q[3] = {0.0, 0.0, 0.0};  // A, B, X of the two-pass Pearson form
#pragma unroll
    for (int k = 0; k < TPT; ++k)
        if (t2 + k * NT < N) {
            const double a = (double)tv[k] - tmean, b = (double)fv[k] - fmean;
            q[0] += a * a;
            q[1] += b * b;
            q[2] += a * b;
        }
    wg_sum<NT, double, 3>(q, sm.redd);
    if (tid == 0) {
        const double ab = q[0] * q[1];
        const double v = ab > 0.0 ? q[2] / sqrt(ab) : 0.0;
        write_result(p, blk, ddx, ddy, ddz, (float)v);
    }
}

template <int B>
__global__ __launch_bounds__(256, FiltShape<B>::WAVES) void k_match_f32_filtered(Params p,
                                                                                 filt::Args fa) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Small sm;
    __shared__ filt::Small fs;
    match_one_filtered<B>(p, fa, p.first + xcd_block(blockIdx.x, gridDim.x), lds, sm, fs);
}

// ------------------------------------------------- large blocks of 12-bit data
//
// Block edges 11, 13 and 15 by 8-bit matrix instructions, exactly: a voxel less
// 2048 is 64 hi + lo with hi in [-32, 31] and lo in [0, 63], the cross term is
// 4096 hi hi + 64 (hi lo + lo hi) + lo lo, and each part sums exactly in int32.
// The ranking and the winner's NCC are the dot2 form's, on the same integers, so
// the results are its bits.
//
// A tile is 16 rows (window bases 4 apart in x and y, and z phases) by the 16
// (dx, dy) offsets of a 4x4 patch; a block plane is WideShape::NS chunks of 64 voxels, the
// block a Toeplitz operand.  A 13^3 block's operands need more registers than
// a wavefront has, so each of the four wavefronts holds a quarter of the block
// planes (operands in registers for the whole search), sweeps the window's
// planes with a ring of TW accumulators, and adds its share of each finished
// displacement plane to 64-bit sums in LDS (integers: the order does not
// matter).
//
// What bounds the dot2 form is its vector issue; here it is the latency of the
// phases before the sweep, and at many blocks the matrix cores (half their
// 8-bit rate at edge 13).  192x192x96 voxels, dot2 form / this, us: edge 11,
// 400 blocks, W = 3 33 / 17, W = 6 83 / 30, W = 12 473 / 162; edge 13, 400
// blocks, W = 6 134 / 35, 3000 blocks 716 / 186; edge 15, 250 blocks, W = 10
// 582 / 93.  The records are read after the sweep: held through it they spill
// (45 us at edge 13), as do the next plane's operands (37).
template <int B>
struct WideShape {
    static constexpr int GX = (B + 6) / 4;  // 4-voxel groups of a row that any offset touches
    static constexpr int RY = B + 3;        // rows
    // K order: rows of four groups, then (edge 15) the fifth group of four rows each
    static constexpr int XG = GX > 4 ? (RY + 3) / 4 : 0;
    static constexpr int NG = RY + XG, NS = (NG + 3) / 4;
    static constexpr int TW = (B + 3) / 4;  // block planes of a wavefront
    static constexpr int PT = 4 * GX;       // T table: row pitch, rows (three above), bytes
    static constexpr int TY = 3 + (XG ? 4 * XG : RY);
    static constexpr int COPY = B * TY * PT;
    static constexpr int WAVES = B == 15 ? 1 : 2;
};
constexpr int kWideTz = 13;     // displacement planes of a phase at most
constexpr int kWideKeep = 12;   // window chunks a thread holds while the operands are built
constexpr int kWideSlack = 8;   // window rows read past the last plane (against zeros)

typedef int int4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4u __attribute__((ext_vector_type(4), aligned(2)));
typedef int int4a __attribute__((ext_vector_type(4), aligned(4)));

struct WideSizes {
    int lo_off, x_off;  // LDS: hi bytes at 0, lo bytes, 64-bit sums
    int tz, lds;
};

// Displacement planes per phase: as few 16-row tiles and sweep steps as may be.
__host__ __device__ inline int wide_phase(int nxy, int dzn, int tw) {
    int best = 1, bc = INT_MAX;
    for (int tz = 1; tz <= (dzn < kWideTz ? dzn : kWideTz); ++tz) {
        const int tiles = (nxy * ((dzn + tz - 1) / tz) + 15) / 16;
        const int c = tiles * ((tz + 2 * tw - 2) / tw * tw + 2);  // + 2: the tile's ranking
        if (c < bc) {
            bc = c;
            best = tz;
        }
    }
    return best;
}

template <int B>
bool wide_sizes(int w, size_t limit, WideSizes *s) {
    using S = WideShape<B>;
    const int d = 2 * w + 1, nb = (d + 3) / 4;
    const int pitch = (4 * (nb - 1) + S::PT + 7) / 8 * 8, e = d + B - 1;
    const size_t half = ((size_t)e * e + kWideSlack) * pitch;
    s->lo_off = (int)half;
    s->x_off = (int)((std::max(2 * half, (size_t)8 * S::COPY) + 15) / 16 * 16);
    s->tz = wide_phase(nb * nb, d, S::TW);
    // (blocks at the volume's faces may take more planes per phase)
    s->lds = s->x_off + std::min(d, kWideTz) * 2048;
    return (size_t)s->lds <= limit;
}

template <int B>
__global__ __launch_bounds__(256, WideShape<B>::WAVES) void k_match_wide(Params p, WideSizes z) {
    using S = WideShape<B>;
    constexpr int H = (B - 1) / 2, N = B * B * B, NT = 256, TW = S::TW, NS = S::NS, PT = S::PT;
    constexpr int TPT = (N + NT - 1) / NT;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double s_red[12];
    __shared__ float s_key[4];
    __shared__ int s_idx[4];
    const int64_t blk = p.first + xcd_block(blockIdx.x, gridDim.x);
    const int tid = threadIdx.x, lane = tid & 63, grp = lane >> 4, n16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Geom g = make_geom(p, blk, H);
    if (!g.inside) {
        if (tid == 0) write_result(p, blk, 0, 0, 0, NAN);
        return;
    }
    const uint16_t *ref = static_cast<const uint16_t *>(p.ref);
    const uint16_t *flt = static_cast<const uint16_t *>(p.flt);
    const int nxy = p.nx * p.ny;
    const uint16_t *tb = ref + ((int64_t)(g.cz - H) * p.ny + (g.cy - H)) * p.nx + (g.cx - H);
    auto voxel = [&](int o) {  // offset of the block's voxel o
        const int oz = o / (B * B), oy = (o / B) % B, ox = o % B;
        return oz * nxy + oy * p.nx + ox;
    };

    // ---- the block's voxels and the window's first chunks, in flight together
    uint16_t tv[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) tv[k] = tb[voxel(min(tid + k * NT, N - 1))];
    const int nbx = (g.dx + 3) / 4, nby = (g.dy + 3) / 4;
    const int ey = g.dy + B - 1, ez = g.dz + B - 1;
    const int cpr = (4 * (nbx - 1) + PT + 7) / 8, pitch = 8 * cpr, plane = ey * pitch;
    const int nchunk = ez * ey * cpr;
    const int64_t w0 = ((int64_t)g.wz0 * p.ny + g.wy0) * p.nx + g.wx0;
    const uint16_t *wb = flt + w0;
    const int64_t end = (int64_t)nxy * p.nz - 1 - w0;  // the volume's last voxel
    const bool edge = (int64_t)(ez - 1) * nxy + (int64_t)(ey - 1) * p.nx + 8 * cpr - 1 > end;
    auto load = [&](int i) {  // 8 voxels of a window row (past the row's end: its neighbours)
        i = min(i, nchunk - 1);
        const int row = quotient(i, cpr), xc = i - row * cpr;
        const int zz = quotient(row, ey), yy = row - zz * ey;
        const int at = zz * nxy + yy * p.nx + 8 * xc;
        if (edge) {  // uniform: voxel by voxel, clamped to the volume's last
            uint4v v = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j / 2] |= (uint32_t)wb[min((int64_t)at + j, end)] << (16 * (j & 1));
            return v;
        }
        return __builtin_bit_cast(uint4v, *reinterpret_cast<const uint4u *>(wb + at));
    };
    uint4v wv[kWideKeep];
#pragma unroll
    for (int k = 0; k < kWideKeep; ++k)
        if (k * NT < nchunk) wv[k] = load(tid + k * NT);

    // ---- T tables: hi and lo bytes, four copies each (copy a moved right by a
    // columns), rows of zeros around each plane
    for (int i = tid; i < S::COPY / 2; i += NT)
        *reinterpret_cast<int4v *>(lds + 16 * i) = int4v{0, 0, 0, 0};
    __syncthreads();
    double st[2] = {0.0, 0.0};  // exact sums of T and T^2
#pragma unroll
    for (int k = 0; k < TPT; ++k)
        if (tid + k * NT < N) {
            const int o = tid + k * NT, oz = o / (B * B), oy = (o / B) % B, ox = o % B;
            const int v = tv[k];
            st[0] += (double)v;
            st[1] += (double)v * (double)v;
            unsigned char *d = lds + (oz * S::TY + oy + 3) * PT + ox;
            const int hi = (v - 2048) >> 6, lo = v & 63;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                d[a * S::COPY + a] = (unsigned char)hi;
                d[(4 + a) * S::COPY + a] = (unsigned char)lo;
            }
        }
    wg_sum<NT, double, 2>(st, s_red);  // its barriers publish the tables
    const long long st0 = (long long)st[0], st1 = (long long)st[1];
    if (N * st1 - st0 * st0 == 0) {  // flat block: all NCC are 0
        if (tid == 0) write_result(p, blk, g.lox, g.loy, g.loz, 0.0f);
        return;
    }
    const int tau0 = wave * TW;
    int4v bh[TW][NS], bl[TW][NS];
    {
        const int oa = n16 & 3, ob = n16 >> 2;
        const unsigned char *t0 = lds + oa * S::COPY;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int gi = 4 * s + grp;
            const bool main = gi < S::RY, real = gi < S::NG;
            const int row = main ? gi : 4 * (gi - S::RY), step = main ? 4 : PT;
            const int at = real ? (row - ob + 3) * PT + (main ? 0 : 16) : 0;
#pragma unroll
            for (int j = 0; j < TW; ++j) {
                const bool on = real && tau0 + j < B;
                const unsigned char *q = t0 + (on ? (tau0 + j) * S::TY * PT + at : 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int h = *reinterpret_cast<const int *>(q + e * step);
                    const int l = *reinterpret_cast<const int *>(q + 4 * S::COPY + e * step);
                    bh[j][s][e] = on ? h : 0;
                    bl[j][s][e] = on ? l : 0;
                }
            }
        }
    }
    __syncthreads();  // every wavefront's operands are built: the window takes their place

    // ---- the window's hi and lo bytes
    auto store = [&](int i, const uint4v &v) {
        if (i >= nchunk) return;
        uint32_t h[2], l[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t a = v[2 * e], b = v[2 * e + 1];
            l[e] = __builtin_amdgcn_perm(b, a, 0x06040200) & 0x3f3f3f3fu;
            // per byte (v >> 6) - 32 without a borrow between bytes
            const uint32_t q = __builtin_amdgcn_perm(b >> 6, a >> 6, 0x06040200);
            h[e] = ((q | 0x80808080u) - 0x20202020u) ^ 0x80808080u;
        }
        *reinterpret_cast<uint2 *>(lds + 8 * i) = make_uint2(h[0], h[1]);
        *reinterpret_cast<uint2 *>(lds + z.lo_off + 8 * i) = make_uint2(l[0], l[1]);
    };
#pragma unroll
    for (int k = 0; k < kWideKeep; ++k)
        if (k * NT < nchunk) store(tid + k * NT, wv[k]);
    for (int i = tid + kWideKeep * NT; i < nchunk; i += 4 * NT) {
        uint4v v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = load(i + k * NT);
#pragma unroll
        for (int k = 0; k < 4; ++k) store(i + k * NT, v[k]);
    }
    unsigned long long *xs = reinterpret_cast<unsigned long long *>(lds + z.x_off);
    const bool whole = g.dx == 2 * p.w + 1 && g.dy == 2 * p.w + 1 && g.dz == 2 * p.w + 1;
    const int tz = whole ? z.tz : wide_phase(nbx * nby, g.dz, TW);
    for (int i = tid; i < tz * 256; i += NT) xs[i] = 0;
    __syncthreads();

    // ---- sweep
    const int nb = nbx * nby, nrows = nb * ((g.dz + tz - 1) / tz);
    const int side = 2 * p.w + 1, plane_rec = p.oy * p.ox;
    const StatU16 *rec0 = static_cast<const StatU16 *>(p.stats) +
                          ((int64_t)g.wz0 * p.oy + g.wy0) * p.ox + g.wx0;
    const double dN = (double)N, tsum = (double)(st0 - 2048ll * N);
    int aoff[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int gi = 4 * s + grp;
        aoff[s] = gi < S::RY ? gi * pitch : gi < S::NG ? 4 * (gi - S::RY) * pitch + 16 : 0;
    }
    float bk = -INFINITY;
    int bi = INT_MAX;
    for (int r0 = 0; r0 < nrows; r0 += 16) {
        // the records of this thread's displacements: row tid / 16, offset tid % 16
        const int rr = r0 + (tid >> 4), rc = rr < nrows ? rr : 0;
        const int rph = quotient(rc, nb) , rxy = rc - rph * nb;
        const int ryi = quotient(rxy, nbx), rxi = rxy - ryi * nbx;
        const int dx = 4 * rxi + (tid & 3), dy = 4 * ryi + (tid >> 2 & 3), dz0 = rph * tz;
        int abase, alim;
        {
            const int r = r0 + n16 < nrows ? r0 + n16 : 0;
            const int ph = quotient(r, nb), xy = r - ph * nb;
            const int yi = quotient(xy, nbx), xi = xy - yi * nbx;
            abase = ph * tz * plane + 4 * yi * pitch + 4 * xi;
            alim = ez - 1 - ph * tz;
        }
        int4v hh[TW], hl[TW], ll[TW];
#pragma unroll
        for (int j = 0; j < TW; ++j) hh[j] = hl[j] = ll[j] = int4v{0, 0, 0, 0};
        auto read = [&](int at, auto sc, int4v &ah, int4v &al) __attribute__((always_inline)) {
            constexpr int s = decltype(sc)::value;
            const unsigned char *q = lds + at + aoff[s];
            if constexpr (4 * s + 3 < S::RY || S::XG == 0) {
                ah = *reinterpret_cast<const int4a *>(q);
                al = *reinterpret_cast<const int4a *>(q + z.lo_off);
            } else {
                const int step = 4 * s + grp < S::RY ? 4 : pitch;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    ah[e] = *reinterpret_cast<const int *>(q + e * step);
                    al[e] = *reinterpret_cast<const int *>(q + e * step + z.lo_off);
                }
            }
        };
        int4v ah, al;  // the window's chunk at hand; the next one is read early
        int at = abase + min(tau0, alim) * plane;
        read(at, std::integral_constant<int, 0>(), ah, al);
        for (int u0 = 0; u0 < tz + TW - 1; u0 += TW) {
            static_for<TW>([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                static_for<NS>([&](auto sc) __attribute__((always_inline)) {
                    constexpr int s = decltype(sc)::value;
                    int4v nh, nl;
                    if constexpr (s == NS - 1) at = abase + min(tau0 + u0 + u + 1, alim) * plane;
                    read(at, std::integral_constant<int, (s + 1) % NS>(), nh, nl);
#pragma unroll
                    for (int j = 0; j < TW; ++j) {
                        const int k = (u - j + TW) % TW;
                        hh[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, bh[j][s], hh[k], 0, 0, 0);
                        hl[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, bl[j][s], hl[k], 0, 0, 0);
                        ll[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, bl[j][s], ll[k], 0, 0, 0);
                        hl[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, bh[j][s], hl[k], 0, 0, 0);
                    }
                    ah = nh;
                    al = nl;
                });
                constexpr int f = (u + 1) % TW;  // the slot whose last block plane this was
                const int dzl = u0 + u - (TW - 1);
                if (dzl >= 0 && dzl < tz) {  // uniform
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        atomicAdd(&xs[(dzl * 16 + 4 * grp + i) * 16 + n16],
                                  (unsigned long long)((long long)hh[f][i] * 4096 +
                                                       (long long)(hl[f][i] * 64 + ll[f][i])));
                }
                hh[f] = hl[f] = ll[f] = int4v{0, 0, 0, 0};
            });
        }
        StatU16 rec[kWideTz];
        {
            const StatU16 *rb = rec0 + min(dy, g.dy - 1) * p.ox + min(dx, g.dx - 1);
#pragma unroll
            for (int k = 0; k < kWideTz; ++k) rec[k] = rb[(int64_t)min(dz0 + k, g.dz - 1) * plane_rec];
        }
        __syncthreads();  // the tile's cross terms
        const bool on = rr < nrows && dx < g.dx && dy < g.dy;
#pragma unroll
        for (int k = 0; k < kWideTz; ++k)
            if (k < tz) {
                const double x = (double)(long long)xs[k * 256 + tid];
                xs[k * 256 + tid] = 0;
                // the dot2 form's key
                const double cov = __builtin_fma(dN, x, -tsum * (double)rec[k].s);
                const float key = (float)cov * rec[k].r;
                const int idx = ((g.loz + dz0 + k + p.w) * side + (g.loy + dy + p.w)) * side +
                                (g.lox + dx + p.w);
                if (on && dz0 + k < g.dz) better(bk, bi, key, idx);
            }
        __syncthreads();  // cleared
    }
    wave_best(bk, bi);
    if (lane == 63) {
        s_key[wave] = bk;
        s_idx[wave] = bi;
    }
    __syncthreads();
    bk = s_key[0];
    bi = s_idx[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) better(bk, bi, s_key[i], s_idx[i]);
    if (bi == INT_MAX) {  // no key compares (a table of NaNs): report, never index
        if (tid == 0) write_result(p, blk, 0, 0, 0, NAN);
        return;
    }

    // ---- exact NCC at the winning displacement, from the volumes
    const int ddx = bi % side - p.w, ddy = (bi / side) % side - p.w, ddz = bi / (side * side) - p.w;
    const uint16_t *fb = flt + ((int64_t)(g.cz - H + ddz) * p.ny + (g.cy - H + ddy)) * p.nx +
                         (g.cx - H + ddx);
    uint16_t fv[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
        const int o = voxel(min(tid + k * NT, N - 1));
        tv[k] = tb[o];
        fv[k] = fb[o];
    }
    double sums[3] = {0.0, 0.0, 0.0};  // F, F^2, TF: exact
#pragma unroll
    for (int k = 0; k < TPT; ++k)
        if (tid + k * NT < N) {
            const double f = (double)fv[k], t = (double)tv[k];
            sums[0] += f;
            sums[1] += f * f;
            sums[2] += t * f;
        }
    wg_sum<NT, double, 3>(sums, s_red);
    if (tid == 0) {
        const long long f0 = (long long)sums[0];
        const long long vt = N * st1 - st0 * st0;
        const long long vf = N * (long long)sums[1] - f0 * f0;
        const long long cv = N * (long long)sums[2] - st0 * f0;
        const double v = (vt > 0 && vf > 0) ? (double)cv / sqrt((double)vt * (double)vf) : 0.0;
        write_result(p, blk, ddx, ddy, ddz, (float)v);
    }
}

// ------------------------------------------------------------ batched search
//
// Many parameter sets (block size, window, selection) over one volume pair in
// one persistent launch: workgroups stride a list of work items (the blocks
// of every set, the most expensive sets first) and switch to the compiled
// shape the set was planned with.  The shapes all run 256 threads.
#define BATCH_F32(X) X(0, 5, 4, 4, 0) X(1, 7, 4, 4, 0) X(2, 9, 4, 4, 0) X(3, 5, 3, 3, 0) \
    X(4, 7, 3, 3, 0) X(5, 9, 3, 3, 0)
#define BATCH_U16(X) X(0, 5, 4, 4, 0) X(1, 7, 3, 7, 1) X(2, 7, 4, 4, 0) X(3, 9, 4, 4, 0) \
    X(4, 9, 5, 5, 0) X(5, 5, 3, 3, 0)

template <typename Vox>
__global__ __launch_bounds__(256) void k_match_batch(const BatchSet *__restrict__ sets, int nsets,
                                                     int64_t nitems) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Small sm;
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        int s = 0;
        while (s + 1 < nsets && sets[s + 1].first_item <= it) ++s;
        const BatchSet &S = sets[s];
        Params p;
        p.ref = S.a.ref;
        p.flt = S.a.flt;
        p.nx = S.a.nx;
        p.ny = S.a.ny;
        p.nz = S.a.nz;
        p.centers = S.a.centers;
        p.n = S.a.n;
        p.first = 0;
        p.w = S.a.window;
        p.cz = S.cz;
        p.stats = S.a.stats;
        p.pv = S.a.pairs;
        p.ox = S.a.ox;
        p.oy = S.a.oy;
        p.disp = S.a.disp;
        p.ncc = S.a.ncc;
        p.conf = S.a.conf;
        p.surface = nullptr;
        const int64_t blk = it - S.first_item;
        if constexpr (sizeof(Vox) == 4) {
#define CASE_F32(ID, B, RX, RY, PF) \
    case ID: match_one<float, FMA, B, RX, RY, 256, PF>(p, blk, lds, sm, threadIdx.x); break;
            switch (S.variant) { BATCH_F32(CASE_F32) }
#undef CASE_F32
        } else {
#define CASE_U16(ID, B, RX, RY, PF) \
    case ID: match_one<uint16_t, DOT2, B, RX, RY, 256, PF>(p, blk, lds, sm, threadIdx.x); break;
            switch (S.variant) { BATCH_U16(CASE_U16) }
#undef CASE_U16
        }
        __syncthreads();  // the next item restages LDS
    }
}

// The float sets of one block edge behind the filter: a workgroup per item
// (one block of one set), the most expensive sets first.
template <int B>
__global__ __launch_bounds__(256, FiltShape<B>::WAVES) void k_match_batch_filtered(
    const BatchSet *__restrict__ sets, int nsets) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Small sm;
    __shared__ filt::Small fs;
    // the item's set: the last whose first item is not past it (64 at a time)
    const int64_t it = blockIdx.x;
    const int lane = threadIdx.x & 63;
    int s = -1;
    for (int s0 = 0; s0 < nsets; s0 += 64) {
        const bool at = s0 + lane < nsets && sets[s0 + lane].first_item <= it;
        s += __popcll(__ballot(at));
    }
    s = __builtin_amdgcn_readfirstlane(s);
    const BatchSet S = uniform_copy(sets[s]);
    Params p;
    p.ref = S.a.ref;
    p.flt = S.a.flt;
    p.nx = S.a.nx;
    p.ny = S.a.ny;
    p.nz = S.a.nz;
    p.centers = S.a.centers;
    p.n = S.a.n;
    p.first = 0;
    p.w = S.a.window;
    p.cz = S.cz;
    p.stats = S.a.stats;
    p.pv = nullptr;
    p.ox = S.a.ox;
    p.oy = S.a.oy;
    p.disp = S.a.disp;
    p.ncc = S.a.ncc;
    p.conf = S.a.conf;
    p.surface = nullptr;
    filt::Args fa;
    fa.z = S.filt;
    for (int i = 0; i < 3; ++i) {
        fa.b[i] = B;
        fa.w[i] = p.w;
    }
    fa.nx = p.nx;
    fa.ny = p.ny;
    fa.nz = p.nz;
    fa.ox = p.ox;
    fa.oy = p.oy;
    fa.flt = p.flt;
    fa.stats = p.stats;
    fa.nstat = (int64_t)p.ox * p.oy * (p.nz - B + 1);
    match_one_filtered<B>(p, fa, it - S.first_item, lds, sm, fs);
}

// ------------------------------------------------------------ dispatch

typedef void (*kernel_t)(Params);
typedef void (*kernel_wide_t)(Params, WideSizes);

struct Variant {
    nrr_dtype dtype;
    int arith, b, rx, ry, nt, pf;
    kernel_t fn;
};

#define V16D(B, RX, RY, NT, PF) \
    {NRR_U16, DOT2, B, RX, RY, NT, PF, k_match<uint16_t, DOT2, B, RX, RY, NT, PF>}
#define V16F(B, RX, RY, NT, PF) \
    {NRR_U16, FMA, B, RX, RY, NT, PF, k_match<uint16_t, FMA, B, RX, RY, NT, PF>}
#define V32F(B, RX, RY, NT, PF) \
    {NRR_F32, FMA, B, RX, RY, NT, PF, k_match<float, FMA, B, RX, RY, NT, PF>}

// Order matters only between equal-cost shapes (the first wins).  The cost
// model counts wavefront rounds, not occupancy, so shapes that lose on
// occupancy are left out rather than modelled: FMA 3x7 tiles at 448 threads
// (b = 7) ran 1.7x slower than at 256 on the 256x256x124 volume (W = 10) and
// 2.5x slower at W = 5.
const Variant kVariants[] = {
    V16D(3, 4, 4, 256, 0),  V16D(5, 4, 4, 256, 0),  V16D(5, 3, 7, 448, 0),
    V16D(7, 3, 7, 256, 1),  V16D(7, 3, 7, 256, 0),  V16D(7, 4, 4, 256, 0),
    V16D(7, 3, 5, 256, 0),  V16D(7, 5, 5, 256, 0),  V16D(9, 4, 4, 256, 0),
    V16D(9, 5, 5, 256, 0),  V16D(11, 3, 3, 256, 0), V16D(13, 3, 3, 256, 0),
    V16D(15, 2, 2, 256, 0), V16F(3, 4, 4, 256, 0),  V16F(5, 4, 4, 256, 0),
    V16F(5, 3, 7, 448, 0),  V16F(7, 4, 4, 256, 0),  V16F(7, 5, 5, 256, 0),
    V16F(7, 3, 7, 256, 0),
    V16F(9, 4, 4, 256, 0),  V16F(9, 5, 5, 256, 0),  V16F(11, 3, 3, 256, 0),
    V16F(13, 3, 3, 256, 0), V16F(15, 2, 2, 256, 0), V32F(3, 4, 4, 256, 0),
    V32F(5, 4, 4, 256, 0),  V32F(7, 4, 4, 256, 0),  V32F(7, 5, 5, 256, 0),
    V32F(7, 3, 7, 256, 0),  V32F(9, 5, 5, 256, 0),
    V32F(9, 4, 4, 256, 0),  V32F(11, 3, 3, 256, 0), V32F(13, 3, 3, 256, 0),
    V32F(15, 2, 2, 256, 0),
};

struct Plan {
    const Variant *v;
    int cz;
    size_t lds;
};

size_t t_table_bytes(const Variant &v) {
    const int bp = (v.b + 3) & ~3;
    const int planes = v.arith == DOT2 ? (v.b + 1) / 2 : v.b;
    return (size_t)planes * v.b * bp * 4;
}

size_t window_plane_bytes(const Variant &v, int w) {
    const int d = 2 * w + 1;
    const int px = (d + v.rx - 1) / v.rx * v.rx + v.b - 1;
    const int py = (d + v.ry - 1) / v.ry * v.ry + v.b - 1;
    if (v.arith == DOT2 || v.dtype == NRR_F32) {  // as the kernel's chunk-staged plane
        const int pl = (px + CW - 1) / CW * CW * py;
        return (size_t)(v.dtype == NRR_F32 ? pl + 1 : pl + (((pl / CW) & 1) ? 0 : CW)) * 4;
    }
    return ((size_t)px * py + ZPAD) * 4;
}

// Wavefront-rounds of one block's search with z-chunks of cz displacement
// planes (the last chunk takes the rest), plus half a round per extra chunk
// for its staging and barriers.  Idle wavefronts of a round skip the tiles.
double chunk_rounds(const Variant &v, int d, int cz) {
    const int per_dz = ((d + v.rx - 1) / v.rx) * ((d + v.ry - 1) / v.ry);
    double r = 0.0;
    for (int z0 = 0; z0 < d; z0 += cz) {
        const int tiles = per_dz * std::min(cz, d - z0);
        r += std::ceil(tiles / 64.0) + (z0 > 0 ? 0.5 : 0.0);
    }
    return r;
}

// z-chunk and LDS size: the whole window if it fits in `target` bytes (two
// workgroups per CU), else the largest balanced chunk of displacement planes
// that still fits in `target`, else the largest that fits in `limit`.
// (Balanced chunks keep the workgroup's LDS small: on the 256x256x124 search,
// 11 + 10 planes with three workgroups per CU beat 12 + 9 with two, although
// the latter packs the tiles into fewer wavefront-rounds.)
bool plan_variant(const Variant &v, int w, size_t limit, size_t target, Plan *out) {
    const int d = 2 * w + 1;
    const size_t fixed = t_table_bytes(v) + 2048;  // + static shared and slack
    const size_t pb = window_plane_bytes(v, w);
    if (fixed + (size_t)v.b * pb > limit) return false;
    int cz = d;
    if (fixed + (size_t)(cz + v.b - 1) * pb > target) {
        const size_t cap = fixed + (size_t)v.b * pb <= target ? target : limit;
        const long fit = (long)((cap - fixed) / pb) - (v.b - 1);
        cz = (int)(fit < d ? fit : d);
        const int nch = (d + cz - 1) / cz;
        cz = (d + nch - 1) / nch;
    }
    out->v = &v;
    out->cz = cz;
    out->lds = t_table_bytes(v) + (size_t)(cz + v.b - 1) * pb;
    return true;
}

// Cost model: padded displacement work over the workgroup's thread rounds.
double plan_cost(const Plan &pl, int w) {
    const Variant &v = *pl.v;
    const int d = 2 * w + 1;
    const double rounds = chunk_rounds(v, d, pl.cz) * 64.0 / v.nt;
    const double planes = v.arith == DOT2 ? (v.b + 1) / 2 : v.b;
    // instructions per tile: multiply-adds (dot2 issues at half the FMA rate)
    const double per = planes * v.rx * v.ry * v.b * v.b * (v.arith == DOT2 ? 2.0 : 1.0) +
                       planes * (v.rx + v.b - 1) * (v.ry + v.b - 1);
    return rounds * v.nt * per;
}

int arith_preference() {
    const char *e = getenv("NRR_ARITH");
    if (!e) return -1;
    if (!strcmp(e, "dot2")) return DOT2;
    if (!strcmp(e, "fma")) return FMA;
    if (!strcmp(e, "mfma")) return kArithMfma;
    return -1;
}

// Measurement overrides: NRR_TILE="rx,ry,nt[,pf]" restricts the shape and
// NRR_CZ=n caps the z-chunk (unknown or infeasible values are ignored).
bool shape_from_env(TileShape *sh) {
    *sh = TileShape{-1, 0, 0, 0, -1, 0};
    if (const char *e = getenv("NRR_TILE")) sscanf(e, "%d,%d,%d,%d", &sh->rx, &sh->ry, &sh->nt, &sh->pf);
    if (const char *e = getenv("NRR_CZ")) sh->cz = atoi(e);
    return sh->rx > 0 || sh->cz > 0;
}

// Shapes chosen by the tuner, per (dtype, block, window), for the process.
struct TunedEntry {
    nrr_dtype dtype;
    int b, w;
    TileShape sh;
    ShapeFrom from;
};
std::mutex g_tuned_mu;
std::vector<TunedEntry> g_tuned;

bool shape_matches(const Variant &v, const TileShape &sh) {
    if (sh.arith >= 0 && v.arith != sh.arith) return false;
    if (sh.rx > 0 && (v.rx != sh.rx || v.ry != sh.ry || v.nt != sh.nt)) return false;
    if (sh.pf >= 0 && v.pf != sh.pf) return false;
    return true;
}

// Best plan by the cost model among compiled shapes of (dtype, b); `force`
// (when given and feasible) restricts the shape and caps the z-chunk.
bool choose_with(nrr_dtype dtype, int b, int w, size_t limit, int arith, const TileShape *force,
                 Plan *best) {
    for (int pass = force ? 0 : 1; pass < 2; ++pass) {
        bool found = false;
        double bc = 0.0;
        for (const Variant &v : kVariants) {
            if (v.dtype != dtype || v.b != b) continue;
            if (arith >= 0 && v.arith != arith) continue;
            if (pass == 0 && !shape_matches(v, *force)) continue;
            Plan pl;
            if (!plan_variant(v, w, limit, limit / 2, &pl)) continue;
            if (pass == 0 && force->cz > 0 && force->cz < pl.cz) {  // a smaller chunk, as given
                pl.cz = force->cz;
                pl.lds = t_table_bytes(v) + (size_t)(pl.cz + v.b - 1) * window_plane_bytes(v, w);
            }
            const double c = plan_cost(pl, w);
            if (!found || c < bc) {
                *best = pl;
                bc = c;
                found = true;
            }
        }
        if (found) return true;
    }
    return false;
}

// Shape priority: an explicit one (the tuner's trials), the environment
// overrides, the tuned table, then the cost model.  12-bit volumes use the
// exact dot2 form when a shape has it (it measures faster than FMA on every
// shape tried); NRR_ARITH=dot2|fma restricts them to one form.
bool choose(nrr_dtype dtype, int b, int w, size_t limit, const TileShape *force, Plan *best) {
    TileShape sh;
    if (!force && shape_from_env(&sh)) force = &sh;
    if (!force && tuned_shape(dtype, b, w, &sh)) force = &sh;
    int pref = arith_preference();
    if (pref == kArithMfma) pref = -1;  // the matrix-core form does not serve this case
    if (pref < 0 && dtype == NRR_U16 && !(force && force->arith >= 0)) pref = DOT2;
    if (pref >= 0 && choose_with(dtype, b, w, limit, pref, force, best)) return true;
    return choose_with(dtype, b, w, limit, -1, force, best);
}

}  // namespace

size_t device_lds_limit() {
    static int cached_dev = -1;
    static size_t cached = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 65536;
    if (dev != cached_dev) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
            v <= 0)
            v = 65536;
        cached = (size_t)v;
        cached_dev = dev;
    }
    return cached;
}

const char *match_unsupported_reason(nrr_dtype dtype, int32_t block, int32_t window) {
    if (block > MAX_B) return "block edge above 15 is not built";
    if (window > 64) return "window above 64 is not supported";
    Plan pl;
    if (!choose(dtype, block, window, device_lds_limit(), nullptr, &pl))
        return "one window plane does not fit in LDS for this block size";
    return nullptr;
}


namespace {
#define ROW_F32(ID, B, RX, RY, PF) {NRR_F32, FMA, B, RX, RY, 256, PF, nullptr},
#define ROW_U16(ID, B, RX, RY, PF) {NRR_U16, DOT2, B, RX, RY, 256, PF, nullptr},
const Variant kBatchF32[] = {BATCH_F32(ROW_F32)};
const Variant kBatchU16[] = {BATCH_U16(ROW_U16)};
#undef ROW_F32
#undef ROW_U16
}  // namespace

bool plan_batch_set(nrr_dtype dtype, int32_t block, int32_t window, int32_t *variant,
                    int32_t *cz, size_t *lds, double *cost_per_block) {
    const Variant *tab = dtype == NRR_F32 ? kBatchF32 : kBatchU16;
    const int nv = dtype == NRR_F32 ? (int)(sizeof(kBatchF32) / sizeof(Variant))
                                    : (int)(sizeof(kBatchU16) / sizeof(Variant));
    const size_t limit = device_lds_limit();
    // a tuned shape for this (dtype, block, window) wins when it is compiled here
    TileShape ts;
    const bool tuned = tuned_shape(dtype, block, window, &ts);
    bool found = false;
    double best = 0.0;
    for (int pass = 0; pass < 2 && !found; ++pass)
        for (int i = 0; i < nv; ++i) {
            const Variant &v = tab[i];
            if (v.b != block) continue;
            if (pass == 0 && (!tuned || !shape_matches(v, ts))) continue;
            Plan pl;
            if (!plan_variant(v, window, limit, limit / 2, &pl)) continue;
            if (pass == 0 && ts.cz > 0 && ts.cz < pl.cz) {
                const int d = 2 * window + 1, nch = (d + ts.cz - 1) / ts.cz;
                pl.cz = (d + nch - 1) / nch;
                pl.lds = t_table_bytes(v) + (size_t)(pl.cz + v.b - 1) * window_plane_bytes(v, window);
            }
            const double c = plan_cost(pl, window);
            if (!found || c < best) {
                best = c;
                *variant = i;
                *cz = pl.cz;
                *lds = pl.lds;
                *cost_per_block = c;
                found = true;
            }
        }
    return found;
}

hipError_t launch_match_batch(nrr_dtype dtype, const BatchSet *sets, int32_t nsets,
                              int64_t nitems, size_t lds, hipStream_t stream) {
    if (nitems <= 0) return hipSuccess;
    const void *fn = dtype == NRR_F32 ? reinterpret_cast<const void *>(k_match_batch<float>)
                                      : reinterpret_cast<const void *>(k_match_batch<uint16_t>);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int per_cu = 0, dev = 0, cus = 0;
    e = dtype == NRR_F32
            ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_match_batch<float>, 256, lds)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_match_batch<uint16_t>, 256,
                                                           lds);
    if (e != hipSuccess) return e;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
        return e;
    const int64_t slots = (int64_t)(per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
    const unsigned grid = (unsigned)(nitems < slots ? nitems : slots);
    if (dtype == NRR_F32)
        hipLaunchKernelGGL(k_match_batch<float>, dim3(grid), dim3(256), lds, stream, sets, nsets,
                           nitems);
    else
        hipLaunchKernelGGL(k_match_batch<uint16_t>, dim3(grid), dim3(256), lds, stream, sets,
                           nsets, nitems);
    return hipGetLastError();
}

bool tuned_shape(nrr_dtype dtype, int32_t block, int32_t window, TileShape *sh) {
    std::lock_guard<std::mutex> lk(g_tuned_mu);
    for (const TunedEntry &t : g_tuned)
        if (t.dtype == dtype && t.b == block && t.w == window) {
            *sh = t.sh;
            return true;
        }
    return false;
}

void set_tuned_shape(nrr_dtype dtype, int32_t block, int32_t window, const TileShape &sh,
                     ShapeFrom from) {
    std::lock_guard<std::mutex> lk(g_tuned_mu);
    for (TunedEntry &t : g_tuned)
        if (t.dtype == dtype && t.b == block && t.w == window) {
            t.sh = sh;
            t.from = from;
            return;
        }
    g_tuned.push_back(TunedEntry{dtype, block, window, sh, from});
}

// Does the table's shape run in place of the matrix-core searches that take no
// shape?  A pinned one does; one the tuner timed against them where it was the
// faster, in the search it timed (a batch shares their launch among its sets).
static bool shape_replaces(nrr_dtype dtype, int32_t block, int32_t window, bool batched) {
    std::lock_guard<std::mutex> lk(g_tuned_mu);
    for (const TunedEntry &t : g_tuned)
        if (t.dtype == dtype && t.b == block && t.w == window)
            return t.from == ShapeFrom::Caller || (t.from == ShapeFrom::TunerFastest && !batched);
    return false;
}

void clear_tuned_shapes() {
    std::lock_guard<std::mutex> lk(g_tuned_mu);
    g_tuned.clear();
}

// The matrix-core form serves a launch when it is asked for (shape, then the
// NRR_ARITH override, then the tuned table) or, by default, whenever it can:
// 12-bit data, block edges 3-9, the whole window in LDS.
static bool wants_mfma(nrr_dtype dtype, int32_t block, int32_t window, const TileShape *shape) {
    if (!mfma_supported(dtype, block, window)) return false;
    if (shape) return shape->arith == kArithMfma;
    TileShape sh;
    if (shape_from_env(&sh)) return false;
    const int pref = arith_preference();
    if (pref >= 0) return pref == kArithMfma;
    if (tuned_shape(dtype, block, window, &sh)) return sh.arith == kArithMfma;
    return true;
}

// The 8-bit matrix-core search serves 12-bit blocks with edges 11 to 15 whose
// window fits in LDS beside its sums, by default: a shape or form asked for by
// the caller (a tuner's trial, a pinned shape, an environment override) runs as
// asked.  Voxel offsets from the window's corner are 32-bit.
static kernel_wide_t wide_plan(nrr_dtype dtype, const MatchArgs &a, const TileShape *shape,
                               WideSizes *z) {
    if (dtype != NRR_U16 || shape || a.block < 11 || a.block > 15) return nullptr;
    TileShape sh;
    if (shape_from_env(&sh) || arith_preference() >= 0 ||
        shape_replaces(dtype, a.block, a.window, false))
        return nullptr;
    const int e = 2 * a.window + a.block;
    if ((int64_t)a.nx * a.ny * e >= (1ll << 31) || (int64_t)e * e * (e / 8 + 2) >= (1 << 20))
        return nullptr;
    const size_t limit = device_lds_limit() - 256;
    switch (a.block) {
    case 11: return wide_sizes<11>(a.window, limit, z) ? k_match_wide<11> : nullptr;
    case 13: return wide_sizes<13>(a.window, limit, z) ? k_match_wide<13> : nullptr;
    default: return wide_sizes<15>(a.window, limit, z) ? k_match_wide<15> : nullptr;
    }
}

// The float search's launch behind the matrix-core filter.
struct FiltPlan {
    filt::Args fa;
    int cz;  // z-chunk of the FMA form, for the blocks the filter leaves
    size_t lds;
};

// The filter serves float volumes with block edges 5, 7 and 9 whose window
// fits in LDS, by default: a shape asked for by the caller (a tuner's trial, a
// pinned shape, an environment override) runs as the FMA form itself.  At
// edge 3 the FMA form's 27 products per displacement cost less than the
// bounds, as do small windows' products at the other edges, unless nearly all
// blocks are in flight at once (two or one a CU), where the FMA form's latency is
// the longer one.  The search alone, FMA form / filter in us, on
// tissue with noise (1,500-15,000 blocks) and on smooth blobs, whose broad
// peaks cost the filter a second look:
//   edge 5  W = 7 128 / 145, 133 / 178   W = 8 201 / 172, 202 / 216
//   edge 7  W = 5 167 / 174, 175 / 233   W = 6 238 / 176, 249 / 244
//   edge 9  W = 6 203 / 192, 237 / 304   W = 7 247 / 194, 284 / 302
// and in one round (64^3): edge 7, W = 5, 365 blocks 28.6 / 21.2, 28.6 / 32.5;
// edge 9, W = 5, 172 blocks 38.7 / 20.5, 38.6 / 37.5.  Sets of a batch share
// their launch, whatever their window.  Record and voxel offsets from the
// window's corner are 32-bit.
static bool filt_plan(nrr_dtype dtype, const MatchArgs &a, const TileShape *shape, FiltPlan *out,
                      bool batched = false) {
    if (dtype != NRR_F32 || shape || (a.block != 5 && a.block != 7 && a.block != 9)) return false;
    const bool few = a.n <= 512;
    const int least = a.block == 5 ? 8 : a.block == 7 ? (few ? 0 : 6) : (few ? 4 : 7);
    if (!batched && a.window < least) return false;
    TileShape sh;
    if (shape_from_env(&sh) || arith_preference() >= 0 ||
        shape_replaces(dtype, a.block, a.window, batched))
        return false;
    const int d = 2 * a.window + 1;
    if ((int64_t)a.nx * a.ny * 16 * (2 * d + 3 * a.block) >= (1ll << 31)) return false;
    const size_t limit = device_lds_limit(), fixed = sizeof(Small) + sizeof(filt::Small) + 64;
    const int32_t b[3] = {a.block, a.block, a.block}, w[3] = {a.window, a.window, a.window};
    if (limit < fixed || !filt::plan(b, w, limit - fixed, &out->fa.z)) return false;
    const Variant v{NRR_F32, FMA, a.block, 4, 4, 256, 0, nullptr};
    Plan fb;
    if (!plan_variant(v, a.window, limit, (size_t)out->fa.z.lds, &fb)) return false;
    out->cz = fb.cz;
    out->lds = std::max((size_t)out->fa.z.lds, fb.lds);
    for (int i = 0; i < 3; ++i) {
        out->fa.b[i] = b[i];
        out->fa.w[i] = w[i];
    }
    out->fa.nx = a.nx;
    out->fa.ny = a.ny;
    out->fa.nz = a.nz;
    out->fa.ox = a.ox;
    out->fa.oy = a.oy;
    out->fa.flt = a.flt;
    out->fa.stats = a.stats;
    out->fa.nstat = (int64_t)a.ox * a.oy * (a.nz - a.block + 1);
    return true;
}

bool plan_batch_filter(nrr_dtype dtype, const MatchArgs &a, FiltSizes *z, int32_t *cz,
                       size_t *lds) {
    FiltPlan fp;
    if (!filt_plan(dtype, a, nullptr, &fp, true)) return false;
    *z = fp.fa.z;
    *cz = fp.cz;
    *lds = fp.lds;
    return true;
}

hipError_t launch_match_batch_filtered(int32_t block, const BatchSet *sets, int32_t nsets,
                                       int64_t nitems, size_t lds, hipStream_t stream) {
    if (nitems <= 0) return hipSuccess;
    if (nitems >= (1ll << 31)) return hipErrorInvalidValue;
    const auto fn = block == 5 ? k_match_batch_filtered<5>
                    : block == 7 ? k_match_batch_filtered<7>
                                 : k_match_batch_filtered<9>;
    const hipError_t e = hipFuncSetAttribute(
        reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3((unsigned)nitems), dim3(256), lds, stream, sets, nsets);
    return hipGetLastError();
}

int match_shapes(nrr_dtype dtype, int32_t block, int32_t window, TileShape *out, int cap) {
    const size_t limit = device_lds_limit();
    const int d = 2 * window + 1;
    int n = 0;
    if (mfma_supported(dtype, block, window)) {
        if (n < cap) out[n] = TileShape{kArithMfma, 0, 0, 256, -1, 0};
        ++n;
    }
    for (const Variant &v : kVariants) {
        if (v.dtype != dtype || v.b != block) continue;
        Plan pl;
        if (!plan_variant(v, window, limit, limit / 2, &pl)) continue;
        // the planned z-chunk and the next two finer splits of the window
        int last = 0;
        for (int nch = (d + pl.cz - 1) / pl.cz; nch <= (d + pl.cz - 1) / pl.cz + 2; ++nch) {
            const int cz = (d + nch - 1) / nch;
            if (cz == last || cz < 1) continue;
            last = cz;
            if (n < cap) out[n] = TileShape{v.arith, v.rx, v.ry, v.nt, v.pf, cz};
            ++n;
        }
    }
    return n < cap ? n : cap;
}

bool match_takes_no_shape(nrr_dtype dtype, const MatchArgs &a) {
    FiltPlan fp;
    WideSizes z;
    return filt_plan(dtype, a, nullptr, &fp) || wide_plan(dtype, a, nullptr, &z);
}

bool match_reads_pairs(nrr_dtype dtype, const MatchArgs &a) {
    if (dtype != NRR_U16) return false;
    TileShape t;
    WideSizes z;
    return !wide_plan(dtype, a, nullptr, &z) &&
           (!match_plan(dtype, a, &t) || t.arith == DOT2);
}

bool match_plan(nrr_dtype dtype, const MatchArgs &a, TileShape *out) {
    if (mfma_fits(a) && wants_mfma(dtype, a.block, a.window, nullptr)) {
        *out = TileShape{kArithMfma, 0, 0, 256, -1, 0};
        return true;
    }
    Plan pl;
    if (!choose(dtype, a.block, a.window, device_lds_limit(), nullptr, &pl)) return false;
    *out = TileShape{pl.v->arith, pl.v->rx, pl.v->ry, pl.v->nt, pl.v->pf, pl.cz};
    return true;
}

bool shape_known(nrr_dtype dtype, int32_t block, int32_t window, const TileShape &sh) {
    if (sh.arith == kArithMfma) return mfma_supported(dtype, block, window);
    const size_t limit = device_lds_limit();
    for (const Variant &v : kVariants)
        if (v.dtype == dtype && v.b == block && v.arith == sh.arith && v.rx == sh.rx &&
            v.ry == sh.ry && v.nt == sh.nt && v.pf == sh.pf) {
            Plan pl;
            if (plan_variant(v, window, limit, limit / 2, &pl)) return true;
        }
    const Variant *tab = dtype == NRR_F32 ? kBatchF32 : kBatchU16;
    const int nv = dtype == NRR_F32 ? (int)(sizeof(kBatchF32) / sizeof(Variant))
                                    : (int)(sizeof(kBatchU16) / sizeof(Variant));
    for (int i = 0; i < nv; ++i)
        if (tab[i].b == block && tab[i].arith == sh.arith && tab[i].rx == sh.rx &&
            tab[i].ry == sh.ry && tab[i].nt == sh.nt && tab[i].pf == sh.pf)
            return true;
    return false;
}

bool batch_variant_shape(nrr_dtype dtype, int32_t variant, int32_t cz, TileShape *out) {
    const Variant *tab = dtype == NRR_F32 ? kBatchF32 : kBatchU16;
    const int nv = dtype == NRR_F32 ? (int)(sizeof(kBatchF32) / sizeof(Variant))
                                    : (int)(sizeof(kBatchU16) / sizeof(Variant));
    if (variant < 0 || variant >= nv) return false;
    const Variant &v = tab[variant];
    *out = TileShape{v.arith, v.rx, v.ry, v.nt, v.pf, cz};
    return true;
}

hipError_t launch_match(nrr_dtype dtype, const MatchArgs &a, hipStream_t stream,
                        const TileShape *shape) {
    if (mfma_fits(a) && wants_mfma(dtype, a.block, a.window, shape))
        return launch_match_mfma(a, stream);
    Plan pl;
    FiltPlan fp;
    WideSizes wz;
    const bool filtered = filt_plan(dtype, a, shape, &fp);
    const kernel_wide_t wide = wide_plan(dtype, a, shape, &wz);
    if (!filtered && !wide && !choose(dtype, a.block, a.window, device_lds_limit(), shape, &pl))
        return hipErrorInvalidValue;
    const auto ffn = a.block == 5 ? k_match_f32_filtered<5>
                     : a.block == 7 ? k_match_f32_filtered<7>
                                    : k_match_f32_filtered<9>;
    const void *fn = filtered ? reinterpret_cast<const void *>(ffn)
                     : wide   ? reinterpret_cast<const void *>(wide)
                              : reinterpret_cast<const void *>(pl.v->fn);
    const size_t lds = filtered ? fp.lds : wide ? (size_t)wz.lds : pl.lds;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
        hipSuccess)
        return hipGetLastError();
    Params p;
    p.ref = a.ref;
    p.flt = a.flt;
    p.nx = a.nx;
    p.ny = a.ny;
    p.nz = a.nz;
    p.centers = a.centers;
    p.n = a.n;
    p.w = a.window;
    p.cz = filtered ? fp.cz : wide ? 0 : pl.cz;
    p.stats = a.stats;
    p.pv = a.pairs;
    p.ox = a.ox;
    p.oy = a.oy;
    p.disp = a.disp;
    p.ncc = a.ncc;
    p.conf = a.conf;
    p.surface = nullptr;
    const int64_t chunk = 1ll << 30;
    for (int64_t first = 0; first < a.n; first += chunk) {
        p.first = first;
        const int64_t cnt = a.n - first < chunk ? a.n - first : chunk;
        if (filtered)
            hipLaunchKernelGGL(ffn, dim3((unsigned)cnt), dim3(256), lds, stream, p, fp.fa);
        else if (wide)
            hipLaunchKernelGGL(wide, dim3((unsigned)cnt), dim3(256), lds, stream, p, wz);
        else
            hipLaunchKernelGGL(pl.v->fn, dim3((unsigned)cnt), dim3(pl.v->nt), lds, stream, p);
    }
    return hipGetLastError();
}

namespace {
__global__ void k_fill(float *p, int64_t n, float v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
}  // namespace

hipError_t launch_fill(float *p, int64_t n, float v, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

namespace {
// Surface-writing instantiations: one shape per (dtype, form, block edge).
#define S16D(B, RX, RY, NT, PF) \
    {NRR_U16, DOT2, B, RX, RY, NT, PF, k_match_surf<uint16_t, DOT2, B, RX, RY, NT, PF>}
#define S16F(B, RX, RY, NT, PF) \
    {NRR_U16, FMA, B, RX, RY, NT, PF, k_match_surf<uint16_t, FMA, B, RX, RY, NT, PF>}
#define S32F(B, RX, RY, NT, PF) \
    {NRR_F32, FMA, B, RX, RY, NT, PF, k_match_surf<float, FMA, B, RX, RY, NT, PF>}
const Variant kSurfVariants[] = {
    S16D(3, 4, 4, 256, 0), S16D(5, 4, 4, 256, 0), S16D(7, 3, 7, 256, 1), S16D(9, 5, 5, 256, 0),
    S16D(11, 3, 3, 256, 0), S16D(13, 3, 3, 256, 0), S16D(15, 2, 2, 256, 0),
    S16F(7, 4, 4, 256, 0),  S32F(3, 4, 4, 256, 0),  S32F(5, 4, 4, 256, 0),
    S32F(7, 4, 4, 256, 0),  S32F(9, 5, 5, 256, 0),
};
#undef S16D
#undef S16F
#undef S32F
}  // namespace

hipError_t launch_match_surface(nrr_dtype dtype, int32_t arith, const MatchArgs &a,
                                float *surface, hipStream_t stream) {
    if (arith == kArithMfma) {
        if (!mfma_supported(dtype, a.block, a.window) || !mfma_fits(a))
            return hipErrorNotSupported;
        return launch_match_mfma(a, stream, surface);
    }
    const size_t limit = device_lds_limit();
    for (const Variant &v : kSurfVariants) {
        if (v.dtype != dtype || v.arith != arith || v.b != a.block) continue;
        Plan pl;
        if (!plan_variant(v, a.window, limit, limit / 2, &pl)) continue;
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(v.fn),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)pl.lds) != hipSuccess)
            return hipGetLastError();
        Params p;
        p.ref = a.ref;
        p.flt = a.flt;
        p.nx = a.nx;
        p.ny = a.ny;
        p.nz = a.nz;
        p.centers = a.centers;
        p.n = a.n;
        p.w = a.window;
        p.cz = pl.cz;
        p.stats = a.stats;
        p.pv = a.pairs;
        p.ox = a.ox;
        p.oy = a.oy;
        p.disp = a.disp;
        p.ncc = a.ncc;
        p.conf = a.conf;
        p.surface = surface;
        const int64_t chunk = 1ll << 30;
        for (int64_t first = 0; first < a.n; first += chunk) {
            p.first = first;
            const int64_t cnt = a.n - first < chunk ? a.n - first : chunk;
            hipLaunchKernelGGL(v.fn, dim3((unsigned)cnt), dim3(v.nt), pl.lds, stream, p);
        }
        return hipGetLastError();
    }
    return hipErrorNotSupported;
}

}  // namespace nrr
