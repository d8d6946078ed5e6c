// Per-voxel statistics of every block (bx x by x bz, cubic for the plain
// search) of the intra-operative volume.
//
// The NCC of the paper's similarity equation needs, for each displaced block
// F, its mean and its spread sum (F - Fbar)^2.  Those depend only on the
// block's position, not on which pre-operative block is being matched, so
// they are computed once per call for every possible block origin (a 3-D box
// filter of F and F^2) instead of once per (block, displacement) pair.
//
//   u16: s = sum (F - 2048) exact in int32, q = sum (F - 2048)^2 exact in
//        uint64, r = 1/sqrt(N q - s^2) as float (0 when the block is flat,
//        i.e. N q == s^2 exactly).
//   f32: s = sum F, q = sum F^2 in FP64, r = 1/sqrt(N q - s^2) in FP64;
//        the block counts as flat when N q - s^2 <= 1e-12 * N q (FP64 cannot
//        resolve a smaller relative spread from these sums).
//
// Layout of the outputs: dense [Oz][Oy][Ox] with O = dims - block + 1 (index =
// lowest corner of the block).
//
// 12-bit data, by voxel columns: a wavefront owns 64 consecutive voxel
// columns (x) over the rows of 8 origin rows (y) and slides along a run of
// origin planes.  Each lane keeps, per row, the sums over the block's current
// bz planes of F - 2048 and of its square (exact integers: each step adds the
// plane entering and subtracts the plane leaving, read again), forms the
// by-row sums in registers and the bx-column sums across lanes through LDS.
// Wavefronts share no data, so the kernel has no barrier.  The plane-pair
// volume that the search reads is written by a separate pass.
//
// Float data, by tiles: a workgroup owns a 64 x 4 tile of (x, y) origins and
// a run of zc origin planes; each input plane is staged in LDS (fetched two
// planes ahead) and summed along x (sliding windows over 4-wide segments)
// then along y; the per-plane sums of the last bz planes sit in a small LDS
// ring and the block sums are re-added from it (no rounding drifts along
// the volume).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "nrr_internal.h"
#include "stats_cols.h"
#include "wave64.h"

namespace nrr {
namespace {

constexpr int TX = 64, TY = 4, ZC = 32, MAXB = 15, SEG = 4;  // ZC: most origin planes per run
constexpr int PW = TX + MAXB - 1, PH = TY + MAXB - 1;
constexpr int PATCH = PH * PW;
constexpr int PER_MAX = (PATCH + 255) / 256;  // patch elements staged per thread

// Workgroup barrier for LDS traffic only.  __syncthreads also orders global
// memory, which on this architecture means waiting for every load in flight
// (loads and stores share one counter), including the planes fetched ahead;
// this kernel's global stores are read by no other thread of the launch.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Body of the float statistics kernel.  V: staged voxel type, A/AQ: row and
// plane sums of F and F^2, AS/AQQ: block sums, re-added from the ring of the
// last bz plane sums.  Global loads run two planes ahead of the plane being
// summed.  B > 0: a cubic block of that edge, its sums unrolled and its ring in
// registers (the planes of a run are stepped through in unrolled rounds of 2 B,
// so that slots and load buffers are constants); 0: any block, the ring in LDS.
// The order of every sum is the same.  What bounds it is the latency of the LDS
// reads between a plane's two barriers: with the ring (half the LDS and its
// traffic) out of LDS twice the workgroups share a CU.
template <int B, typename V, typename A, typename AQ, typename AS, typename AQQ, typename Src,
          typename Conv, typename Emit>
__device__ inline void stats_body(const Src *__restrict__ flt, int nx, int ny, int nz, int bx_,
                                  int by_, int bz_, int ox, int oy, int oz, int zc, int tile_x,
                                  int tile_y, int run, V *patch /*[2][PATCH]*/, A *rs, AQ *rq,
                                  A *ringP, AQ *ringQ, Conv conv, Emit emit) {
    const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;  // output (tx, ty)
    const int bx = B > 0 ? B : bx_, by = B > 0 ? B : by_, bz = B > 0 ? B : bz_;
    constexpr int PER = B > 0 ? ((TY + B - 1) * (TX + B - 1) + 255) / 256 : PER_MAX;
    [[maybe_unused]] A regP[B > 0 ? B : 1];
    [[maybe_unused]] AQ regQ[B > 0 ? B : 1];
    const int x0 = tile_x * TX, y0 = tile_y * TY, z0 = run * zc;
    const int ph = TY + by - 1, pw = TX + bx - 1;
    const int zend = min(z0 + zc + bz - 1, nz);  // input planes [z0, zend)
    // this thread's patch elements: fixed offsets inside a plane
    int goff[PER];
    bool gok[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = tid + 256 * k, r = e / pw, c = e - r * pw;
        gok[k] = e < ph * pw && x0 + c < nx && y0 + r < ny;
        goff[k] = r * nx + c;
    }
    const int64_t pstride = (int64_t)ny * nx;
    const Src *pbase = flt + (int64_t)y0 * nx + x0;
    // Loads are issued unconditionally (elements outside the volume or past
    // the run read the tile's first voxel of a plane inside the volume) and
    // kept raw; the mask and the conversion are applied when the values go
    // to LDS a plane later, so no wait follows a load in the step it is
    // issued in.
    struct Raw {
        Src v[PER];
        uint32_t ok;  // bit k: element k is inside the volume and the run
    };
    auto fetch = [&](Raw &r, int zi) {
        const Src *pl = pbase + (int64_t)min(zi, nz - 1) * pstride;
        r.ok = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const bool ok = gok[k] && zi < zend;
            r.ok |= (uint32_t)ok << k;
            r.v[k] = pl[ok ? goff[k] : 0];
        }
    };
    auto value = [&](const Raw &r, int k) { return ((r.ok >> k) & 1) ? conv(r.v[k]) : V(0); };
    Raw r1, r2;
    fetch(r1, z0);
#pragma unroll
    for (int k = 0; k < PER; ++k) patch[tid + 256 * k] = value(r1, k);
    fetch(r1, z0 + 1);
    lds_barrier();
    const int nseg = ph * (TX / SEG);
    // one plane step; rn holds plane zi + 1 (fetched a step earlier), rf
    // receives plane zi + 2.  The loop runs two steps per iteration with the
    // buffers' roles swapped, so no register copy waits on a load in flight.
    auto step = [&](int zi, Raw &rn, Raw &rf, auto slot_c) {
        constexpr int SLOT = decltype(slot_c)::value;  // of this plane (B > 0)
        const int cur = (zi - z0) & 1;
        const V *pc = patch + cur * PATCH;
        fetch(rf, zi + 2);
        // sums along x: SEG outputs per segment by a sliding window
        for (int sg = tid; sg < nseg; sg += 256) {
            const int r = sg / (TX / SEG), xs = (sg % (TX / SEG)) * SEG;
            const V *row = pc + r * pw + xs;
            A sv = 0;
            AQ qv = 0;
            auto add = [&](int k) {
                const A v = (A)row[k];
                sv += v;
                qv += (AQ)(v * v);
            };
            if constexpr (B > 0)
                static_for<B>(add);
            else
                for (int k = 0; k < bx; ++k) add(k);
            rs[r * TX + xs] = sv;
            rq[r * TX + xs] = qv;
#pragma unroll
            for (int u = 1; u < SEG; ++u) {
                const A vin = (A)row[u + bx - 1], vout = (A)row[u - 1];
                sv += vin - vout;
                qv += (AQ)(vin * vin) - (AQ)(vout * vout);
                rs[r * TX + xs + u] = sv;
                rq[r * TX + xs + u] = qv;
            }
        }
        lds_barrier();
        A P = 0;  // then along y
        AQ Q = 0;
        auto add = [&](int k) {
            P += rs[(ty + k) * TX + tx];
            Q += rq[(ty + k) * TX + tx];
        };
        if constexpr (B > 0)
            static_for<B>(add);
        else
            for (int k = 0; k < by; ++k) add(k);
        if constexpr (B > 0) {
            regP[SLOT] = P;
            regQ[SLOT] = Q;
        } else {
            const int slot = (zi - z0) % bz;
            ringP[slot * 256 + tid] = P;
            ringQ[slot * 256 + tid] = Q;
        }
        if (zi - z0 >= bz - 1) {  // the last bz plane sums give the block sums
            const int z = zi - bz + 1, x = x0 + tx, y = y0 + ty;
            if (x < ox && y < oy && z < oz) {
                AS sb = 0;
                AQQ qb = 0;
                if constexpr (B > 0) {
#pragma unroll
                    for (int k = 0; k < B; ++k) {
                        sb += (AS)regP[k];
                        qb += (AQQ)regQ[k];
                    }
                } else {
                    for (int k = 0; k < bz; ++k) {
                        sb += (AS)ringP[k * 256 + tid];
                        qb += (AQQ)ringQ[k * 256 + tid];
                    }
                }
                emit(((int64_t)z * oy + y) * ox + x, sb, qb);
            }
        }
        V *pn = patch + (cur ^ 1) * PATCH;
#pragma unroll
        for (int k = 0; k < PER; ++k) pn[tid + 256 * k] = value(rn, k);
        lds_barrier();
    };
    if constexpr (B > 0) {
        for (int zb = z0; zb < zend; zb += 2 * B)
            static_for<2 * B>([&](auto u) {
                constexpr int U = decltype(u)::value;
                const std::integral_constant<int, U % B> slot;
                if (zb + U < zend) {  // uniform
                    if constexpr (U % 2 == 0)
                        step(zb + U, r1, r2, slot);
                    else
                        step(zb + U, r2, r1, slot);
                }
            });
    } else {
        const std::integral_constant<int, 0> none;
        for (int zi = z0; zi < zend; zi += 2) {
            step(zi, r1, r2, none);
            if (zi + 1 < zend) step(zi + 1, r2, r1, none);
        }
    }
}

// 12-bit statistics by voxel columns (see the top of the file): four
// independent wavefronts per workgroup.
template <int BY, int BC>
__global__ __launch_bounds__(256) void k_stats_u16(const uint16_t *__restrict__ flt, int nx,
                                                   int ny, int nz, int bx_rt, int bz_rt, int ox,
                                                   int oy, int oz, int zc,
                                                   StatU16 *__restrict__ out) {
    __shared__ uint2 xch[4][SC_RY][SC_LW];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    stats_cols_wave<BY, BC>(flt, nx, ny, nz, bx_rt, bz_rt, ox, oy, oz, zc, out, blockIdx.x,
                            blockIdx.y * 4 + w, blockIdx.z, xch[w]);
}

// A float record from the block's sums.
__device__ inline StatF32 record_f32(double n, double S, double QQ) {
    const double nq = n * QQ;
    const double var = nq - S * S;
    StatF32 rec;
    rec.s = S;
    rec.r = var > 1e-12 * nq ? 1.0 / sqrt(var) : 0.0;
    return rec;
}

// LDS of a float statistics workgroup but the ring: arrays of their own, so that
// the compiler sees that the row sums' stores do not touch the patch (in one struct
// every step waited for them: 281x163x140, 7x9x3 100 us against 92; 256x256x124,
// edge 7 60 against 54, edge 13 105 against 86).
#define STATS_F32_LDS                        \
    __shared__ float patch[2 * PATCH + 256]; \
    __shared__ double rs[PH * TX], rq[PH * TX]

template <int B>
__device__ __attribute__((always_inline)) inline void stats_f32_tile(
    const float *__restrict__ flt, int nx, int ny, int nz, int bx, int by, int bz, int ox, int oy,
    int oz, int zc, int tile_x, int tile_y, int run, float *patch, double *rs, double *rq,
    double *ring, StatF32 *__restrict__ out) {
    const double n = (double)bx * by * bz;
    stats_body<B, float, double, double, double, double>(
        flt, nx, ny, nz, bx, by, bz, ox, oy, oz, zc, tile_x, tile_y, run, patch, rs, rq, ring,
        ring + (size_t)bz * 256, [](float v) { return v; },
        [&](int64_t o, double S, double QQ) { out[o] = record_f32(n, S, QQ); });
}

template <int B>
__global__ __launch_bounds__(256) void k_stats_f32(const float *__restrict__ flt, int nx, int ny,
                                                   int nz, int bx, int by, int bz, int ox, int oy,
                                                   int oz, int zc, StatF32 *__restrict__ out) {
    STATS_F32_LDS;
    extern __shared__ __align__(16) double dyn_f32[];
    stats_f32_tile<B>(flt, nx, ny, nz, bx, by, bz, ox, oy, oz, zc, blockIdx.x, blockIdx.y,
                      blockIdx.z, patch, rs, rq, dyn_f32, out);
}

// One cubic block edge's share of a several-edge float statistics launch.
struct StatsF32Job {
    int b, ox, oy, oz, zc;
    int tiles_x, tiles_y, z_first;  // its tiles, and its first grid z (its runs follow)
    StatF32 *out;
};
struct StatsF32Jobs {
    StatsF32Job job[kStatsJobs];
    int n;
};

// Float statistics of several block edges over one volume in one launch:
// grid z holds each edge's runs in turn, and a workgroup past its edge's x
// or y tiles leaves at once.  The same body and records as k_stats_f32.
__global__ __launch_bounds__(256) void k_stats_f32_multi(const float *__restrict__ flt, int nx,
                                                         int ny, int nz, StatsF32Jobs J) {
    STATS_F32_LDS;
    extern __shared__ __align__(16) double dyn_f32m[];
    StatsF32Job jb = J.job[0];
#pragma unroll
    for (int i = 1; i < kStatsJobs; ++i)  // constant indices: the table stays in kernel arguments
        if (i < J.n && (int)blockIdx.z >= J.job[i].z_first) jb = J.job[i];
    if ((int)blockIdx.x >= jb.tiles_x || (int)blockIdx.y >= jb.tiles_y) return;
    switch (jb.b) {
#define NRR_JOB(B)                                                                              \
    case B:                                                                                     \
        stats_f32_tile<B>(flt, nx, ny, nz, B, B, B, jb.ox, jb.oy, jb.oz, jb.zc, blockIdx.x,     \
                          blockIdx.y, (int)blockIdx.z - jb.z_first, patch, rs, rq, dyn_f32m,    \
                          jb.out);                                                              \
        break;
        NRR_JOB(5)
        NRR_JOB(7)
        NRR_JOB(9)
#undef NRR_JOB
    default:
        stats_f32_tile<0>(flt, nx, ny, nz, jb.b, jb.b, jb.b, jb.ox, jb.oy, jb.oz, jb.zc,
                          blockIdx.x, blockIdx.y, (int)blockIdx.z - jb.z_first, patch, rs, rq,
                          dyn_f32m, jb.out);
    }
}

// Plane-pair copy of a 12-bit volume: one 4-byte word per voxel holding the
// voxel and the one a plane above, both offset by -2048 into int16 (the next
// plane's half is 0 on the last plane).  Four consecutive voxels per thread.
__global__ __launch_bounds__(256) void k_pair_volume(const uint16_t *__restrict__ flt,
                                                     int64_t nvox, int64_t pstride,
                                                     uint32_t *__restrict__ out) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= nvox) return;
    auto word = [&](int64_t j) {
        const uint32_t lo = (uint16_t)((int)flt[j] - 2048);
        const uint32_t hi = j + pstride < nvox ? (uint16_t)((int)flt[j + pstride] - 2048) : 0u;
        return lo | hi << 16;
    };
    if (i + 4 <= nvox) {
        uint4 w;
        w.x = word(i);
        w.y = word(i + 1);
        w.z = word(i + 2);
        w.w = word(i + 3);
        *reinterpret_cast<uint4 *>(out + i) = w;
    } else {
        for (int64_t j = i; j < nvox; ++j) out[j] = word(j);
    }
}

// Directional confidence (the FEM update's confidence matrix S, no formula in
// the paper): S = conf * J / trace(J) with J the block's intensity structure
// tensor, sum over its voxels of g g^T, g by central differences of `ref`
// (one-sided on the volume's border planes).  One wavefront per block, FP64
// sums (exact for 12-bit data), S as (xx, yy, zz, xy, xz, yz).  What bounds it
// was the L1 requests of six neighbours a voxel; a block that touches no face
// is staged with its halo in LDS, four voxels a load, CU loads of a lane in
// flight together, the sums cross lanes by register moves, and neighbouring
// blocks run on one XCD, whose L2 then holds the lines they share.  256x256x124
// 12-bit voxels: 5508 blocks of edge 7 20.9 -> 15.3 us (17.1 without the XCD
// order), 5000 of edge 13 65 -> 45.
constexpr int CU = 4;
// The staged blocks of a workgroup take at most this much: five workgroups per
// CU (12-bit edges to 13, float to 9).  Above, the plain form is the faster one:
// float edge 13 staged 75 us, plain 68.
constexpr size_t kConfLds = 32 << 10;

// LDS row pitch of a staged block with its halo (whole 4-voxel loads).
__host__ __device__ inline int conf_pitch(int b) { return (b + 2 + 3) / 4 * 4; }

template <typename Vox>
__global__ __launch_bounds__(256) void k_structure_conf(const Vox *__restrict__ ref, int nx, int ny,
                                                        int nz, const int32_t *__restrict__ centers,
                                                        int64_t n, int b, bool staged,
                                                        const float *__restrict__ conf,
                                                        float *__restrict__ out) {
    typedef Vox Aligned4 __attribute__((ext_vector_type(4)));
    typedef Vox Chunk4 __attribute__((ext_vector_type(4), aligned(sizeof(Vox))));
    extern __shared__ __align__(16) unsigned char conf_lds[];  // a region per wavefront
    // consecutive blocks (which share lines of the volume) on one XCD
    const unsigned part = gridDim.x / 8, rest = gridDim.x % 8, xcd = blockIdx.x % 8;
    const unsigned wg = xcd * part + min(xcd, rest) + blockIdx.x / 8;
    const int64_t k = (int64_t)wg * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (k >= n) return;  // whole wavefront leaves together
    const int h = (b - 1) / 2;
    const int cx = centers[3 * k], cy = centers[3 * k + 1], cz = centers[3 * k + 2];
    const bool inside = cx - h >= 0 && cy - h >= 0 && cz - h >= 0 && cx + h < nx && cy + h < ny &&
                        cz + h < nz;
    double j[6] = {0, 0, 0, 0, 0, 0};
    if (inside) {
        const int64_t sy = nx, sz = (int64_t)nx * ny;
        auto at = [&](int x, int y, int z) {
            return (double)ref[(int64_t)z * sz + (int64_t)y * sy + x];
        };
        auto diff = [&](int x, int y, int z, int dx, int dy, int dz, int p, int len) {
            if (len == 1) return 0.0;
            if (p == 0) return at(x + dx, y + dy, z + dz) - at(x, y, z);
            if (p == len - 1) return at(x, y, z) - at(x - dx, y - dy, z - dz);
            return 0.5 * (at(x + dx, y + dy, z + dz) - at(x - dx, y - dy, z - dz));
        };
        const int nb = b * b * b, bb = b * b;
        auto add = [&](double gx, double gy, double gz) {
            j[0] += gx * gx;
            j[1] += gy * gy;
            j[2] += gz * gz;
            j[3] += gx * gy;
            j[4] += gx * gz;
            j[5] += gy * gz;
        };
        const int e = b + 2, pitch = conf_pitch(b), plane = e * pitch;
        const int64_t corner = (int64_t)(cz - h - 1) * sz + (int64_t)(cy - h - 1) * sy + (cx - h - 1);
        if (staged && cx - h > 0 && cy - h > 0 && cz - h > 0 && cx + h < nx - 1 &&
            cy + h < ny - 1 && cz + h < nz - 1 &&
            corner + (e - 1) * (sz + sy) + pitch <= sz * nz) {  // uniform: no voxel on a face
            Vox *blk = reinterpret_cast<Vox *>(conf_lds) + (threadIdx.x >> 6) * e * plane;
            const int cpr = pitch / 4, nc = e * e * cpr;
            for (int i0 = lane; i0 - lane < nc; i0 += 64 * CU) {
                Chunk4 v[CU];
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    const int i = min(i0 + 64 * u, nc - 1);
                    const int row = quotient(i, cpr), z = quotient(row, e), y = row - z * e;
                    v[u] = *reinterpret_cast<const Chunk4 *>(ref + corner + z * sz + y * sy +
                                                             4 * (i - row * cpr));
                }
#pragma unroll
                for (int u = 0; u < CU; ++u)
                    if (i0 + 64 * u < nc) *reinterpret_cast<Aligned4 *>(blk + 4 * (i0 + 64 * u)) = v[u];
            }
            wave_lds_sync();
            for (int o = lane; o < nb; o += 64) {
                const int z = quotient(o, bb), r = o - z * bb, y = quotient(r, b);
                const Vox *q = blk + (z + 1) * plane + (y + 1) * pitch + (r - y * b + 1);
                add(0.5 * ((double)q[1] - (double)q[-1]),
                    0.5 * ((double)q[pitch] - (double)q[-pitch]),
                    0.5 * ((double)q[plane] - (double)q[-plane]));
            }
        } else {
            for (int o = lane; o < nb; o += 64) {
                const int x = cx - h + o % b, y = cy - h + (o / b) % b, z = cz - h + o / bb;
                add(diff(x, y, z, 1, 0, 0, x, nx), diff(x, y, z, 0, 1, 0, y, ny),
                    diff(x, y, z, 0, 0, 1, z, nz));
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) j[e] = wave_xor_sum(j[e]);
    if (lane < 6) {
        const double tr = j[0] + j[1] + j[2];
        double v = 0.0;
#pragma unroll
        for (int e = 0; e < 6; ++e)
            if (e == lane) v = j[e];
        out[6 * k + lane] = tr > 0.0 ? (float)((double)conf[k] * v / tr) : 0.0f;
    }
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

hipError_t launch_structure_conf(const void *ref, nrr_dtype dtype, const int32_t dims[3],
                                 const int32_t *centers, int64_t n, int32_t block,
                                 const float *conf, float *out, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const dim3 grid((unsigned)((n + 3) / 4));
    const size_t bytes = (size_t)4 * (block + 2) * (block + 2) * conf_pitch(block) *
                         (dtype == NRR_U16 ? 2 : 4);
    const bool staged = bytes <= kConfLds;
    const size_t lds = staged ? bytes : 0;
    if (dtype == NRR_U16)
        hipLaunchKernelGGL(k_structure_conf<uint16_t>, grid, dim3(256), lds, stream,
                           static_cast<const uint16_t *>(ref), dims[0], dims[1], dims[2], centers,
                           n, block, staged, conf, out);
    else
        hipLaunchKernelGGL(k_structure_conf<float>, grid, dim3(256), lds, stream,
                           static_cast<const float *>(ref), dims[0], dims[1], dims[2], centers, n,
                           block, staged, conf, out);
    return hipGetLastError();
}

StatsLayout stats_layout(nrr_dtype dtype, const int32_t dims[3], const int32_t block[3],
                         bool pairs) {
    StatsLayout L;
    L.ox = dims[0] - block[0] + 1;
    L.oy = dims[1] - block[1] + 1;
    L.oz = dims[2] - block[2] + 1;
    // slack after the table: the search reads whole tiles of records, up to
    // kTileSlack rows and columns past the last valid origin
    const size_t nvox = (size_t)L.ox * L.oy * L.oz + (size_t)kTileSlack * (L.ox + 1);
    L.total = align_up(nvox * (dtype == NRR_U16 ? sizeof(StatU16) : sizeof(StatF32)), 256);
    L.pair_off = 0;
    if (pairs && dtype == NRR_U16) {  // + slack: staging reads whole 4-word row chunks
        L.pair_off = L.total;
        L.total += align_up(((size_t)dims[0] * dims[1] * dims[2] + 64) * 4, 256);
    }
    return L;
}

StatsLayout stats_layout(nrr_dtype dtype, const int32_t dims[3], int32_t block) {
    const int32_t b3[3] = {block, block, block};
    return stats_layout(dtype, dims, b3, true);
}

namespace {
// Origin planes per float statistics workgroup: ZC, fewer when that leaves
// the device with too few workgroups (small volumes), never below 4; then
// the same number of runs, of balanced lengths (a workgroup's time is its
// run plus bz - 1 planes: 256x256x124 at b = 7 takes 30+30+30+28 instead of
// 32+32+32+22).
int f32_run_planes(const StatsLayout &L) {
    const int64_t per_slab = (int64_t)((L.ox + TX - 1) / TX) * ((L.oy + TY - 1) / TY);
    const int64_t slabs = (512 + per_slab - 1) / per_slab;
    int zc = (int)((L.oz + slabs - 1) / slabs);
    zc = zc < 4 ? 4 : (zc > ZC ? ZC : zc);
    const int runs = (L.oz + zc - 1) / zc;
    return (L.oz + runs - 1) / runs;
}
}  // namespace

hipError_t launch_stats(const void *flt, nrr_dtype dtype, const int32_t dims[3],
                        const int32_t block[3], bool pairs, void *workspace, hipStream_t stream) {
    StatsLayout L = stats_layout(dtype, dims, block, pairs);
    char *ws = static_cast<char *>(workspace);
    const int bx = block[0], by = block[1], bz = block[2];
    if (dtype == NRR_U16) {
        // a run first sums bz planes: runs of one or two origin planes cost more
        // than the wavefronts they add (192x192x96, runs of one plane / three,
        // us: edge 9 24 / 17, 11 30 / 21, 13 32 / 24, 15 40 / 28; at bz = 3 one
        // plane is best, 17.9 against 18.9)
        const ColsGrid cg = cols_grid(L, bx, SC_WAVES, bz >= 9 ? 3 : bz >= 5 ? 2 : 1);
        const int zc = cg.zc;
        const dim3 grid((unsigned)cg.nwx, (unsigned)((cg.nwy + 3) / 4), (unsigned)cg.runs);
        StatU16 *out = reinterpret_cast<StatU16 *>(ws);
        const uint16_t *f = static_cast<const uint16_t *>(flt);
        switch (by) {
#define NRR_STATS_BY(BY)                                                                         \
    case BY:                                                                                     \
        if (bx == BY && bz == BY)                                                                \
            hipLaunchKernelGGL((k_stats_u16<BY, BY>), grid, dim3(256), 0, stream, f, dims[0],    \
                               dims[1], dims[2], bx, bz, L.ox, L.oy, L.oz, zc, out);             \
        else                                                                                     \
            hipLaunchKernelGGL((k_stats_u16<BY, 0>), grid, dim3(256), 0, stream, f, dims[0],     \
                               dims[1], dims[2], bx, bz, L.ox, L.oy, L.oz, zc, out);             \
        break;
            NRR_STATS_BY(1)
            NRR_STATS_BY(3)
            NRR_STATS_BY(5)
            NRR_STATS_BY(7)
            NRR_STATS_BY(9)
            NRR_STATS_BY(11)
            NRR_STATS_BY(13)
            NRR_STATS_BY(15)
#undef NRR_STATS_BY
        default:
            return hipErrorInvalidValue;  // block edges are odd, 1 .. 15
        }
        if (L.pair_off) {
            const int64_t nvox = (int64_t)dims[0] * dims[1] * dims[2];
            hipLaunchKernelGGL(k_pair_volume, dim3((unsigned)((nvox + 1023) / 1024)), dim3(256), 0,
                               stream, f, nvox, (int64_t)dims[0] * dims[1],
                               reinterpret_cast<uint32_t *>(ws + L.pair_off));
        }
        return hipGetLastError();
    }
    const int zc = f32_run_planes(L);
    dim3 grid((L.ox + TX - 1) / TX, (L.oy + TY - 1) / TY, (L.oz + zc - 1) / zc);
    const bool cubic = bx == by && by == bz;
    const auto fn = cubic && bx == 3    ? k_stats_f32<3>
                    : cubic && bx == 5  ? k_stats_f32<5>
                    : cubic && bx == 7  ? k_stats_f32<7>
                    : cubic && bx == 9  ? k_stats_f32<9>
                    : cubic && bx == 11 ? k_stats_f32<11>
                    : cubic && bx == 13 ? k_stats_f32<13>
                    : cubic && bx == 15 ? k_stats_f32<15>
                                        : k_stats_f32<0>;
    hipLaunchKernelGGL(fn, grid, dim3(256), fn == k_stats_f32<0> ? (size_t)bz * 256 * 16 : 0,
                       stream, static_cast<const float *>(flt), dims[0], dims[1], dims[2], bx, by,
                       bz, L.ox, L.oy, L.oz, zc, reinterpret_cast<StatF32 *>(ws));
    return hipGetLastError();
}

// Voxels outside the dtype's contract (12-bit data above 4095, float data
// not finite), counted into *bad.
__global__ __launch_bounds__(256) void k_check_u16(const uint16_t *__restrict__ v, int64_t n,
                                                   unsigned long long *__restrict__ bad) {
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        c += v[i] > 4095;
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(bad, c);
}

__global__ __launch_bounds__(256) void k_check_f32(const float *__restrict__ v, int64_t n,
                                                   unsigned long long *__restrict__ bad) {
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        c += !isfinite(v[i]);
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(bad, c);
}

__global__ void k_zero_u64(unsigned long long *p) {
    if (threadIdx.x == 0) *p = 0;
}

hipError_t launch_check_volume(const void *vol, nrr_dtype dtype, int64_t n, int64_t *bad,
                               hipStream_t stream) {
    unsigned long long *b = reinterpret_cast<unsigned long long *>(bad);
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, stream, b);
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    if (n > 0) {
        if (dtype == NRR_U16)
            hipLaunchKernelGGL(k_check_u16, dim3(blocks), dim3(256), 0, stream,
                               static_cast<const uint16_t *>(vol), n, b);
        else
            hipLaunchKernelGGL(k_check_f32, dim3(blocks), dim3(256), 0, stream,
                               static_cast<const float *>(vol), n, b);
    }
    return hipGetLastError();
}

hipError_t launch_pair_volume(const uint16_t *flt, const int32_t dims[3], uint32_t *pairs,
                              hipStream_t stream) {
    const int64_t nvox = (int64_t)dims[0] * dims[1] * dims[2];
    hipLaunchKernelGGL(k_pair_volume, dim3((unsigned)((nvox + 1023) / 1024)), dim3(256), 0, stream,
                       flt, nvox, (int64_t)dims[0] * dims[1], pairs);
    return hipGetLastError();
}

hipError_t launch_stats(const void *flt, nrr_dtype dtype, const int32_t dims[3], int32_t block,
                        void *workspace, hipStream_t stream) {
    const int32_t b3[3] = {block, block, block};
    return launch_stats(flt, dtype, dims, b3, true, workspace, stream);
}

hipError_t launch_stats_f32_multi(const float *flt, const int32_t dims[3], const int32_t *blocks,
                                  void *const *outs, int n, hipStream_t stream) {
    if (n < 1 || n > kStatsJobs) return hipErrorInvalidValue;
    StatsF32Jobs J{};
    J.n = n;
    int gx = 0, gy = 0, gz = 0, maxb = 0;
    for (int i = 0; i < n; ++i) {
        if (blocks[i] < 1 || blocks[i] > MAXB) return hipErrorInvalidValue;
        const int32_t b3[3] = {blocks[i], blocks[i], blocks[i]};
        const StatsLayout L = stats_layout(NRR_F32, dims, b3, false);
        StatsF32Job &j = J.job[i];
        j.b = blocks[i];
        j.ox = L.ox;
        j.oy = L.oy;
        j.oz = L.oz;
        j.zc = f32_run_planes(L);
        j.tiles_x = (L.ox + TX - 1) / TX;
        j.tiles_y = (L.oy + TY - 1) / TY;
        j.z_first = gz;
        gz += (L.oz + j.zc - 1) / j.zc;
        j.out = static_cast<StatF32 *>(outs[i]);
        gx = std::max(gx, j.tiles_x);
        gy = std::max(gy, j.tiles_y);
        if (blocks[i] != 5 && blocks[i] != 7 && blocks[i] != 9)  // its ring is in LDS
            maxb = std::max(maxb, (int)blocks[i]);
    }
    hipLaunchKernelGGL(k_stats_f32_multi, dim3((unsigned)gx, (unsigned)gy, (unsigned)gz), dim3(256),
                       (size_t)maxb * 256 * 16, stream, flt, dims[0], dims[1], dims[2], J);
    return hipGetLastError();
}

}  // namespace nrr
