// Reprojection (Sec. 3.4, Eq. 3-5) and hole classification (Sec. 3.1
// Stage 3, Sec. 3.5 Steps 1-2) for gfx950.
//
// This file is compiled without floating-point contraction: the fp64
// reprojection, the Eq. 6-8 extrema and the fp32 interpolation sums are
// evaluated operation by operation in a fixed order, so that their integer
// outcomes (target pixels, hole masks, widths, labels, boxes) are exactly
// reproducible.
#include <algorithm>
#include <cfloat>
#include <climits>

#include "bgs_internal.h"

namespace bgs {

RelPose rel_pose(const bgs_camera& src, const bgs_camera& dst) {
    RelPose P;
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q) {
            double p0 = dst.R[0 * 3 + r] * src.R[0 * 3 + q];
            double p1 = dst.R[1 * 3 + r] * src.R[1 * 3 + q];
            double p2 = dst.R[2 * 3 + r] * src.R[2 * 3 + q];
            P.M[r * 3 + q] = (p0 + p1) + p2;
        }
    double d0 = src.t[0] - dst.t[0], d1 = src.t[1] - dst.t[1], d2 = src.t[2] - dst.t[2];
    for (int r = 0; r < 3; ++r) {
        double p0 = dst.R[0 * 3 + r] * d0;
        double p1 = dst.R[1 * 3 + r] * d1;
        double p2 = dst.R[2 * 3 + r] * d2;
        P.c[r] = (p0 + p1) + p2;
    }
    return P;
}

namespace {

// X' = M X (+ c): a source-frame point in the destination frame.
__device__ inline void map_point(const RelPose& P, bool with_t, double X, double Y, double Z, double out[3]) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        double p0 = P.M[r * 3 + 0] * X;
        double p1 = P.M[r * 3 + 1] * Y;
        double p2 = P.M[r * 3 + 2] * Z;
        double s = (p0 + p1) + p2;
        out[r] = with_t ? s + P.c[r] : s;
    }
}

// Pinhole projection (Eq. 3) in pixels, unrounded.
__device__ inline void project(const WarpCam& c, const double X[3], double* u, double* v) {
    double qx = X[0] / X[2];
    double qy = X[1] / X[2];
    double sx = c.fx * qx;
    double sy = c.fy * qy;
    *u = sx + c.cx;
    *v = sy + c.cy;
}

__device__ inline uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, off, 64));
    return v;
}
__device__ inline uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
    return v;
}
__device__ inline uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
    return v;
}

// Block-wide reductions for 256-thread blocks; every thread gets the result.
// s4 is a 4-entry LDS scratch that the caller does not touch in between.
__device__ inline uint32_t block_sum_u32(uint32_t v, uint32_t* s4) {
    v = wave_sum_u32(v);
    if ((threadIdx.x & 63) == 0) s4[threadIdx.x >> 6] = v;
    __syncthreads();
    const uint32_t r = s4[0] + s4[1] + s4[2] + s4[3];
    __syncthreads();
    return r;
}
__device__ inline uint32_t block_min_u32(uint32_t v, uint32_t* s4) {
    v = wave_min_u32(v);
    if ((threadIdx.x & 63) == 0) s4[threadIdx.x >> 6] = v;
    __syncthreads();
    const uint32_t r = min(min(s4[0], s4[1]), min(s4[2], s4[3]));
    __syncthreads();
    return r;
}
__device__ inline uint32_t block_max_u32(uint32_t v, uint32_t* s4) {
    v = wave_max_u32(v);
    if ((threadIdx.x & 63) == 0) s4[threadIdx.x >> 6] = v;
    __syncthreads();
    const uint32_t r = max(max(s4[0], s4[1]), max(s4[2], s4[3]));
    __syncthreads();
    return r;
}

// Image kernels in 2D: a 256-thread block covers 64 columns x kBandRows
// rows, a wave per row at a time (coalesced), so no pixel index is divided.
constexpr int kBandRows = 16;
inline dim3 band_grid(int W, int H) { return dim3((unsigned)((W + 63) / 64), (unsigned)((H + kBandRows - 1) / kBandRows)); }

__global__ void k_warp_reset(DevStatus* st) {
    st->n_holes = 0;
    st->n_gap = 0;
    st->n_center = 0;
    st->n_rowfill = 0;
    st->n_boxes = 0;
    st->n_edge = 0;
    st->dmin_inv = 0u;
    st->dmax_bits = 0u;
    st->overflow &= ~2u;
}

__global__ __launch_bounds__(256) void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// Where source pixel (i, j) with alpha A and raw depth Dr lands: the
// fixed-order fp64 recipe of Eq. 4-5.  Returns false when it lands nowhere;
// *df gets the fp32 depth proxy of a covered source pixel (else stays
// untouched).
__device__ inline bool splat_target(const WarpCam& src, const WarpCam& dst, const RelPose& P, float a_min, float A,
                                      float Dr, int i, int j, int64_t* fu_out, int64_t* fv_out,
                                      unsigned long long* key, float* df_out) {
    const int64_t s = (int64_t)j * src.W + i;
    const double xn = ((double)i - src.cx) / src.fx;
    const double yn = ((double)j - src.cy) / src.fy;
    double Xp[3];
    bool ok;
    float zf;
    if (A >= a_min) {
        const float df = Dr / A;
        *df_out = df;
        const double d = (double)df;
        map_point(P, true, d * xn, d * yn, d, Xp);
        ok = Xp[2] > dst.z_near;
        zf = (float)Xp[2];
    } else {
        map_point(P, false, xn, yn, 1.0, Xp);
        ok = Xp[2] > 0.0;
        zf = INFINITY;
    }
    if (!ok) return false;
    double u, v;
    project(dst, Xp, &u, &v);
    const double fu = floor(u + 0.5), fv = floor(v + 0.5);
    if (!(fu >= 0.0 && fu <= (double)(dst.W - 1) && fv >= 0.0 && fv <= (double)(dst.H - 1))) return false;
    *fu_out = (int64_t)fu;
    *fv_out = (int64_t)fv;
    *key = ((unsigned long long)__float_as_uint(zf) << 32) | (unsigned long long)(uint32_t)s;
    return true;
}

// Forward splat of every source pixel into the destination z-buffer.
__global__ __launch_bounds__(256) void k_reproject_scatter(WarpCam src, WarpCam dst, RelPose P, float a_min,
                                                           const float* __restrict__ draw,
                                                           const float* __restrict__ alpha,
                                                           unsigned long long* __restrict__ zbuf, DevStatus* st) {
    __shared__ uint32_t s4[4];
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    uint32_t dmin = 0xFFFFFFFFu, dmax = 0u;
    // All of the thread's pixels are loaded first, so none waits on another.
    constexpr int kP = kBandRows / 4;
    float Av[kP], Dv[kP];
#pragma unroll
    for (int q = 0; q < kP; ++q) {
        const int j = blockIdx.y * kBandRows + (threadIdx.x >> 6) + 4 * q;
        const bool in = i < src.W && j < src.H;
        Av[q] = in ? alpha[(int64_t)j * src.W + i] : 0.f;
        Dv[q] = in ? draw[(int64_t)j * src.W + i] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kP; ++q) {
        const int j = blockIdx.y * kBandRows + (threadIdx.x >> 6) + 4 * q;
        if (i >= src.W || j >= src.H) continue;
        int64_t fu, fv;
        unsigned long long key;
        float df = -1.f;
        const bool hit = splat_target(src, dst, P, a_min, Av[q], Dv[q], i, j, &fu, &fv, &key, &df);
        if (df >= 0.f) {
            dmin = min(dmin, __float_as_uint(df));
            dmax = max(dmax, __float_as_uint(df));
        }
        if (hit) atomicMin(&zbuf[fv * dst.W + fu], key);
    }
    dmin = block_min_u32(dmin, s4);
    dmax = block_max_u32(dmax, s4);
    if (threadIdx.x == 0) {
        // Both words only grow, so a block whose range a read finds covered
        // need not queue for them (1603x1061, 1742 blocks: 47 -> 28 us).
        const uint32_t lo = __hip_atomic_load(&st->dmin_inv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t hi = __hip_atomic_load(&st->dmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (dmin != 0xFFFFFFFFu && ~dmin > lo) atomicMax(&st->dmin_inv, ~dmin);
        if (dmax > hi) atomicMax(&st->dmax_bits, dmax);
    }
}

// Row-preserving form (the host has proven that every splat stays on its
// source row, as for a rig that keeps the orientation and moves along x):
// one block of NT threads per row, the row's z-buffer in LDS (64-bit LDS
// atomicMin), the z-test and the resolve in one kernel.  Same recipe, same
// result as the scatter/resolve pair.  Each thread takes kRowPix pixels of a
// chunk of NT * kRowPix and issues all of their loads before any arithmetic,
// so the row's memory latency is paid once per chunk rather than once per
// pixel; the row's four counters are reduced in one LDS exchange.
// kStage: the source row's colour and alpha are loaded with its alpha and
// depth (coalesced, in the same burst) and kept in LDS, so the resolve
// reads them there instead of gathering them from memory after the z-test.
constexpr int kRowThreads = 512, kRowItems = 2;  // threads per row block, pixels per thread per chunk
constexpr int kRowStageLds = 48 * 1024;         // LDS bytes of a staged row block (z row + source row)
constexpr int kRowStageMinW = 1024;             // source rows at least this long are staged
template <int NT, int kRowPix, bool kStage>
__global__ __launch_bounds__(NT) void k_reproject_rows(WarpCam src, WarpCam dst, RelPose P, float a_min,
                                                       const float* __restrict__ draw,
                                                       const float* __restrict__ alpha,
                                                       const float* __restrict__ rgb, float* __restrict__ rgb_dst,
                                                       float* __restrict__ z_dst, float* __restrict__ a_dst,
                                                       uint8_t* __restrict__ hole, uint4* __restrict__ wpart) {
    extern __shared__ unsigned long long zrow[];
    __shared__ uint4 s_red[NT / 64];
    // Staged: the source row's r, g, b and alpha planes follow the z row.
    float* s_src = reinterpret_cast<float*>(zrow + dst.W);
    const int j = blockIdx.x;
    const int64_t ns = (int64_t)src.W * src.H;
    for (int t = threadIdx.x; t < dst.W; t += NT) zrow[t] = ~0ull;
    __syncthreads();
    uint32_t dmin = 0xFFFFFFFFu, dmax = 0u, off_row = 0;
    const int64_t srow = (int64_t)j * src.W;
    for (int base = 0; base < src.W; base += NT * kRowPix) {
        float Av[kRowPix], Dv[kRowPix], Rv[kRowPix], Gv[kRowPix], Bv[kRowPix];
#pragma unroll
        for (int k = 0; k < kRowPix; ++k) {
            const int i = base + threadIdx.x + NT * k;
            Av[k] = i < src.W ? alpha[srow + i] : 0.f;
            Dv[k] = i < src.W ? draw[srow + i] : 0.f;
            if (kStage) {
                Rv[k] = i < src.W ? rgb[srow + i] : 0.f;
                Gv[k] = i < src.W ? rgb[ns + srow + i] : 0.f;
                Bv[k] = i < src.W ? rgb[2 * ns + srow + i] : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < kRowPix; ++k) {
            const int i = base + threadIdx.x + NT * k;
            if (i >= src.W) continue;
            if (kStage) {
                s_src[i] = Rv[k];
                s_src[src.W + i] = Gv[k];
                s_src[2 * src.W + i] = Bv[k];
                s_src[3 * src.W + i] = Av[k];
            }
            int64_t fu, fv;
            unsigned long long key;
            float df = -1.f;
            const bool hit = splat_target(src, dst, P, a_min, Av[k], Dv[k], i, j, &fu, &fv, &key, &df);
            if (df >= 0.f) {
                dmin = min(dmin, __float_as_uint(df));
                dmax = max(dmax, __float_as_uint(df));
            }
            if (hit) {
                if (fv == j) atomicMin(&zrow[fu], key);
                else off_row = 1;
            }
        }
    }
    __syncthreads();
    const int64_t nd = (int64_t)dst.W * dst.H;
    const int64_t drow = (int64_t)j * dst.W;
    uint32_t holes = 0;
    for (int base = 0; base < dst.W; base += NT * kRowPix) {
        unsigned long long kv[kRowPix];
        float c0[kRowPix], c1[kRowPix], c2[kRowPix], av[kRowPix];
#pragma unroll
        for (int k = 0; k < kRowPix; ++k) {
            const int t = base + threadIdx.x + NT * k;
            kv[k] = t < dst.W ? zrow[t] : ~0ull;
            const uint32_t sidx = (uint32_t)(kv[k] & 0xFFFFFFFFull);
            const bool have = kv[k] != ~0ull;
            if (kStage) {
                // A splat of this row comes from this row of the source.
                const int i = have ? (int)((int64_t)sidx - srow) : 0;
                c0[k] = have ? s_src[i] : 0.f;
                c1[k] = have ? s_src[src.W + i] : 0.f;
                c2[k] = have ? s_src[2 * src.W + i] : 0.f;
                av[k] = have ? s_src[3 * src.W + i] : 0.f;
            } else {
                c0[k] = have ? rgb[sidx] : 0.f;
                c1[k] = have ? rgb[ns + sidx] : 0.f;
                c2[k] = have ? rgb[2 * ns + sidx] : 0.f;
                av[k] = have ? alpha[sidx] : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < kRowPix; ++k) {
            const int t = base + threadIdx.x + NT * k;
            if (t >= dst.W) continue;
            const int64_t g = drow + t;
            const bool have = kv[k] != ~0ull;
            rgb_dst[g] = c0[k];
            rgb_dst[nd + g] = c1[k];
            rgb_dst[2 * nd + g] = c2[k];
            z_dst[g] = have ? __uint_as_float((uint32_t)(kv[k] >> 32)) : INFINITY;
            a_dst[g] = av[k];
            hole[g] = have ? 0 : 1;
            holes += have ? 0u : 1u;
        }
    }
    // The row's partial: max of ~dmin, max of dmax, hole count, off-row flag.
    uint32_t x = wave_max_u32(~dmin), y = wave_max_u32(dmax), h = wave_sum_u32(holes), f = wave_max_u32(off_row);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = make_uint4(x, y, h, f);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint4 r = s_red[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) {
            const uint4 q = s_red[w];
            r.x = max(r.x, q.x);
            r.y = max(r.y, q.y);
            r.z += q.z;
            r.w = max(r.w, q.w);
        }
        // off_row cannot be set when the host's bound holds (overflow bit 2).
        wpart[j] = make_uint4(r.x, r.y, r.z, r.w ? 4u : 0u);
    }
}

// Fold the per-row partials of k_reproject_rows (n of them; none for the
// scatter form, which reduces with atomics) into the status block, from
// every thread of a 256-thread block.  Returns the depth-proxy range of the
// covered pixels, or [z_near, z_far] when none was covered, to every thread.
// The kernel is a single workgroup on the critical path, so its latency is
// what counts: the status words and four partials per thread are loaded
// together, and the four reductions share one barrier.
__device__ inline void fold_warp_parts(const uint4* __restrict__ wpart, int n, DevStatus* st, float z_near,
                                       float z_far, float* r0, float* r1) {
    __shared__ uint4 s_w[4];
    const uint32_t a0 = st->dmin_inv, b0 = st->dmax_bits, h0 = st->n_holes, f0 = st->overflow;
    uint32_t a = 0u, b = 0u, h = 0u, f = 0u;  // 0 is the identity of each fold
    for (int i0 = threadIdx.x; i0 < n; i0 += 1024) {
        uint4 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = i0 + 256 * u < n ? wpart[i0 + 256 * u] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a = max(a, q[u].x);
            b = max(b, q[u].y);
            h += q[u].z;
            f |= q[u].w;
        }
    }
    a = wave_max_u32(a);
    b = wave_max_u32(b);
    h = wave_sum_u32(h);
    f = wave_max_u32(f);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = make_uint4(a, b, h, f);
    __syncthreads();
    a = a0;
    b = b0;
    h = 0u;
    f = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint4 q = s_w[w];
        a = max(a, q.x);
        b = max(b, q.y);
        h += q.z;
        f = max(f, q.w);
    }
    if (threadIdx.x == 0) {
        st->dmin_inv = a;
        st->dmax_bits = b;
        st->n_holes = h0 + h;
        if (f) st->overflow = f0 | f;
    }
    if (a == 0u) {
        *r0 = z_near;
        *r1 = z_far;
    } else {
        *r0 = __uint_as_float(~a);
        *r1 = __uint_as_float(b);
    }
}

// 1024 threads: a quarter of the blocks, whose counts queue for one word
// (1603x1061: 29 -> 15 us).
__global__ __launch_bounds__(1024) void k_reproject_resolve(int64_t nd, int64_t ns,
                                                           const unsigned long long* __restrict__ zbuf,
                                                           const float* __restrict__ rgb,
                                                           const float* __restrict__ alpha,
                                                           float* __restrict__ rgb_dst, float* __restrict__ z_dst,
                                                           float* __restrict__ a_dst, uint8_t* __restrict__ hole,
                                                           DevStatus* st) {
    __shared__ uint32_t s_h[16];
    // Four pixels per thread, the keys loaded together and then the source
    // pixels they name: two memory latencies per block, not two per pixel.
    const int64_t t0 = (int64_t)blockIdx.x * 4096 + threadIdx.x;
    unsigned long long key[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) key[q] = t0 + 1024 * q < nd ? zbuf[t0 + 1024 * q] : ~0ull;
    float c0[4], c1[4], c2[4], a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool have = key[q] != ~0ull;
        const uint32_t s = (uint32_t)(key[q] & 0xFFFFFFFFull);
        c0[q] = have ? rgb[s] : 0.f;
        c1[q] = have ? rgb[ns + s] : 0.f;
        c2[q] = have ? rgb[2 * ns + s] : 0.f;
        a[q] = have ? alpha[s] : 0.f;
    }
    uint32_t h = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t t = t0 + 1024 * q;
        if (t >= nd) continue;
        const bool have = key[q] != ~0ull;
        rgb_dst[t] = c0[q];
        rgb_dst[nd + t] = c1[q];
        rgb_dst[2 * nd + t] = c2[q];
        z_dst[t] = have ? __uint_as_float((uint32_t)(key[q] >> 32)) : INFINITY;
        a_dst[t] = a[q];
        hole[t] = have ? 0 : 1;
        h += have ? 0u : 1u;
    }
    h = wave_sum_u32(h);
    if ((threadIdx.x & 63) == 0) s_h[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0) {
        h = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) h += s_h[w];
        if (h) atomicAdd(&st->n_holes, h);
    }
}

// Standalone reprojection: fold the partials and write the depth range.
__global__ __launch_bounds__(256) void k_warp_finish(const uint4* __restrict__ wpart, int n, DevStatus* st,
                                                     float z_near, float z_far, float* range) {
    float r0, r1;
    fold_warp_parts(wpart, n, st, z_near, z_far, &r0, &r1);
    if (threadIdx.x == 0) {
        range[0] = r0;
        range[1] = r1;
    }
}

// ---------------------------------------------------------------------------
// Step 1: edge ROIs (Eq. 6-8).  One block.
// ---------------------------------------------------------------------------
// Sample k of N along an edge of L pixels: the nearest pixel to
// k (L - 1) / (N - 1), halves rounded down, i.e. floor((2k(L-1) + N-1) /
// (2(N-1))).  The quotient is taken in double (exact operands below 2^53,
// so within one of the floor) and corrected in integers, which costs far
// less than a 64-bit integer division.
__device__ inline int edge_pos(int k, int N, int L) {
    if (N <= 1) return 0;
    const int64_t a = 2 * (int64_t)k * (L - 1) + (N - 1), b = 2 * (int64_t)(N - 1);
    int64_t q = (int64_t)((double)a / (double)b);
    if (q * b > a) --q;
    else if ((q + 1) * b <= a) ++q;
    return (int)q;
}
__device__ inline double snap(double x) {
    double r = rint(x);
    return fabs(x - r) <= 1e-6 ? r : x;
}
__device__ inline double clampd(double x, double a, double b) { return x < a ? a : (x > b ? b : x); }
__device__ inline int64_t align_down(int64_t x, int64_t T) { return (x / T) * T; }
__device__ inline int64_t align_up(int64_t x, int64_t T) { return ((x + T - 1) / T) * T; }

// With tm set, also writes the edge boxes' tiles into the ROI tile mask
// (every tile covered by an edge box is 1, all others 0); k_gap_fill does
// that instead when it runs, over its many workgroups.  depth_range null: the range
// comes from the reprojection just run, whose partials (n_wpart, possibly
// none) it folds into the status block first.
__global__ __launch_bounds__(256) void k_edge_rois(WarpCam src, WarpCam dst, RelPose P, int N, int margin, int T,
                                                   int edge_bounds, const float* __restrict__ depth_range,
                                                   const uint4* __restrict__ wpart, int n_wpart, DevStatus* st,
                                                   bgs_box* boxes, int box_cap, uint8_t* __restrict__ tm) {
    __shared__ double red[8][4];
    __shared__ int32_t sbx[4][6];
    __shared__ int snb;
    float r0, r1;
    if (depth_range) {
        r0 = depth_range[0];
        r1 = depth_range[1];
    } else {
        fold_warp_parts(wpart, n_wpart, st, (float)src.z_near, (float)src.z_far, &r0, &r1);
    }
    const double hyp0 = (double)r0, hyp1 = (double)r1;
    double xmin = INFINITY, xmax = -INFINITY, ymin = INFINITY, ymax = -INFINITY;
    // Per side, the worst case of its own edge (edge_bounds = 1): largest x
    // of the left edge, smallest x of the right, largest y of the top,
    // smallest y of the bottom.
    double lmax = -INFINITY, rmin = INFINITY, tmax = -INFINITY, bmin = INFINITY;
    const int total = 4 * N;  // N <= 65536
    for (int q = threadIdx.x; q < total; q += 256) {
        const int edge = q / N;
        const int k = q - edge * N;
        int i, j;
        if (edge == 0) { i = edge_pos(k, N, src.W); j = 0; }
        else if (edge == 1) { i = edge_pos(k, N, src.W); j = src.H - 1; }
        else if (edge == 2) { i = 0; j = edge_pos(k, N, src.H); }
        else { i = src.W - 1; j = edge_pos(k, N, src.H); }
        const double xn = ((double)i - src.cx) / src.fx;
        const double yn = ((double)j - src.cy) / src.fy;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double d = h ? hyp1 : hyp0;
            double Xp[3];
            map_point(P, true, d * xn, d * yn, d, Xp);
            if (!(Xp[2] > dst.z_near)) continue;
            double u, v;
            project(dst, Xp, &u, &v);
            xmin = fmin(xmin, u);
            xmax = fmax(xmax, u);
            ymin = fmin(ymin, v);
            ymax = fmax(ymax, v);
            if (edge == 0) tmax = fmax(tmax, v);
            else if (edge == 1) bmin = fmin(bmin, v);
            else if (edge == 2) lmax = fmax(lmax, u);
            else rmin = fmin(rmin, u);
        }
    }
    // min / max are exact in any order: wave shuffles, then the four waves.
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        xmin = fmin(xmin, __shfl_xor(xmin, off, 64));
        xmax = fmax(xmax, __shfl_xor(xmax, off, 64));
        ymin = fmin(ymin, __shfl_xor(ymin, off, 64));
        ymax = fmax(ymax, __shfl_xor(ymax, off, 64));
        lmax = fmax(lmax, __shfl_xor(lmax, off, 64));
        rmin = fmin(rmin, __shfl_xor(rmin, off, 64));
        tmax = fmax(tmax, __shfl_xor(tmax, off, 64));
        bmin = fmin(bmin, __shfl_xor(bmin, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        red[0][w] = xmin;
        red[1][w] = xmax;
        red[2][w] = ymin;
        red[3][w] = ymax;
        red[4][w] = lmax;
        red[5][w] = rmin;
        red[6][w] = tmax;
        red[7][w] = bmin;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double rx0 = fmin(fmin(red[0][0], red[0][1]), fmin(red[0][2], red[0][3]));
        const double rx1 = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
        const double ry0 = fmin(fmin(red[2][0], red[2][1]), fmin(red[2][2], red[2][3]));
        const double ry1 = fmax(fmax(red[3][0], red[3][1]), fmax(red[3][2], red[3][3]));
        const double el = fmax(fmax(red[4][0], red[4][1]), fmax(red[4][2], red[4][3]));
        const double er = fmin(fmin(red[5][0], red[5][1]), fmin(red[5][2], red[5][3]));
        const double et = fmax(fmax(red[6][0], red[6][1]), fmax(red[6][2], red[6][3]));
        const double eb = fmin(fmin(red[7][0], red[7][1]), fmin(red[7][2], red[7][3]));
        const bool pe = edge_bounds != 0;
        const double W = dst.W, H = dst.H, m = margin;
        const double hw = floor(W / 2.0), hh = floor(H / 2.0);
        // A side whose own edge has no valid projection keeps Eq. 6.
        const double umin = snap(pe && el > -INFINITY ? el : rx0), umax = snap(pe && er < INFINITY ? er : rx1);
        const double vmin = snap(pe && et > -INFINITY ? et : ry0), vmax = snap(pe && eb < INFINITY ? eb : ry1);
        const double lw = umin > 0.0 ? clampd(ceil(umin) + m, 0.0, hw) : 0.0;
        const double rw = umax < W - 1.0 ? clampd((W - 1.0) - floor(umax) + m, 0.0, hw) : 0.0;
        const double th = vmin > 0.0 ? clampd(ceil(vmin) + m, 0.0, hh) : 0.0;
        const double bh = vmax < H - 1.0 ? clampd((H - 1.0) - floor(vmax) + m, 0.0, hh) : 0.0;
        const int w4[4] = {(int)lw, (int)rw, (int)th, (int)bh};
        const int64_t Wi = dst.W, Hi = dst.H;
        int nb = 0;
        int32_t (*bx)[6] = sbx;  // LDS: indexed by the running box count
        if (w4[0] > 0) {
            int64_t x1 = align_up(w4[0], T);
            int32_t b[6] = {0, 0, (int32_t)(x1 < Wi ? x1 : Wi), (int32_t)Hi, BGS_BOX_LEFT, -1};
            for (int q = 0; q < 6; ++q) bx[nb][q] = b[q];
            ++nb;
        }
        if (w4[1] > 0) {
            int32_t b[6] = {(int32_t)align_down(Wi - w4[1], T), 0, (int32_t)Wi, (int32_t)Hi, BGS_BOX_RIGHT, -1};
            for (int q = 0; q < 6; ++q) bx[nb][q] = b[q];
            ++nb;
        }
        if (w4[2] > 0) {
            int64_t y1 = align_up(w4[2], T);
            int32_t b[6] = {0, 0, (int32_t)Wi, (int32_t)(y1 < Hi ? y1 : Hi), BGS_BOX_TOP, -1};
            for (int q = 0; q < 6; ++q) bx[nb][q] = b[q];
            ++nb;
        }
        if (w4[3] > 0) {
            int32_t b[6] = {0, (int32_t)align_down(Hi - w4[3], T), (int32_t)Wi, (int32_t)Hi, BGS_BOX_BOTTOM, -1};
            for (int q = 0; q < 6; ++q) bx[nb][q] = b[q];
            ++nb;
        }
        for (int q = 0; q < 4; ++q) st->widths[q] = w4[q];
        st->n_edge = (uint32_t)nb;
        snb = nb;
        for (int b = 0; b < nb; ++b) {
            for (int q = 0; q < 6; ++q) st->edge_boxes[b * 6 + q] = bx[b][q];
            if (b < box_cap) {
                boxes[b].x0 = bx[b][0];
                boxes[b].y0 = bx[b][1];
                boxes[b].x1 = bx[b][2];
                boxes[b].y1 = bx[b][3];
                boxes[b].kind = bx[b][4];
                boxes[b].label = bx[b][5];
            }
        }
    }
    __syncthreads();
    if (!tm) return;  // the gap fill writes the mask
    // The mask: box b covers tile columns [x0 / T, ceil(x1 / T)) and rows
    // [y0 / T, ceil(y1 / T)).  The tile ranges sit in registers (the byte
    // stores could alias LDS through a generic pointer, which would reload
    // them per tile), and a thread takes four consecutive tiles per step,
    // so that one division places them all.
    const int tiles_x = (dst.W + T - 1) / T, n_tiles = tiles_x * ((dst.H + T - 1) / T);
    const int nbx = snb;
    int tr[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const bool on = b < nbx;
        tr[b][0] = on ? sbx[b][0] / T : 0;
        tr[b][1] = on ? sbx[b][1] / T : 0;
        tr[b][2] = on ? (sbx[b][2] + T - 1) / T : 0;
        tr[b][3] = on ? (sbx[b][3] + T - 1) / T : 0;
    }
    for (int t0 = 4 * threadIdx.x; t0 < n_tiles; t0 += 4 * 256) {
        int ty = t0 / tiles_x, tx = t0 - ty * tiles_x;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (t0 + u < n_tiles) {
                bool hit = false;
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    hit = hit || (tx >= tr[b][0] && tx < tr[b][2] && ty >= tr[b][1] && ty < tr[b][3]);
                tm[t0 + u] = hit ? 1 : 0;
            }
            if (++tx == tiles_x) {
                tx = 0;
                ++ty;
            }
        }
    }
}

__device__ inline bool in_edge(const DevStatus* st, int x, int y) {
    const int ne = (int)st->n_edge;
    for (int b = 0; b < ne; ++b) {
        const int32_t* e = st->edge_boxes + b * 6;
        if (x >= e[0] && x < e[2] && y >= e[1] && y < e[3]) return true;
    }
    return false;
}

// The (at most four) edge boxes, read once into registers.
struct EdgeBoxes {
    int n;
    int b[4][4];  // x0, y0, x1, y1
    __device__ explicit EdgeBoxes(const DevStatus* st) {
        n = (int)st->n_edge;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) b[k][q] = st->edge_boxes[k * 6 + q];
    }
    __device__ bool contains(int x, int y) const {
        bool in = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) in = in || (k < n && x >= b[k][0] && x < b[k][2] && y >= b[k][1] && y < b[k][3]);
        return in;
    }
    // Does a box overlap the T x T tile whose first pixel is (x0, y0)?
    __device__ bool overlaps(int x0, int y0, int T) const {
        bool in = false;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            in = in || (k < n && x0 < b[k][2] && b[k][0] < x0 + T && y0 < b[k][3] && b[k][1] < y0 + T);
        return in;
    }
};

// ---------------------------------------------------------------------------
// Gap interpolation, Jacobi passes done in place.  tag[p] = 0 for a pixel
// that was never a hole, k for a hole filled in pass k, 255 for a hole.  In
// pass k a neighbour counts as valid iff its tag is below k, which is the
// state before the pass; a pixel filled in pass k is written only where no
// other pixel of pass k reads it.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tag_init(int64_t n, const uint8_t* __restrict__ cls, uint8_t* __restrict__ tag) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p < n) tag[p] = cls[p] ? 255 : 0;
}

__global__ __launch_bounds__(256) void k_gap_pass(int W, int H, int pass, float* rgb, float* z, float* alpha,
                                                  uint8_t* tag, uint8_t* __restrict__ cls, DevStatus* st) {
    __shared__ uint32_t s4[4];
    const int64_t n = (int64_t)W * H;
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    uint32_t filled = 0;
    for (int r = threadIdx.x >> 6; r < kBandRows; r += 4) {
        const int y = blockIdx.y * kBandRows + r;
        if (x >= W || y >= H) continue;
        const int64_t p = (int64_t)y * W + x;
        if (tag[p] != 255 || in_edge(st, x, y)) continue;
        {
            const int NX[8] = {-1, 0, 1, -1, 1, -1, 0, 1};
            const int NY[8] = {-1, -1, -1, 0, 0, 1, 1, 1};
            int cnt = 0;
            float s0 = 0.f, s1 = 0.f, s2 = 0.f, sa = 0.f, zm = -INFINITY;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int xx = x + NX[q], yy = y + NY[q];
                if (xx < 0 || yy < 0 || xx >= W || yy >= H) continue;
                const int64_t r = (int64_t)yy * W + xx;
                if ((int)tag[r] >= pass) continue;  // a hole, or filled in this pass
                s0 = s0 + rgb[r];
                s1 = s1 + rgb[n + r];
                s2 = s2 + rgb[2 * n + r];
                sa = sa + alpha[r];
                const float zr = z[r];
                if (zr > zm) zm = zr;
                ++cnt;
            }
            if (cnt > 0) {
                const float fc = (float)cnt;
                rgb[p] = s0 / fc;
                rgb[n + p] = s1 / fc;
                rgb[2 * n + p] = s2 / fc;
                alpha[p] = sa / fc;
                z[p] = zm;
                tag[p] = (uint8_t)pass;
                cls[p] = (uint8_t)BGS_CLS_GAP;
                ++filled;
            }
        }
    }
    filled = block_sum_u32(filled, s4);
    if (threadIdx.x == 0 && filled) atomicAdd(&st->n_gap, filled);
}

// The same gap passes and the center mask in one kernel: a block loads its
// 64 x kBandRows tile plus a halo of kH >= passes pixels into LDS, runs the
// passes there (pass j is final for pixels at least j from the halo's
// edge, which after all passes includes the tile), and writes the tile's filled
// pixels, tags and center mask.  Per pixel it computes exactly what
// k_tag_init, k_gap_pass and k_center_mask compute.  It also writes the
// ROI tile mask's edge-box tiles (the center boxes are added after it).
// Its filled and center counts go to gpart (one entry per block) rather
// than to shared counters, so that hundreds of blocks do not serialise on
// one cache line; the component-box kernels add them up.
constexpr int kGapMaxHalo = 4;
constexpr uint8_t kTagEdge = 253, kTagOut = 254;

// Workgroups are dispatched to the 8 XCDs in turn (block b to XCD b % 8),
// and each XCD has its own L2.  Tile t of an image's gx * gy tiles is
// given to a block of the XCD that owns its row-major eighth of the tiles,
// so neighbouring tiles, which read each other's edge pixels as halo, are
// mostly read through the same L2.  A bijection of [0, gx * gy).
__device__ inline void xcd_tile(uint32_t b, uint32_t gx, uint32_t gy, int* tx, int* ty) {
    const uint32_t n = gx * gy, q = n / 8, r = n % 8;
    const uint32_t xcd = b % 8, k = b / 8;
    const uint32_t t = xcd * q + min(xcd, r) + k;
    *tx = (int)(t % gx);
    *ty = (int)(t / gx);
}

// kH: the halo the LDS region is sized for (passes <= kH).  1D grid of
// ceil(W / 64) * ceil(H / kBandRows) blocks.
template <int kH>
__global__ __launch_bounds__(256) void k_gap_fill(int W, int H, int passes, float* __restrict__ rgb,
                                                  float* __restrict__ z, float* __restrict__ alpha,
                                                  uint8_t* __restrict__ tag_out, uint8_t* __restrict__ cls,
                                                  uint8_t* __restrict__ center, const DevStatus* st,
                                                  uint2* __restrict__ gpart, int T, int tiles_x, int tiles_y,
                                                  uint8_t* __restrict__ tm) {
    constexpr int RW = 64 + 2 * kH, RH = kBandRows + 2 * kH;
    __shared__ float s_c[3][RH * RW];
    __shared__ float s_a[RH * RW], s_z[RH * RW];
    // Tag per pixel: 0 no hole, k a hole filled in pass k, 255 a hole still
    // open, kTagEdge a hole inside an edge ROI (never filled), kTagOut
    // outside the image.  In pass k a neighbour is valid iff its tag is
    // below k.
    __shared__ uint8_t s_tag[RH * RW];
    __shared__ uint16_t s_hl[RH * RW];  // the open holes one pixel or more inside the region
    __shared__ uint32_t s_nh;
    __shared__ uint32_t s4[4];
    const uint32_t gx = (uint32_t)(W + 63) / 64, gy = (uint32_t)(H + kBandRows - 1) / kBandRows;
    int bx, by;
    xcd_tile(blockIdx.x, gx, gy, &bx, &by);
    const uint32_t gb = (uint32_t)by * gx + (uint32_t)bx;
    const int64_t n = (int64_t)W * H;
    // The halo is kH pixels whatever the number of passes: a wider halo
    // changes nothing inside the tile (pass j is final for the pixels j or
    // more from the region's edge).
    const int x0 = bx * 64 - kH, y0 = by * kBandRows - kH;
    const EdgeBoxes eb(st);
    if (threadIdx.x == 0) s_nh = 0;
    {
        // The edge ROIs in the tile mask: the tiles whose first pixel lies
        // in this block's region (so each tile is written by one block).
        const int rx = bx * 64, ry = by * kBandRows;
        const int tx0 = (rx + T - 1) / T, tx1 = min(tiles_x, (rx + 64 + T - 1) / T);
        const int ty0 = (ry + T - 1) / T, ty1 = min(tiles_y, (ry + kBandRows + T - 1) / T);
        const int ntx = tx1 - tx0, nty = ty1 - ty0;
        for (int k = threadIdx.x; ntx > 0 && k < ntx * nty; k += 256) {
            const int ty = ty0 + k / ntx, tx = tx0 + k % ntx;
            tm[(int64_t)ty * tiles_x + tx] = eb.overlaps(tx * T, ty * T, T) ? 1 : 0;
        }
    }
    // The classes of the tile and its halo first.  Holes are sparse: without
    // an open one in the tile (a hole outside the edge ROIs), or without any
    // filled pixel around them, no pass changes the tile and the images are
    // not read (2064x2208: 60 -> 55 us).
    constexpr int kLoads = (RW * RH + 255) / 256;
    uint8_t lh[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int i = threadIdx.x + 256 * q;
        const int lx = i % RW, ly = i / RW, x = x0 + lx, y = y0 + ly;
        const bool ok = i < RW * RH && x >= 0 && y >= 0 && x < W && y < H;
        lh[q] = !ok ? kTagOut : cls[(int64_t)y * W + x] ? 255 : 0;
    }
    bool open = false, full = false;
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int i = threadIdx.x + 256 * q;
        if (i >= RW * RH) continue;
        const int lx = i % RW, ly = i / RW, x = x0 + lx, y = y0 + ly;
        const uint8_t t = lh[q] == 255 && eb.contains(x, y) ? kTagEdge : lh[q];
        s_tag[i] = t;
        full = full || t == 0;
        open = open || (t == 255 && lx >= kH && lx < kH + 64 && ly >= kH && ly < kH + kBandRows);
    }
    const bool any_open = __syncthreads_or(open), any_full = __syncthreads_or(full);
    if (!any_open || !any_full) {
        uint32_t centers = 0;
        for (int i = threadIdx.x; i < 64 * kBandRows; i += 256) {
            const int lx = kH + (i & 63), ly = kH + (i >> 6), x = x0 + lx, y = y0 + ly;
            if (x >= W || y >= H) continue;
            const int64_t p = (int64_t)y * W + x;
            const uint8_t t = s_tag[ly * RW + lx];
            tag_out[p] = t >= kTagEdge ? 255 : t;
            const uint32_t c = t == 255 ? 1u : 0u;
            center[p] = (uint8_t)c;
            centers += c;
        }
        if (any_open) centers = block_sum_u32(centers, s4);
        if (threadIdx.x == 0) gpart[gb] = make_uint2(0u, centers);
        return;
    }
    // The images' values there: all loads first (unrolled, so none waits on
    // another), then the LDS stores.
    float lc0[kLoads], lc1[kLoads], lc2[kLoads], la[kLoads], lz[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int i = threadIdx.x + 256 * q;
        const int lx = i % RW, ly = i / RW, x = x0 + lx, y = y0 + ly;
        const bool ok = lh[q] == 0;
        const int64_t p = ok ? (int64_t)y * W + x : 0;
        lc0[q] = ok ? rgb[p] : 0.f;
        lc1[q] = ok ? rgb[n + p] : 0.f;
        lc2[q] = ok ? rgb[2 * n + p] : 0.f;
        la[q] = ok ? alpha[p] : 0.f;
        lz[q] = ok ? z[p] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int i = threadIdx.x + 256 * q;
        if (i >= RW * RH) continue;
        s_c[0][i] = lc0[q];
        s_c[1][i] = lc1[q];
        s_c[2][i] = lc2[q];
        s_a[i] = la[q];
        s_z[i] = lz[q];
    }
    __syncthreads();
    // The open holes, listed once (in no particular order: a pass reads
    // only tags below its own number, so its pixels are independent), so
    // that the passes visit nothing else.
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const int i = threadIdx.x + 256 * q;
        const int lx = i % RW, ly = i / RW;
        const bool open = i < RW * RH && lx >= 1 && lx < RW - 1 && ly >= 1 && ly < RH - 1 && s_tag[i] == 255;
        const unsigned long long bal = __ballot(open);
        const int lane = threadIdx.x & 63;
        uint32_t base = 0;
        if (lane == 0 && bal) base = atomicAdd(&s_nh, (uint32_t)__popcll(bal));
        base = __shfl(base, 0, 64);
        if (open) s_hl[base + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)i;
    }
    __syncthreads();
    const int nh = (int)s_nh;
    for (int pass = 1; pass <= passes; ++pass) {
        for (int e = threadIdx.x; e < nh; e += 256) {
            const int li = s_hl[e];
            const int ly = li / RW, lx = li - ly * RW;
            // pixels at least `pass` from the region's edge, not yet filled
            if (lx < pass || lx >= RW - pass || ly < pass || ly >= RH - pass || s_tag[li] != 255) continue;
            const int NX[8] = {-1, 0, 1, -1, 1, -1, 0, 1};
            const int NY[8] = {-1, -1, -1, 0, 0, 1, 1, 1};
            // All eight neighbours' values are read together (no read waits
            // on another), then the valid ones are summed in neighbour order.
            bool ok[8];
            float v0[8], v1[8], v2[8], va[8], vz[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int r = (ly + NY[q]) * RW + lx + NX[q];
                ok[q] = (int)s_tag[r] < pass;  // not outside, not a hole, not filled in this pass
                v0[q] = s_c[0][r];
                v1[q] = s_c[1][r];
                v2[q] = s_c[2][r];
                va[q] = s_a[r];
                vz[q] = s_z[r];
            }
            int cnt = 0;
            float s0 = 0.f, s1 = 0.f, s2 = 0.f, sa = 0.f, zm = -INFINITY;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (!ok[q]) continue;
                s0 = s0 + v0[q];
                s1 = s1 + v1[q];
                s2 = s2 + v2[q];
                sa = sa + va[q];
                if (vz[q] > zm) zm = vz[q];
                ++cnt;
            }
            if (cnt > 0) {
                const float fc = (float)cnt;
                s_c[0][li] = s0 / fc;
                s_c[1][li] = s1 / fc;
                s_c[2][li] = s2 / fc;
                s_a[li] = sa / fc;
                s_z[li] = zm;
                s_tag[li] = (uint8_t)pass;
            }
        }
        __syncthreads();
    }
    uint32_t filled = 0, centers = 0;
    for (int i = threadIdx.x; i < 64 * kBandRows; i += 256) {
        const int lx = kH + (i & 63), ly = kH + (i >> 6), x = x0 + lx, y = y0 + ly;
        if (x >= W || y >= H) continue;
        const int li = ly * RW + lx;
        const int64_t p = (int64_t)y * W + x;
        const uint8_t t = s_tag[li];
        tag_out[p] = t >= kTagEdge ? 255 : t;
        if (t != 0 && t < kTagEdge) {
            rgb[p] = s_c[0][li];
            rgb[n + p] = s_c[1][li];
            rgb[2 * n + p] = s_c[2][li];
            alpha[p] = s_a[li];
            z[p] = s_z[li];
            cls[p] = (uint8_t)BGS_CLS_GAP;
            ++filled;
        }
        const uint32_t c = t == 255 ? 1u : 0u;
        center[p] = (uint8_t)c;
        centers += c;
    }
    filled = block_sum_u32(filled, s4);
    centers = block_sum_u32(centers, s4);
    if (threadIdx.x == 0) gpart[gb] = make_uint2(filled, centers);
}

// Holes left after interpolation and outside the edge ROIs.
__global__ __launch_bounds__(256) void k_center_mask(int W, int H, const uint8_t* __restrict__ tag,
                                                     uint8_t* __restrict__ center, DevStatus* st) {
    __shared__ uint32_t s4[4];
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    uint32_t count = 0;
    for (int r = threadIdx.x >> 6; r < kBandRows; r += 4) {
        const int y = blockIdx.y * kBandRows + r;
        if (x >= W || y >= H) continue;
        const int64_t p = (int64_t)y * W + x;
        const uint32_t c = (tag[p] == 255 && !in_edge(st, x, y)) ? 1u : 0u;
        center[p] = (uint8_t)c;
        count += c;
    }
    count = block_sum_u32(count, s4);
    if (threadIdx.x == 0 && count) atomicAdd(&st->n_center, count);
}

// ---------------------------------------------------------------------------
// Row fill (center step off): nearest non-hole pixel left and right on the
// row via block max/min scans; the farther candidate wins.  One block/row.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_row_fill(int W, int H, const uint8_t* __restrict__ tag,
                                                  const uint8_t* __restrict__ center, float bg0, float bg1, float bg2,
                                                  float* __restrict__ rgb, float* __restrict__ z,
                                                  float* __restrict__ alpha, uint8_t* __restrict__ cls,
                                                  DevStatus* st) {
    __shared__ int s_left[256], s_right[256];
    const int y = blockIdx.x;
    const int64_t n = (int64_t)W * H;
    const int64_t row = (int64_t)y * W;
    const int chunk = (W + 255) / 256;
    const int xa = threadIdx.x * chunk, xb = min(xa + chunk, W);
    int last = -1, first = INT_MAX;
    for (int x = xa; x < xb; ++x)
        if (tag[row + x] != 255) {
            last = x;
            if (first == INT_MAX) first = x;
        }
    s_left[threadIdx.x] = last;
    s_right[threadIdx.x] = first;
    __syncthreads();
    // Inclusive scans: max from the left, min from the right.
    for (int off = 1; off < 256; off <<= 1) {
        int l = (int)threadIdx.x >= off ? s_left[threadIdx.x - off] : -1;
        int r = (int)threadIdx.x + off < 256 ? s_right[threadIdx.x + off] : INT_MAX;
        __syncthreads();
        s_left[threadIdx.x] = max(s_left[threadIdx.x], l);
        s_right[threadIdx.x] = min(s_right[threadIdx.x], r);
        __syncthreads();
    }
    int left = threadIdx.x > 0 ? s_left[threadIdx.x - 1] : -1;
    const int right_after = threadIdx.x < 255 ? s_right[threadIdx.x + 1] : INT_MAX;
    uint32_t filled = 0;
    // Nearest valid to the right of x inside the chunk, else right_after.
    for (int x = xa; x < xb; ++x) {
        const int64_t p = row + x;
        if (center[p]) {
            int right = right_after;
            for (int xx = x + 1; xx < xb; ++xx)
                if (tag[row + xx] != 255) {
                    right = xx;
                    break;
                }
            int pick = -1;
            if (left >= 0 && right != INT_MAX) pick = z[row + right] > z[row + left] ? right : left;
            else if (left >= 0) pick = left;
            else if (right != INT_MAX) pick = right;
            if (pick >= 0) {
                const int64_t r = row + pick;
                rgb[p] = rgb[r];
                rgb[n + p] = rgb[n + r];
                rgb[2 * n + p] = rgb[2 * n + r];
                z[p] = z[r];
                alpha[p] = alpha[r];
            } else {
                rgb[p] = bg0;
                rgb[n + p] = bg1;
                rgb[2 * n + p] = bg2;
                z[p] = INFINITY;
                alpha[p] = 0.f;
            }
            cls[p] = (uint8_t)BGS_CLS_ROWFILL;
            ++filled;
        }
        if (tag[p] != 255) left = x;
    }
    __shared__ uint32_t s4[4];
    filled = block_sum_u32(filled, s4);
    if (threadIdx.x == 0 && filled) atomicAdd(&st->n_rowfill, filled);
}

// ---------------------------------------------------------------------------
// Connected components: union-find in LDS over tiles of 64x16 pixels, then
// unions across tile borders with global atomicMin, then flattening.  Links
// always go from the larger to the smaller index, so the root of every
// component is its smallest linear index.
//
// The unions, each a chain of dependent reads and an atomic, are what these
// kernels wait for, so they are few: a wave holds a row's 64 pixels as the
// bits of one word, the nodes of a tile are its rows' runs of set pixels,
// and the words say where two adjacent runs first touch.  (A union per
// pixel and neighbour, over 16x16 tiles: 2064x2208 with 16 components, tiles
// 26 -> 16 us, borders 126 -> 15; 1603x1061, 20 -> 9 and 21 -> 8.)
// ---------------------------------------------------------------------------
constexpr int kCclRows = 16;  // rows per tile (64 columns)

// First bit of the run of set bits that holds bit x of w.
__device__ inline int run_start(unsigned long long w, int x) {
    const unsigned long long zeros = ~w & ((1ull << x) - 1ull);
    return zeros ? 64 - __clzll((long long)zeros) : 0;
}

// Where pixels of a row are joined to the row above, one pair of touching
// runs at a time: vertically where the overlap of two runs begins, and, with
// 8 neighbours, diagonally where two runs touch at a corner only (were the
// pixel above or the pixel beside set as well, the runs overlap there).
// The neighbours left and right of the word come in with cl, cr, ul, ur.
struct RowLinks {
    unsigned long long vert, left, right;  // to the pixel above; above left; above right
    __device__ RowLinks(unsigned long long cur, unsigned long long up, int conn, unsigned long long cl = 0,
                        unsigned long long cr = 0, unsigned long long ul = 0, unsigned long long ur = 0) {
        const unsigned long long o = cur & up;
        vert = o & ~(o << 1);
        left = conn == 8 ? cur & ((up << 1) | ul) & ~up & ~((cur << 1) | cl) : 0ull;
        right = conn == 8 ? cur & ((up >> 1) | (ur << 63)) & ~up & ~((cur >> 1) | (cr << 63)) : 0ull;
    }
};

__device__ inline int find_root_lds(int* L, int x) {
    int p = __hip_atomic_load(&L[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (p != x) {
        x = p;
        p = __hip_atomic_load(&L[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return x;
}

// In global memory.  Parents only ever get smaller and every value a node
// has had is an ancestor of it, so a read that another XCD's unions have
// overtaken still leads towards the root: it may come out of this XCD's
// cache (kScope: the scope of the reads).
template <int kScope = __HIP_MEMORY_SCOPE_WORKGROUP>
__device__ inline int find_root_g(const int* L, int x, int* hops = nullptr) {
    int p = __hip_atomic_load(&L[x], __ATOMIC_RELAXED, kScope);
    while (p != x) {
        x = p;
        if (hops) ++*hops;
        p = __hip_atomic_load(&L[x], __ATOMIC_RELAXED, kScope);
    }
    return x;
}

// The same for a union; where the path was long, the next finds from this
// tile's piece (x's parent) go straight to the root.
template <int kScope>
__device__ inline int find_root_union(int* L, int x) {
    const int piece = __hip_atomic_load(&L[x], __ATOMIC_RELAXED, kScope);
    int hops = 0;
    const int r = find_root_g<kScope>(L, piece, &hops);
    if (hops > 1) (void)__hip_atomic_fetch_min(&L[piece], r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return r;
}

// Ends whatever the finds read: the atomic returns the current parent, and
// the larger index strictly falls from round to round.  The first finds may
// read this XCD's cache; one whose root turns out to have a parent is
// repeated past it, or each step of the path since would take an atomic that
// fails (a serpentine of one-pixel lines, 1503x1001: 110-250 -> 65 us in
// all; nothing changes where components are small).
__device__ inline void unite_g(int* L, int a, int b) {
    a = find_root_union<__HIP_MEMORY_SCOPE_WORKGROUP>(L, a);
    b = find_root_union<__HIP_MEMORY_SCOPE_WORKGROUP>(L, b);
    while (a != b) {
        if (a < b) {
            int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(&L[a], b);
        if (old == a) return;
        // a had gained a parent meanwhile; unite that one with b
        a = find_root_union<__HIP_MEMORY_SCOPE_AGENT>(L, old);
        b = find_root_union<__HIP_MEMORY_SCOPE_AGENT>(L, b);
    }
}

__device__ inline void unite_lds(int* L, int a, int b) {
    while (true) {
        a = find_root_lds(L, a);
        b = find_root_lds(L, b);
        if (a == b) return;
        if (a < b) {
            int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(&L[a], b);
        if (old == a) return;
        a = old;
    }
}

// Tile-local labelling.  With pflag/pbox given, it also records every
// tile-local piece (its root pixel gets pflag = 1 and the piece's half-open
// bounding box in pbox), so that component boxes can be formed from pieces
// instead of pixels.
__global__ __launch_bounds__(256) void k_ccl_local(int W, int H, int conn, const uint8_t* __restrict__ mask,
                                                   int* __restrict__ labels, uint8_t* __restrict__ pflag,
                                                   int4* __restrict__ pbox) {
    constexpr int kR = kCclRows / 4;  // rows per wave
    __shared__ unsigned long long s_row[kCclRows];
    __shared__ int L[64 * kCclRows];  // parents of run starts
    __shared__ int bx0[64 * kCclRows], bx1[64 * kCclRows], by1[64 * kCclRows];
    const int lane = threadIdx.x & 63, row0 = (threadIdx.x >> 6) * kR;
    const int x = blockIdx.x * 64 + lane, y = blockIdx.y * kCclRows + row0;
    const int64_t g0 = (int64_t)y * W + x;
    bool set[kR];
#pragma unroll
    for (int q = 0; q < kR; ++q) set[q] = x < W && y + q < H && mask[g0 + (int64_t)q * W];
    unsigned long long w[kR], any = 0;
#pragma unroll
    for (int q = 0; q < kR; ++q) {
        w[q] = __ballot(set[q]);
        any |= w[q];
        if (lane == 0) s_row[row0 + q] = w[q];
    }
    if (!__syncthreads_or(any != 0)) {  // an empty tile (the usual case for a sparse mask)
#pragma unroll
        for (int q = 0; q < kR; ++q)
            if (x < W && y + q < H) {
                labels[g0 + (int64_t)q * W] = -1;
                if (pflag) pflag[g0 + (int64_t)q * W] = 0;
            }
        return;
    }
#pragma unroll
    for (int q = 0; q < kR; ++q) {
        const int li = (row0 + q) * 64 + lane;
        if (((w[q] & ~(w[q] << 1)) >> lane) & 1) {
            L[li] = li;
            bx0[li] = INT_MAX;
            bx1[li] = -1;
            by1[li] = -1;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kR; ++q) {
        const int ly = row0 + q;
        if (ly == 0) continue;
        const unsigned long long up = q > 0 ? w[q > 0 ? q - 1 : 0] : s_row[ly - 1];
        const RowLinks k(w[q], up, conn);
        if (((k.vert | k.left | k.right) >> lane) & 1) {
            const int me = ly * 64 + run_start(w[q], lane), above = (ly - 1) * 64;
            if ((k.vert >> lane) & 1) unite_lds(L, me, above + run_start(up, lane));
            if ((k.left >> lane) & 1) unite_lds(L, me, above + run_start(up, lane - 1));
            if ((k.right >> lane) & 1) unite_lds(L, me, above + run_start(up, lane + 1));
        }
    }
    __syncthreads();
    int root[kR];  // of the run that starts at this lane, then of this lane's run
#pragma unroll
    for (int q = 0; q < kR; ++q) {
        root[q] = -1;
        if (((w[q] & ~(w[q] << 1)) >> lane) & 1) {
            root[q] = find_root_lds(L, (row0 + q) * 64 + lane);
            if (pbox) {
                const unsigned long long after = ~(w[q] >> lane);
                const int len = after ? __ffsll((long long)after) - 1 : 64;
                atomicMin(&bx0[root[q]], lane);
                atomicMax(&bx1[root[q]], lane + len);
                atomicMax(&by1[root[q]], row0 + q + 1);
            }
        }
        root[q] = __shfl(root[q], run_start(w[q], lane), 64);
    }
    __syncthreads();
    const int X = blockIdx.x * 64, Y = blockIdx.y * kCclRows;
#pragma unroll
    for (int q = 0; q < kR; ++q) {
        if (x >= W || y + q >= H) continue;
        const int64_t g = g0 + (int64_t)q * W;
        const int li = (row0 + q) * 64 + lane, r = root[q];
        labels[g] = set[q] ? (Y + (r >> 6)) * W + X + (r & 63) : -1;
        if (pflag) {
            const bool is_root = set[q] && r == li;
            pflag[g] = is_root ? 1 : 0;
            // The root is the piece's first pixel: its row is the box's first.
            if (is_root) pbox[g] = make_int4(X + bx0[li], y + q, X + bx1[li], Y + by1[li]);
        }
    }
}

// Unions across tile borders: a wave per tile, for the tile's first row
// against the row above and its first column against the column before,
// and the corners that its last column shares with the column after.
// What lies inside one tile is joined already, and each tile leaves to its
// neighbours what lies between those.
__global__ __launch_bounds__(256) void k_ccl_border(int W, int H, int conn, int tiles_x, int n_tiles,
                                                    const uint8_t* __restrict__ mask, int* labels) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= n_tiles) return;
    const int ty = t / tiles_x, X = (t - ty * tiles_x) * 64, Y = ty * kCclRows;
    // The two rows; and, in lanes k and 32 + k for k <= kCclRows, row
    // Y - 1 + k of the two columns at the left and at the right border.
    const int x = X + lane, k = lane & 31, yk = Y - 1 + k, xk = lane < 32 ? X - 1 : X + 63;
    const int64_t p = (int64_t)Y * W + x, pk = (int64_t)yk * W + xk;
    const bool on = k <= kCclRows && yk >= 0 && yk < H;
    const uint8_t vc = x < W ? mask[p] : 0, vu = x < W && Y > 0 ? mask[p - W] : 0;
    const uint8_t va = on && xk >= 0 && xk < W ? mask[pk] : 0, vb = on && xk + 1 < W ? mask[pk + 1] : 0;
    const unsigned long long cur = __ballot(vc != 0), up = __ballot(vu != 0);
    const unsigned long long ca = __ballot(va != 0), cb = __ballot(vb != 0);  // bit k: row Y - 1 + k
    const RowLinks r(cur, up, conn, (ca >> 1) & 1, (cb >> 33) & 1, ca & 1, (cb >> 32) & 1);
    if ((r.vert >> lane) & 1) unite_g(labels, (int)p, (int)p - W);
    if ((r.left >> lane) & 1) unite_g(labels, (int)p, (int)p - W - 1);
    if ((r.right >> lane) & 1) unite_g(labels, (int)p, (int)p - W + 1);
    // Columns a | b side by side: joined where both are set, unless both
    // are set in the tile's row above too; corners where only those touch.
    const unsigned long long low = (1ull << kCclRows) - 1ull, rows = low << 1, in = low << 2 & rows;
    const unsigned long long both = ca & cb;
    const unsigned long long side = both & rows & ~((both << 1) & in);
    const unsigned long long dl = conn == 8 ? cb & (ca << 1) & ~(cb << 1) & ~ca & in : 0ull;
    const unsigned long long dr = conn == 8 ? ca & (cb << 1) & ~(ca << 1) & ~cb & (in << 32) : 0ull;
    if ((side >> lane) & 1) unite_g(labels, (int)pk + 1, (int)pk);
    if ((dl >> lane) & 1) unite_g(labels, (int)pk + 1, (int)pk - W);
    if ((dr >> lane) & 1) unite_g(labels, (int)pk, (int)pk - W + 1);
}

__global__ __launch_bounds__(256) void k_ccl_flatten(int64_t n, int* labels) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const int l = labels[p];
    if (l < 0) return;
    labels[p] = find_root_g(labels, l);
}

// ---------------------------------------------------------------------------
// Center boxes.  Component c (in order of root pixel) gets box slot
// n_edge + c.  A component's root is its smallest pixel index, so the
// component roots are the pixels with labels[p] == p; per-block root counts
// (scanned) and root masks give each its slot, so no per-pixel slot map is
// needed.  The box of a component is formed where the box of the piece with
// its root is.
// ---------------------------------------------------------------------------
// One workgroup scans the counts, so they are few: 1024 pixels each.
constexpr int kRootBlock = 1024;

// Widen the box at e by b.  A bound that a read already shows to hold is
// left alone (bounds only ever widen, so one read late holds too): the
// pieces of a large component otherwise wait for each other at its four
// words.
__device__ inline void widen_box(int32_t* e, int4 b) {
    int32_t now[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) now[q] = __hip_atomic_load(&e[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (b.x < now[0]) atomicMin(&e[0], b.x);
    if (b.y < now[1]) atomicMin(&e[1], b.y);
    if (b.z > now[2]) atomicMax(&e[2], b.z);
    if (b.w > now[3]) atomicMax(&e[3], b.w);
}

// Flatten every label to its root (as k_ccl_flatten), widen the box at the
// component's root pixel by those of its other pieces, and record, per block
// of kRootBlock pixels, the mask of component roots and its population.
// (2064x2208: 25 us, and 7 for the boxes' records and tiles; flattening and
// boxes took 10 + 62 + 9 with a kernel of their own for the pieces and every
// piece's four atomics sent.)
__global__ __launch_bounds__(256) void k_ccl_flatten_roots(int64_t n, int* labels, const uint8_t* __restrict__ pflag,
                                                           int4* pbox, uint32_t* __restrict__ bcount,
                                                           unsigned long long* __restrict__ rmask) {
    constexpr int kP = kRootBlock / 256;
    __shared__ uint32_t cnt[4];
    const int64_t p0 = (int64_t)blockIdx.x * kRootBlock + threadIdx.x;
    int l[kP];
#pragma unroll
    for (int q = 0; q < kP; ++q) l[q] = p0 + 256 * q < n ? labels[p0 + 256 * q] : -1;
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < kP; ++q) {
        const int64_t p = p0 + 256 * q;
        const bool root = l[q] >= 0 && l[q] == (int)p;
        if (l[q] >= 0 && !root) {
            const int r = find_root_g(labels, l[q]);
            labels[p] = r;
            if (pflag[p]) widen_box(reinterpret_cast<int32_t*>(pbox + r), pbox[p]);
        }
        const unsigned long long m = __ballot(root);
        // A word per 64 pixels; those past the image have none.
        if ((threadIdx.x & 63) == 0 && p < n) rmask[p >> 6] = m;
        c += (uint32_t)__popcll(m);
    }
    if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) bcount[blockIdx.x] = cnt[0] + cnt[1] + cnt[2] + cnt[3];
}

// One workgroup: the gap-fill counts, an exclusive scan of the nb block
// counts in place (bcount[nb] gets the component count), the box count and
// the capacity flag.
//
// Adds the gap-fill block counts (n_gpart entries) to the status block.  The
// status words are read first and up to four partials per thread are
// loaded together: this runs on one workgroup, where load latency is most
// of the time.
__device__ inline void fold_gap_parts(const uint2* __restrict__ gpart, int n_gpart, DevStatus* st) {
    __shared__ uint32_t s_g[2][16];
    const uint32_t g0 = st->n_gap, c0 = st->n_center;
    uint32_t f = 0u, c = 0u;
    const int nt = (int)blockDim.x;
    for (int i0 = threadIdx.x; i0 < n_gpart; i0 += 4 * nt) {
        uint2 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = i0 + u * nt < n_gpart ? gpart[i0 + u * nt] : make_uint2(0u, 0u);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            f += q[u].x;
            c += q[u].y;
        }
    }
    f = wave_sum_u32(f);
    c = wave_sum_u32(c);
    if ((threadIdx.x & 63) == 0) {
        s_g[0][threadIdx.x >> 6] = f;
        s_g[1][threadIdx.x >> 6] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tf = 0u, tc = 0u;
        for (int w = 0; w < nt / 64; ++w) {
            tf += s_g[0][w];
            tc += s_g[1][w];
        }
        st->n_gap = g0 + tf;
        st->n_center = c0 + tc;
    }
}

// Block counts up to kRootLds are staged in LDS with coalesced loads (all
// issued together), scanned there and written back coalesced; larger
// images walk per-thread chunks in global memory.
constexpr int kRootLds = 16384;

__global__ __launch_bounds__(1024) void k_root_scan(int64_t nb, uint32_t* bcount, int box_cap,
                                                    int32_t* __restrict__ n_boxes, const uint2* __restrict__ gpart,
                                                    int n_gpart, DevStatus* st) {
    __shared__ uint32_t s_cnt[kRootLds];
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n_edge = st->n_edge;
    const bool staged = nb <= kRootLds;
    if (staged) {
        constexpr int kU = kRootLds / 1024;
        uint32_t v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = tid + 1024 * u < nb ? bcount[tid + 1024 * u] : 0u;
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (tid + 1024 * u < nb) s_cnt[tid + 1024 * u] = v[u];
    }
    fold_gap_parts(gpart, n_gpart, st);  // its barrier also publishes s_cnt
    const int64_t per = (nb + 1023) / 1024;
    const int64_t b0 = min(nb, (int64_t)tid * per), b1 = min(nb, b0 + per);
    uint32_t sum = 0;
    if (staged)
        for (int64_t b = b0; b < b1; ++b) sum += s_cnt[b];
    else
        for (int64_t b = b0; b < b1; ++b) sum += bcount[b];
    // Exclusive scan of the 1024 chunk sums: within each wave by shuffles,
    // then over the 16 wave totals.
    uint32_t x = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t run = x - sum, total = 0;
    for (int w = 0; w < 16; ++w) {
        const uint32_t ws = wsum[w];
        if (w < wave) run += ws;
        total += ws;
    }
    if (staged) {
        for (int64_t b = b0; b < b1; ++b) {
            const uint32_t c = s_cnt[b];
            s_cnt[b] = run;
            run += c;
        }
        __syncthreads();
        for (int64_t b = tid; b < nb; b += 1024) bcount[b] = s_cnt[b];
    } else {
        for (int64_t b = b0; b < b1; ++b) {
            const uint32_t c = bcount[b];
            bcount[b] = run;
            run += c;
        }
    }
    if (tid == 0) {
        bcount[nb] = total;
        const uint32_t tot = n_edge + total;
        st->n_boxes = tot;
        if ((int64_t)tot > box_cap) atomicOr(&st->overflow, 2u);
        *n_boxes = (int32_t)tot;
    }
}

// The components whose roots lie in this block's kRootBlock pixels, a wave per
// component in turn (large boxes: all four): margin, clip, tile alignment, the box record, and its tiles in
// the mask.
__global__ __launch_bounds__(256) void k_center_boxes(int W, int H, int margin, int T, int tiles_x,
                                                      const uint32_t* __restrict__ boff,
                                                      const unsigned long long* __restrict__ rmask,
                                                      const int4* __restrict__ pbox, bgs_box* __restrict__ boxes,
                                                      int box_cap, uint8_t* tm, const DevStatus* st) {
    constexpr int kWords = kRootBlock / 64;
    const uint32_t c0 = boff[blockIdx.x], c1 = boff[blockIdx.x + 1];
    if (c0 == c1) return;
    int word = blockIdx.x * kWords;
    unsigned long long left = rmask[word];
    for (uint32_t c = c0; c < c1; ++c) {
        while (left == 0) left = rmask[++word];  // the block's masks hold c1 - c0 roots
        const int root = 64 * word + __ffsll((long long)left) - 1;
        left &= left - 1;
        const bool mine = ((c - c0) & 3u) == threadIdx.x >> 6;
        const int lane = threadIdx.x & 63;
        const int4 e = pbox[root];
        int64_t x0 = e.x - margin, y0 = e.y - margin;
        int64_t x1 = (int64_t)e.z + margin, y1 = (int64_t)e.w + margin;
        if (x0 < 0) x0 = 0;
        if (y0 < 0) y0 = 0;
        if (x1 > W) x1 = W;
        if (y1 > H) y1 = H;
        x0 = align_down(x0, T);
        y0 = align_down(y0, T);
        x1 = align_up(x1, T);
        y1 = align_up(y1, T);
        if (x1 > W) x1 = W;
        if (y1 > H) y1 = H;
        if (mine && lane == 0) {
            const int64_t slot = (int64_t)st->n_edge + c;
            if (slot < box_cap) {
                boxes[slot].x0 = (int32_t)x0;
                boxes[slot].y0 = (int32_t)y0;
                boxes[slot].x1 = (int32_t)x1;
                boxes[slot].y1 = (int32_t)y1;
                boxes[slot].kind = BGS_BOX_CENTER;
                boxes[slot].label = root;
            }
        }
        const int tx0 = (int)(x0 / T), ty0 = (int)(y0 / T);
        const int bw = (int)((x1 + T - 1) / T) - tx0, bh = (int)((y1 + T - 1) / T) - ty0;
        const bool large = bw * bh > 1024;
        if (!mine && !large) continue;
        for (int q = large ? (int)threadIdx.x : lane; q < bw * bh; q += large ? 256 : 64) {
            const int r = q / bw;
            tm[(int64_t)(ty0 + r) * tiles_x + tx0 + q - r * bw] = 1;
        }
    }
}

// Box count without center ROIs: the edge boxes only.  256 threads.
__global__ __launch_bounds__(256) void k_box_count(int box_cap, int32_t* n_boxes, const uint2* __restrict__ gpart,
                                                   int n_gpart, DevStatus* st) {
    fold_gap_parts(gpart, n_gpart, st);
    if (threadIdx.x != 0) return;
    const uint32_t tot = st->n_edge;
    st->n_boxes = tot;
    if ((int64_t)tot > box_cap) st->overflow |= 2u;
    *n_boxes = (int32_t)tot;
}

__global__ __launch_bounds__(256) void k_fill_i32(int64_t n, int32_t* p, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

inline unsigned grid(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// True when every splat provably stays on its source row: same row count,
// same fy and cy, and the fp64 bound on |v - j| over the image for any valid
// depth is below a quarter pixel.  With M = I + E (|E| <= eps) and a point
// at depth d >= d_lo, v - j = fy (num / den) with
// |num| <= g + |c1|/d_lo + |yn| (g + |c2|/d_lo), den >= 1 - g - |c2|/d_lo,
// g = eps (|xn| + |yn| + 1); valid splats need Z' > z_near, hence d_lo.
static bool rows_preserved(const WarpCam& src, const WarpCam& dst, const RelPose& P) {
    if (src.H != dst.H || src.fy != dst.fy || src.cy != dst.cy || dst.W > 8192) return false;
    double eps = 0.0;
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q) eps = fmax(eps, fabs(P.M[r * 3 + q] - (r == q ? 1.0 : 0.0)));
    const double xn = fmax(fabs(0.0 - src.cx), fabs((src.W - 1.0) - src.cx)) / src.fx;
    const double yn = fmax(fabs(0.0 - src.cy), fabs((src.H - 1.0) - src.cy)) / src.fy;
    const double g = eps * (xn + yn + 1.0);
    const double d_lo = (dst.z_near - fabs(P.c[2])) / (1.0 + g);
    if (!(d_lo > 0.0)) return false;
    const double c1 = fabs(P.c[1]) / d_lo, c2 = fabs(P.c[2]) / d_lo;
    const double den = 1.0 - g - c2;
    if (!(den > 0.5)) return false;
    const double bound = dst.fy * (g + c1 + yn * (g + c2)) / den + 1e-9 * (dst.H + 1.0);
    return bound < 0.25;
}

int warp_parts(const WarpCam& src, const WarpCam& dst, const RelPose& P) {
    return rows_preserved(src, dst, P) ? dst.H : 0;
}

hipError_t launch_reproject(const WarpCam& src, const WarpCam& dst, const RelPose& P, float a_min, const float* rgb,
                            const float* draw, const float* alpha, unsigned long long* zbuf, float* rgb_dst,
                            float* z_dst, float* alpha_dst, uint8_t* hole, float* depth_range, bool reset,
                            uint4* wpart, DevStatus* st, hipStream_t s) {
    const int64_t ns = (int64_t)src.W * src.H, nd = (int64_t)dst.W * dst.H;
    if (reset) hipLaunchKernelGGL(k_warp_reset, dim3(1), dim3(1), 0, s, st);
    if (rows_preserved(src, dst, P)) {
        // Staging pays on long rows (1600 pixels: 20.6 -> 19.5 us); on short
        // ones the larger LDS footprint costs more than the gathers it saves
        // (800 pixels: 8.2 -> 9.0 us).
        const size_t zb = sizeof(unsigned long long) * dst.W, sb = zb + 4 * sizeof(float) * src.W;
        if (src.W >= kRowStageMinW && sb <= (size_t)kRowStageLds)
            hipLaunchKernelGGL((k_reproject_rows<kRowThreads, kRowItems, true>), dim3(dst.H), dim3(kRowThreads), sb, s,
                               src, dst, P, a_min, draw, alpha, rgb, rgb_dst, z_dst, alpha_dst, hole, wpart);
        else
            hipLaunchKernelGGL((k_reproject_rows<kRowThreads, kRowItems, false>), dim3(dst.H), dim3(kRowThreads), zb,
                               s, src, dst, P, a_min, draw, alpha, rgb, rgb_dst, z_dst, alpha_dst, hole, wpart);
    } else {
        hipLaunchKernelGGL(k_fill_u64, dim3(grid(nd)), dim3(256), 0, s, zbuf, nd, ~0ull);
        hipLaunchKernelGGL(k_reproject_scatter, band_grid(src.W, src.H), dim3(256), 0, s, src, dst, P, a_min, draw,
                           alpha, zbuf, st);
        hipLaunchKernelGGL(k_reproject_resolve, dim3((unsigned)((nd + 4095) / 4096)), dim3(1024), 0, s, nd, ns, zbuf, rgb,
                           alpha, rgb_dst, z_dst, alpha_dst, hole, st);
    }
    if (depth_range)
        hipLaunchKernelGGL(k_warp_finish, dim3(1), dim3(256), 0, s, wpart, warp_parts(src, dst, P), st,
                           (float)src.z_near, (float)src.z_far, depth_range);
    return hipGetLastError();
}

// Tile-local labels and the unions across tile borders, unflattened.
static void launch_ccl_tiles(const uint8_t* mask, int W, int H, int conn, int32_t* labels, uint8_t* pflag, int4* pbox,
                             hipStream_t s) {
    const int tx = (W + 63) / 64, ty = (H + kCclRows - 1) / kCclRows;
    hipLaunchKernelGGL(k_ccl_local, dim3(tx, ty), dim3(256), 0, s, W, H, conn, mask, labels, pflag, pbox);
    hipLaunchKernelGGL(k_ccl_border, dim3((tx * ty + 3) / 4), dim3(256), 0, s, W, H, conn, tx, tx * ty, mask, labels);
}

hipError_t launch_label_components(const uint8_t* mask, int W, int H, int conn, int32_t* labels, hipStream_t s) {
    const int64_t n = (int64_t)W * H;
    if (n == 0) return hipSuccess;
    launch_ccl_tiles(mask, W, H, conn, labels, nullptr, nullptr, s);
    hipLaunchKernelGGL(k_ccl_flatten, dim3(grid(n)), dim3(256), 0, s, n, labels);
    return hipGetLastError();
}

hipError_t launch_classify(const WarpCam& src, const WarpCam& dst, const RelPose& P, const bgs_roi_params& roi,
                           const float bg[3], const float* depth_range, float* rgb, float* z, float* alpha,
                           uint8_t* cls, int32_t* labels, bgs_box* boxes, int32_t box_cap, int32_t* n_boxes,
                           uint8_t* tile_mask, const ClassifyBufs& b, DevStatus* st, hipStream_t s) {
    const int W = dst.W, H = dst.H, T = roi.tile;
    const int64_t n = (int64_t)W * H;
    const int tiles_x = (W + T - 1) / T, tiles_y = (H + T - 1) / T;
    const bool fused = roi.gap_passes <= kGapMaxHalo;  // k_gap_fill writes the edge tiles of the mask
    hipLaunchKernelGGL(k_edge_rois, dim3(1), dim3(256), 0, s, src, dst, P, roi.edge_samples, roi.margin, T,
                       roi.edge_bounds, depth_range, b.wpart, depth_range ? 0 : warp_parts(src, dst, P), st, boxes, box_cap,
                       fused ? nullptr : tile_mask);
    const dim3 gg = band_grid(W, H);
    int n_gpart = 0;
    uint8_t* tag = b.hole;
    uint8_t* center = b.hole2;
    if (fused) {
        const dim3 g1(gg.x * gg.y);
        if (roi.gap_passes <= 2)
            hipLaunchKernelGGL(k_gap_fill<2>, g1, dim3(256), 0, s, W, H, roi.gap_passes, rgb, z, alpha, tag, cls,
                               center, st, b.gpart, T, tiles_x, tiles_y, tile_mask);
        else
            hipLaunchKernelGGL(k_gap_fill<kGapMaxHalo>, g1, dim3(256), 0, s, W, H, roi.gap_passes, rgb, z, alpha, tag,
                               cls, center, st, b.gpart, T, tiles_x, tiles_y, tile_mask);
        n_gpart = (int)(gg.x * gg.y);
    } else {
        hipLaunchKernelGGL(k_tag_init, dim3(grid(n)), dim3(256), 0, s, n, cls, tag);
        for (int pass = 1; pass <= roi.gap_passes; ++pass)
            hipLaunchKernelGGL(k_gap_pass, band_grid(W, H), dim3(256), 0, s, W, H, pass, rgb, z, alpha, tag, cls, st);
        hipLaunchKernelGGL(k_center_mask, band_grid(W, H), dim3(256), 0, s, W, H, tag, center, st);
    }
    if (roi.center_roi) {
        const int64_t nb = (n + kRootBlock - 1) / kRootBlock;
        launch_ccl_tiles(center, W, H, 8, labels, b.pflag, b.pbox, s);
        hipLaunchKernelGGL(k_ccl_flatten_roots, dim3((unsigned)nb), dim3(256), 0, s, n, labels, b.pflag, b.pbox, b.bcount,
                           b.rmask);
        hipLaunchKernelGGL(k_root_scan, dim3(1), dim3(1024), 0, s, nb, b.bcount, box_cap, n_boxes, b.gpart, n_gpart,
                           st);
        hipLaunchKernelGGL(k_center_boxes, dim3((unsigned)nb), dim3(256), 0, s, W, H, roi.margin, T, tiles_x, b.bcount,
                           b.rmask, b.pbox, boxes, box_cap, tile_mask, st);
    } else {
        hipLaunchKernelGGL(k_fill_i32, dim3(grid(n)), dim3(256), 0, s, n, labels, -1);
        hipLaunchKernelGGL(k_row_fill, dim3(H), dim3(256), 0, s, W, H, tag, center, bg[0], bg[1], bg[2], rgb, z, alpha,
                           cls, st);
        hipLaunchKernelGGL(k_box_count, dim3(1), dim3(256), 0, s, box_cap, n_boxes, b.gpart, n_gpart, st);
    }
    return hipGetLastError();
}

}  // namespace bgs
