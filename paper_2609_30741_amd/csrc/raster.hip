// 2DGS tile rasteriser for gfx950: per-surfel preprocess, binning of the
// depth-ordered surfels into tile lists and front-to-back blending with
// the joint depth proxy (Sec. 3.1 Stage 1, Sec. 3.3 Eq. 1-2).
#include <cmath>

#include <algorithm>
#include <climits>

#include "bgs_internal.h"

namespace bgs {

namespace {

// ---------------------------------------------------------------------------
// Preprocess: one thread per surfel.
// ---------------------------------------------------------------------------

// Compositing-order key: fp32 centre depth with one fixed operation order,
// ((r20*px + r21*py) + r22*pz) + tz, every operation rounded separately.
__device__ inline float centre_depth_key(const float zc[4], float px, float py, float pz) {
#pragma clang fp contract(off)
    float a = zc[0] * px;
    float b = zc[1] * py;
    float s = a + b;
    float c = zc[2] * pz;
    s = s + c;
    return s + zc[3];
}

// Real spherical harmonics (Condon-Shortley phase) in Cartesian form for a
// unit direction; the constants are sqrt((2l+1)/(4 pi) (l-m)!/(l+m)!)
// (times sqrt(2) for m != 0) folded with the polynomial normalisation.
__device__ inline void sh_basis(int deg, float x, float y, float z, float* Y) {
    Y[0] = 0.28209479177387814f;
    if (deg < 1) return;
    const float c1 = 0.4886025119029199f;
    Y[1] = -c1 * y;
    Y[2] = c1 * z;
    Y[3] = -c1 * x;
    if (deg < 2) return;
    const float xx = x * x, yy = y * y, zz = z * z;
    Y[4] = 1.0925484305920792f * x * y;
    Y[5] = -1.0925484305920792f * y * z;
    Y[6] = 0.31539156525252005f * (2.f * zz - xx - yy);
    Y[7] = -1.0925484305920792f * x * z;
    Y[8] = 0.5462742152960396f * (xx - yy);
    if (deg < 3) return;
    Y[9] = -0.5900435899266435f * y * (3.f * xx - yy);
    Y[10] = 2.890611442640554f * x * y * z;
    Y[11] = -0.4570457994644658f * y * (4.f * zz - xx - yy);
    Y[12] = 0.3731763325901154f * z * (2.f * zz - 3.f * xx - 3.f * yy);
    Y[13] = -0.4570457994644658f * x * (4.f * zz - xx - yy);
    Y[14] = 1.445305721320277f * z * (xx - yy);
    Y[15] = -0.5900435899266435f * x * (xx - 3.f * yy);
}

// ---------------------------------------------------------------------------
// Strip band of a surfel: a direction n (snorm16 pair) and an interval
// [n.mu + c - w, n.mu + c + w] (fp16 c, w) of n.x that holds every pixel x
// the surfel can reach with alpha >= alpha_min.  The blend skips a record
// for a wave's 8x8 pixel region that lies outside the band, which is exact:
// such a record is a no-op on every pixel of the region.  n is the
// footprint's narrowest direction when that confines the regions of a tile
// column better than the y extent, else the y axis.  The band is computed
// for the quantised n the blend decodes, and padded for the fp16 rounding
// and for the blend's fp32 arithmetic.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float snorm16_value(int q) { return (float)q * (1.0f / 32767.0f); }

__device__ __forceinline__ uint32_t half_bits(float x) {
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x);
}

__device__ __forceinline__ float half_value(uint32_t bits) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(bits & 0xFFFFu));
}

// Smallest fp16 value >= x (x >= 0), +inf beyond the fp16 range.
__device__ __forceinline__ uint32_t half_bits_up(double x) {
    if (!(x <= 65504.0)) return 0x7C00u;
    uint32_t h = half_bits((float)x);
    while ((double)half_value(h) < x) ++h;
    return h;
}

// Interval of n.x over the conic's outline (dual conic C in normalised
// camera coordinates) for a pixel-space direction n: the tangent lines
// n.x = s solve m^T C2 m - 2 s' m.c3 + s'^2 c22 = 0 with m = (fx nx, fy ny)
// and s = s' + n.(cx, cy).
__device__ __forceinline__ void conic_extent(double nx, double ny, double c00, double c01, double c02, double c11,
                                             double c12, double c22, const PreCam& cam, double& lo, double& hi) {
    const double mx = cam.fx * nx, my = cam.fy * ny;
    const double mc = mx * c02 + my * c12;
    const double mm = mx * mx * c00 + 2.0 * mx * my * c01 + my * my * c11;
    const double d = sqrt(fmax(mc * mc - c22 * mm, 0.0));
    const double s0 = (mc - d) / c22, s1 = (mc + d) / c22;
    const double off = nx * cam.cx + ny * cam.cy;
    lo = fmin(s0, s1) + off;
    hi = fmax(s0, s1) + off;
}

__device__ uint2 strip_band(bool bounded, double c00, double c01, double c02, double c11, double c12, double c22,
                            const PreCam& cam, double mux, double muy, double r_lowpass, double xmin, double xmax,
                            double ymin, double ymax) {
    int qx = 0, qy = 32767;
    if (bounded) {
        // Narrowest direction: smallest eigenvector of F (c3 c3^T - c22 C2) F.
        const double s00 = cam.fx * cam.fx * (c02 * c02 - c22 * c00);
        const double s11 = cam.fy * cam.fy * (c12 * c12 - c22 * c11);
        const double s01 = cam.fx * cam.fy * (c02 * c12 - c22 * c01);
        const double h = 0.5 * (s00 - s11);
        const double lmin = 0.5 * (s00 + s11) - sqrt(h * h + s01 * s01);
        double ex = s01, ey = lmin - s00;
        const double fx2 = lmin - s11, fy2 = s01;
        if (fx2 * fx2 + fy2 * fy2 > ex * ex + ey * ey) {
            ex = fx2;
            ey = fy2;
        }
        const double en = sqrt(ex * ex + ey * ey);
        if (en > 0.0 && isfinite(en)) {
            ex /= en;
            ey /= en;
            if (ey < 0.0) {
                ex = -ex;
                ey = -ey;
            }
            const int cx = (int)rint(ex * 32767.0), cy = (int)rint(ey * 32767.0);
            const double nx = snorm16_value(cx), ny = snorm16_value(cy);
            double lo, hi;
            conic_extent(nx, ny, c00, c01, c02, c11, c12, c22, cam, lo, hi);
            const double nmu = nx * mux + ny * muy, rn = r_lowpass * sqrt(nx * nx + ny * ny);
            lo = fmin(lo, nmu - rn);
            hi = fmax(hi, nmu + rn);
            // Half-length of the rows of one tile column whose 8x8 regions
            // pass, along n and along y.
            const double pass_n = ny > 1e-6 ? (0.5 * (hi - lo) + 3.5 * fabs(nx) + 3.5 * ny) / ny : INFINITY;
            const double pass_y = 0.5 * (ymax - ymin) + 3.5;
            if (pass_n < pass_y) {
                qx = cx;
                qy = cy;
            }
        }
    }
    const double nx = snorm16_value(qx), ny = snorm16_value(qy);
    double lo, hi;
    if (!bounded) {
        lo = -INFINITY;
        hi = INFINITY;
    } else if (qx == 0 && qy == 32767) {
        lo = ny * ymin;  // ymin/ymax already hold the low-pass disc
        hi = ny * ymax;
    } else {
        conic_extent(nx, ny, c00, c01, c02, c11, c12, c22, cam, lo, hi);
        const double nmu = nx * mux + ny * muy, rn = r_lowpass * sqrt(nx * nx + ny * ny);
        lo = fmin(lo, nmu - rn);
        hi = fmax(hi, nmu + rn);
    }
    const uint32_t nbits = ((uint32_t)qx & 0xFFFFu) | ((uint32_t)qy << 16);
    if (!(isfinite(lo) && isfinite(hi))) return make_uint2(nbits, 0u | (0x7C00u << 16));
    const double nmu = nx * (double)(float)mux + ny * (double)(float)muy;
    const double c = 0.5 * (lo + hi) - nmu;
    const uint32_t cb = half_bits((float)c);
    const double rx = fmax(fabs(xmin - mux), fabs(xmax - mux)), ry = fmax(fabs(ymin - muy), fabs(ymax - muy));
    const double pad = 0.05 + 1e-6 * (fabs(mux) + fabs(muy) + sqrt(rx * rx + ry * ry) + cam.W + cam.H) +
                       fabs(nmu - (nx * mux + ny * muy));
    const double w = 0.5 * (hi - lo) + fabs(c - (double)half_value(cb)) + pad;
    return make_uint2(nbits, cb | (half_bits_up(w) << 16));
}


// ---------------------------------------------------------------------------
// Tile binning by band: of row ty of a surfel's tile rect, the columns
// [*a, *b] (empty when *b < *a) whose 16x16 tile meets the record's strip
// band.  A tile that misses the band is missed by every pixel region in it,
// so the record is a no-op there and needs no key.  fp64, from the record's
// own (fp32 centre, snorm16 direction, fp16 interval) values, with half a
// pixel of margin: the preprocess, the masked counts and the emission call
// this one function on the same values, so counts and keys agree exactly.
// ---------------------------------------------------------------------------
struct BandRows {
    // k(ty) = k0 + k16 ty; columns where |16 nx tx + k| <= r.  r has the sign
    // of nx, so that the interval's ends come out in order; inv = 1 / (16 nx),
    // or 0 where nx = 0 (or no direction): whole rows in or out.
    double k0, k16, r, inv;
    __device__ BandRows() : k0(0.0), k16(0.0), r(-1.0), inv(0.0) {}  // no tile
    __device__ BandRows(double k0, double k16, double r, double inv) : k0(k0), k16(k16), r(r), inv(inv) {}
    __device__ explicit BandRows(const SurfelRec& rec)
        : BandRows(rec.a.x, rec.a.y, __float_as_uint(rec.c.w), __float_as_uint(rec.d.w)) {}
    __device__ BandRows(float mux, float muy, uint32_t nq, uint32_t bq) {
#pragma clang fp contract(off)
        const double nx = (double)snorm16_value((int)(int16_t)(nq & 0xFFFFu));
        const double ny = (double)snorm16_value((int)(int16_t)(nq >> 16));
        const double c = (double)half_value(bq);
        r = (double)half_value(bq >> 16) + 7.5 * (fabs(nx) + fabs(ny)) + 0.5;
        k0 = nx * (7.5 - (double)mux) + ny * (7.5 - (double)muy) - c;
        k16 = 16.0 * ny;
        inv = !(fabs(nx) > 1e-9) ? 0.0 : 1.0 / (16.0 * nx);
        if (inv < 0.0) r = -r;
    }
};

// The same, prepared for the rows of one surfel's rect.  Rows are where the
// counting and the emission spend their time (vector instructions, in fp64),
// so there is one path for both kinds of bands, without branches: a whole
// row's interval is [0, kFar], or a row out of the band (|k| > rv).  (1.2M
// surfels at 1920x1080: counting 78 -> 68 us, emission 90 -> 77; with the
// wave scans by DPP 64 and 74.)
struct BandRect {
    static constexpr double kFar = 1e9;
    double k0, k16, r, inv, rv, far, x0, x1;
    __device__ BandRect(const BandRows& b, int tx0, int tx1) : k0(b.k0), k16(b.k16), r(b.r), inv(b.inv) {
        const bool whole = inv == 0.0;  // also an infinite band (r = inf): every column
        rv = whole ? r : INFINITY;
        far = whole ? kFar : 0.0;
        x0 = (double)tx0;
        x1 = (double)tx1;
    }
    // Columns [*a, *b] of row ty; empty when *b < *a, or when false.
    __device__ bool row(int ty, int* a, int* b) const {
#pragma clang fp contract(off)
        const double k = fma(k16, (double)ty, k0);
        const double lo = (-r - k) * inv, hi = (r - k) * inv + far;
        // (An infinite whole row's ends are NaN, which fmax and fmin pass over.)
        *a = (int)fmin(fmax(ceil(lo), x0), x1 + 1.0);
        *b = (int)fmax(fmin(floor(hi), x1), x0 - 1.0);
        return !(fabs(k) > rv);
    }
};

// Tiles of a surfel's rect that its band meets.
__device__ inline uint32_t band_count(const BandRows& br, int tx0, int ty0, int tx1, int ty1) {
    uint32_t cnt = 0;
    const BandRect rect(br, tx0, tx1);
    for (int y = ty0; y <= ty1; ++y) {
        int a, b;
        if (rect.row(y, &a, &b) && b >= a) cnt += (uint32_t)(b - a + 1);
    }
    return cnt;
}

// The band's tiles in cell row cr (tile rows 8 cr .. 8 cr + 7) of a surfel's
// rect: f(cx, m) for every cell cx of the row from the first tile to the
// last, m the cell's tiles as a mask (bit 8 (row & 7) + (column & 7)), which
// may be empty.
template <typename F>
__device__ inline void cell_masks(const BandRows& br, int tx0, int ty0, int tx1, int ty1, int cr, F&& f) {
    constexpr int kNone = 1 << 14;  // an empty row: [kNone, kNone), past every column
    const BandRect rect(br, tx0, tx1);
    int a[8], e[8], lo = kNone, hi = -1;  // columns [a, e)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int y = 8 * cr + u;
        int b;
        const bool ok = rect.row(y, &a[u], &b) && y >= ty0 && y <= ty1 && b >= a[u];
        a[u] = ok ? a[u] : kNone;
        e[u] = ok ? b + 1 : kNone;
        lo = min(lo, a[u]);
        hi = max(hi, ok ? b : -1);
    }
    if (hi < 0) return;
    for (int cx = lo >> 3; cx <= hi >> 3; ++cx) {
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int s = min(max(a[u] - 8 * cx, 0), 8), t = min(max(e[u] - 8 * cx, 0), 8);  // s <= t
            w[u >> 2] |= ((1u << t) - (1u << s)) << (8 * (u & 3));
        }
        f(cx, (uint64_t)w[0] | ((uint64_t)w[1] << 32));
    }
}

// A surfel seen from one camera: its tile rect and every record word but
// the colour (geometry in fp64, Sec. 3.3).  drawn = false: no pixel of this
// camera can get alpha >= alpha_min from it.
struct SurfelView {
    bool drawn;
    int tx0, ty0, tx1, ty1;
    SurfelRec rec;  // rec.d.xyz (colour) left for the caller
};

__device__ __forceinline__ void surfel_view(const PreCam& cam, float px, float py, float pz, float op,
                                            const double tu[3], const double tv[3], double su, double sv,
                                            float alpha_min, int lowpass, SurfelView& v) {
    v.drawn = false;
    // ---- geometry in fp64 ----
    const double d0 = (double)px - cam.t[0], d1 = (double)py - cam.t[1], d2 = (double)pz - cam.t[2];
    double pc[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) pc[r] = cam.Rt[r * 3 + 0] * d0 + cam.Rt[r * 3 + 1] * d1 + cam.Rt[r * 3 + 2] * d2;
    double a[3], b[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        a[r] = cam.Rt[r * 3 + 0] * tu[0] + cam.Rt[r * 3 + 1] * tu[1] + cam.Rt[r * 3 + 2] * tu[2];
        b[r] = cam.Rt[r * 3 + 0] * tv[0] + cam.Rt[r * 3 + 1] * tv[1] + cam.Rt[r * 3 + 2] * tv[2];
    }
    const double nv[3] = {a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]};
    const double pzc = pc[2];
    const double mux = cam.fx * pc[0] / pzc + cam.cx;
    const double muy = cam.fy * pc[1] / pzc + cam.cy;

    // ---- conservative pixel bounds of {alpha >= alpha_min} ----
    // Surfel term: the disc u^2+v^2 <= 2 ln(o/alpha_min) of the surfel plane;
    // its outline E(t) = p + cos t A + sin t B projects to a conic whose
    // dual is A A^T + B B^T - p p^T, giving the extreme tangent lines
    // directly.  If the disc reaches z <= 0 the bound is the whole screen.
    const double lr = log((double)op / (double)alpha_min);
    const double rho = sqrt(2.0 * lr) * (1.0 + 1e-5);
    double xmin = INFINITY, xmax = -INFINITY, ymin = INFINITY, ymax = -INFINITY;
    bool bounded = false;
    double c00 = 0, c01 = 0, c02 = 0, c11 = 0, c12 = 0, c22 = -1;
    {
        const double A[3] = {rho * su * a[0], rho * su * a[1], rho * su * a[2]};
        const double B[3] = {rho * sv * b[0], rho * sv * b[1], rho * sv * b[2]};
        const double zr2 = A[2] * A[2] + B[2] * B[2];
        if (pzc > 0.0 && pzc * pzc > zr2 * (1.0 + 1e-6) + 1e-12) {
            bounded = true;
            c22 = zr2 - pzc * pzc;
            c00 = A[0] * A[0] + B[0] * B[0] - pc[0] * pc[0];
            c01 = A[0] * A[1] + B[0] * B[1] - pc[0] * pc[1];
            c02 = A[0] * A[2] + B[0] * B[2] - pc[0] * pzc;
            c11 = A[1] * A[1] + B[1] * B[1] - pc[1] * pc[1];
            c12 = A[1] * A[2] + B[1] * B[2] - pc[1] * pzc;
            const double dx = sqrt(fmax(c02 * c02 - c00 * c22, 0.0));
            const double dy = sqrt(fmax(c12 * c12 - c11 * c22, 0.0));
            const double kx0 = (c02 - dx) / c22, kx1 = (c02 + dx) / c22;
            const double ky0 = (c12 - dy) / c22, ky1 = (c12 + dy) / c22;
            xmin = cam.fx * fmin(kx0, kx1) + cam.cx;
            xmax = cam.fx * fmax(kx0, kx1) + cam.cx;
            ymin = cam.fy * fmin(ky0, ky1) + cam.cy;
            ymax = cam.fy * fmax(ky0, ky1) + cam.cy;
        } else {
            xmin = -INFINITY;
            xmax = INFINITY;
            ymin = -INFINITY;
            ymax = INFINITY;
        }
    }
    // Low-pass term: exp(-|x - mu|^2) >= alpha_min / o on a disc around mu.
    if (lowpass) {
        const double r2 = sqrt(lr) * (1.0 + 1e-5);
        xmin = fmin(xmin, mux - r2);
        xmax = fmax(xmax, mux + r2);
        ymin = fmin(ymin, muy - r2);
        ymax = fmax(ymax, muy + r2);
    }
    const double padx = 0.02 + 1e-7 * (fabs(xmin) + fabs(xmax));
    const double pady = 0.02 + 1e-7 * (fabs(ymin) + fabs(ymax));
    const double fx0 = fmax(ceil(xmin - padx), 0.0), fx1 = fmin(floor(xmax + padx), (double)(cam.W - 1));
    const double fy0 = fmax(ceil(ymin - pady), 0.0), fy1 = fmin(floor(ymax + pady), (double)(cam.H - 1));
    if (!(fx0 <= fx1 && fy0 <= fy1)) return;
    const int x0 = (int)fx0, x1 = (int)fx1, y0 = (int)fy0, y1 = (int)fy1;
    const uint2 band = strip_band(bounded, c00, c01, c02, c11, c12, c22, cam, mux, muy,
                                  lowpass ? sqrt(lr) * (1.0 + 1e-5) : 0.0, xmin, xmax, ymin, ymax);
    v.tx0 = x0 / kTile;
    v.tx1 = x1 / kTile;
    v.ty0 = y0 / kTile;
    v.ty1 = y1 / kTile;
    v.drawn = true;

    // ---- plane-to-screen homography centred at the projected centre ----
    // With r_c = p/p_z and delta = ((i-mu_x)/fx, (j-mu_y)/fy, 0) the pixel
    // ray is r = r_c + delta; the plane n.X = n.p meets it at
    // lambda = p_z / (1 + n.delta / n.r_c), and the in-plane coordinates
    // u = (lambda r - p).t_u / s_u, v likewise, reduce to ratios of linear
    // forms in (dx, dy): the form stays well conditioned near the centre.
    float C1 = 0.f, C2 = 0.f, D1 = 0.f, D2 = 0.f, N1 = 0.f, N2 = 0.f, lam_num = -1.f;
    {
        const double np = nv[0] * pc[0] + nv[1] * pc[1] + nv[2] * pc[2];
        const double nn = sqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
        const double pn = sqrt(pc[0] * pc[0] + pc[1] * pc[1] + pc[2] * pc[2]);
        if (fabs(np) > 1e-12 * nn * pn) {
            const double nrc = np / pzc;
            const double as[3] = {a[0] / su, a[1] / su, a[2] / su};
            const double bs[3] = {b[0] / sv, b[1] / sv, b[2] / sv};
            const double pa = pc[0] * as[0] + pc[1] * as[1] + pc[2] * as[2];
            const double pb = pc[0] * bs[0] + pc[1] * bs[1] + pc[2] * bs[2];
            const double n1 = nv[0] / (cam.fx * nrc), n2 = nv[1] / (cam.fy * nrc);
            // u and v are stored scaled by sqrt(1/2): the blend then takes
            // -(u^2 + v^2) as the exponent of G3 = exp(-(u^2 + v^2) / 2).
            constexpr double kRootHalf = 0.70710678118654752440;
            C1 = (float)(kRootHalf * (pzc * as[0] / cam.fx - n1 * pa));
            C2 = (float)(kRootHalf * (pzc * as[1] / cam.fy - n2 * pa));
            D1 = (float)(kRootHalf * (pzc * bs[0] / cam.fx - n1 * pb));
            D2 = (float)(kRootHalf * (pzc * bs[1] / cam.fy - n2 * pb));
            N1 = (float)n1;
            N2 = (float)n2;
            // A surfel without extent (scale 0) has coefficients that are no
            // numbers: it counts as edge-on, so that the blend takes its
            // low-pass term everywhere.  (Below 1e28 no product with a pixel
            // offset overflows, which could make one plane coordinate NaN.)
            const float most = 1e28f;
            if (fabsf(C1) < most && fabsf(C2) < most && fabsf(D1) < most && fabsf(D2) < most) lam_num = (float)pzc;
        }
    }
    v.rec.a = make_float4((float)mux, (float)muy, C1, C2);
    v.rec.b = make_float4(D1, D2, N1, N2);
    v.rec.c = make_float4(lam_num, (float)pzc, op, __uint_as_float(band.x));
    v.rec.d = make_float4(0.f, 0.f, 0.f, __uint_as_float(band.y));
}

__device__ __forceinline__ void sh_dir(const PreCam& cam, float px, float py, float pz, float* d) {
    float dirx = (float)((double)px - cam.t[0]), diry = (float)((double)py - cam.t[1]),
          dirz = (float)((double)pz - cam.t[2]);
    const float inv = rsqrtf(dirx * dirx + diry * diry + dirz * dirz);
    d[0] = dirx * inv;
    d[1] = diry * inv;
    d[2] = dirz * inv;
}

// Does a tile rect hold a masked tile?
__device__ inline bool rect_masked(const CellMask& m, int tx0, int ty0, int tx1, int ty1) {
    for (int cy = ty0 >> 3; cy <= ty1 >> 3; ++cy) {
        const int y0 = max(ty0 - 8 * cy, 0), y1 = min(ty1 - 8 * cy, 7);
        const uint64_t rows = (~0ull >> (8 * (7 - y1))) & (~0ull << (8 * y0));
        for (int cx = tx0 >> 3; cx <= tx1 >> 3; ++cx) {
            const int x0 = max(tx0 - 8 * cx, 0), x1 = min(tx1 - 8 * cx, 7);
            const uint64_t cols = (uint64_t)((0xFFu >> (7 - x1)) & (0xFFu << x0)) * 0x0101010101010101ull;
            if (m.cells[cy * m.cells_x + cx] & rows & cols) return true;
        }
    }
    return false;
}

// Per surfel: the centre-depth key, tile rect and record for `cam` (and with
// kCounts the tiles its band meets, which only bgs_preprocess_debug asks
// for); with kTwo also the key, rect and record for cam2, the other eye of
// a stereo frame.  With a mask, a surfel whose rect holds no masked tile is
// dropped before its colour is read.
// The scene is read once; the colours of both eyes come from one pass over
// the SH coefficients, each toward its own camera centre.
template <bool kTwo, bool kCounts>
__global__ __launch_bounds__(256) void k_preprocess(SceneArgs sc, PreCam cam, PreCam cam2, float alpha_min,
                                                    int lowpass, CellMask mask, SurfelRec* __restrict__ recs,
                                                    uint32_t* __restrict__ zkeys, uint2* __restrict__ rects,
                                                    uint32_t* __restrict__ counts, SurfelRec* __restrict__ recs2,
                                                    uint32_t* __restrict__ zkeys2, uint2* __restrict__ rects2) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= sc.n) return;
    const int n = sc.n;
    const float px = sc.pos[k], py = sc.pos[n + k], pz = sc.pos[2 * n + k];
    const float op = sc.opacity[k];
    const uint2 empty = make_uint2(0xFFFFFFFFu, 0u);
    const float zf = centre_depth_key(cam.zc, px, py, pz);
    const bool in1 = (double)zf > cam.z_near;
    float zf2 = 0.f;
    bool in2 = false;
    if (kTwo) {
        zf2 = centre_depth_key(cam2.zc, px, py, pz);
        in2 = (double)zf2 > cam2.z_near;
        zkeys2[k] = in2 ? __float_as_uint(zf2) : 0xFFFFFFFFu;
    }
    zkeys[k] = in1 ? __float_as_uint(zf) : 0xFFFFFFFFu;
    // alpha = min(0.99, o G) <= o can never reach alpha_min below it.
    const bool live = op >= alpha_min;
    SurfelView v1, v2;
    v1.drawn = v2.drawn = false;
    if (live && (in1 || in2)) {
        double qw = sc.quat[k], qx = sc.quat[n + k], qy = sc.quat[2 * n + k], qz = sc.quat[3 * n + k];
        const double qn = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
        qw *= qn; qx *= qn; qy *= qn; qz *= qn;
        // Columns t_u, t_v of the quaternion's rotation matrix (Sec. 3.3).
        const double tu[3] = {1.0 - 2.0 * (qy * qy + qz * qz), 2.0 * (qx * qy + qw * qz), 2.0 * (qx * qz - qw * qy)};
        const double tv[3] = {2.0 * (qx * qy - qw * qz), 1.0 - 2.0 * (qx * qx + qz * qz), 2.0 * (qy * qz + qw * qx)};
        const double su = sc.scale[k], sv = sc.scale[n + k];
        if (in1) surfel_view(cam, px, py, pz, op, tu, tv, su, sv, alpha_min, lowpass, v1);
        if (kTwo && in2) surfel_view(cam2, px, py, pz, op, tu, tv, su, sv, alpha_min, lowpass, v2);
    }
    if (mask.cells && v1.drawn) v1.drawn = rect_masked(mask, v1.tx0, v1.ty0, v1.tx1, v1.ty1);
    rects[k] = v1.drawn ? make_uint2((uint32_t)v1.tx0 | ((uint32_t)v1.ty0 << 16),
                                     (uint32_t)v1.tx1 | ((uint32_t)v1.ty1 << 16))
                        : empty;
    if (kCounts) counts[k] = v1.drawn ? band_count(BandRows(v1.rec), v1.tx0, v1.ty0, v1.tx1, v1.ty1) : 0u;
    if (kTwo)
        rects2[k] = v2.drawn ? make_uint2((uint32_t)v2.tx0 | ((uint32_t)v2.ty0 << 16),
                                          (uint32_t)v2.tx1 | ((uint32_t)v2.ty1 << 16))
                             : empty;
    const bool col1 = v1.drawn, col2 = kTwo && v2.drawn;
    if (!col1 && !col2) return;
    // ---- colour: SH towards the surfel from each camera's centre ----
    // (With two eyes, the second eye's colour is also kept for every surfel
    // the first eye bins, drawn in the second eye or not: the view-colour
    // transfer composites it with the first eye's weights.)
    float d1[3] = {0.f, 0.f, 1.f}, d2[3] = {0.f, 0.f, 1.f};
    if (col1) sh_dir(cam, px, py, pz, d1);
    if (kTwo && (col1 || col2)) sh_dir(cam2, px, py, pz, d2);
    float Y1[16], Y2[16];
    sh_basis(sc.sh_degree, d1[0], d1[1], d1[2], Y1);
    if (kTwo) sh_basis(sc.sh_degree, d2[0], d2[1], d2[2], Y2);
    const int nc = (sc.sh_degree + 1) * (sc.sh_degree + 1);
    float acc1[3] = {0.f, 0.f, 0.f}, acc2[3] = {0.f, 0.f, 0.f};
    // Eight coefficients' loads are in flight together: a wave that waits for
    // each in turn pays the memory's latency nc times.  (1.2M surfels of degree
    // 3, one eye: 115 -> 106 us; 1M, both eyes: 113 -> 90.  All sixteen, with
    // their registers: 214 and 196.)
    constexpr int kAhead = 8;
#pragma unroll
    for (int c0 = 0; c0 < 16; c0 += kAhead) {
        if (c0 >= nc) break;
        float q[kAhead][3];
#pragma unroll
        for (int j = 0; j < kAhead; ++j)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) q[j][ch] = c0 + j < nc ? sc.sh[(int64_t)((c0 + j) * 3 + ch) * n + k] : 0.f;
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (c0 + j >= nc) break;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                acc1[ch] += Y1[c0 + j] * q[j][ch];
                if (kTwo) acc2[ch] += Y2[c0 + j] * q[j][ch];
            }
        }
    }
    if (col1) {
        v1.rec.d.x = fmaxf(acc1[0] + 0.5f, 0.f);
        v1.rec.d.y = fmaxf(acc1[1] + 0.5f, 0.f);
        v1.rec.d.z = fmaxf(acc1[2] + 0.5f, 0.f);
        recs[k] = v1.rec;
    }
    if (col2) {
        v2.rec.d.x = fmaxf(acc2[0] + 0.5f, 0.f);
        v2.rec.d.y = fmaxf(acc2[1] + 0.5f, 0.f);
        v2.rec.d.z = fmaxf(acc2[2] + 0.5f, 0.f);
        recs2[k] = v2.rec;
    } else if (kTwo && col1) {
        // Not drawn in the second eye: only the colour part, for the transfer.
        recs2[k].d = make_float4(fmaxf(acc2[0] + 0.5f, 0.f), fmaxf(acc2[1] + 0.5f, 0.f), fmaxf(acc2[2] + 0.5f, 0.f),
                                 0.f);
    }
}

// ---------------------------------------------------------------------------
// Binning: the surfels of every tile in compositing order, from the depth
// order.  The image's tiles are grouped in cells of 8x8 tiles.  A surfel has
// one entry per cell that its band meets: its index and the cell's tiles it
// meets as a 64-bit mask.  Entries are placed cell by cell in compositing
// order (k_bin_count, k_bin_scan, k_bin_emit), and each cell's entries are
// then expanded into its 64 tile lists with one lane per entry: a ballot of one
// mask bit gives the entries of a tile (k_tile_count, k_tile_scan,
// k_tile_plan, k_tile_write).
//
// Bound by memory on large frames and by launch latency on small ones.  A
// (surfel, tile) key costs its 4 bytes in the list and a share of a 12-byte
// entry, which several tiles share.  Emitting the keys one by one and
// sorting them by tile id wrote them, read them for a histogram and moved
// them once per digit, 16 bytes a key and pass: binning took 1220 us of the
// 1.2M-surfel 1920x1080 frame (8.3e7 keys) and takes 240.
// ---------------------------------------------------------------------------
constexpr int kBinWin = 1024;   // cells per bitmap window of the emission (32 KiB of LDS)
constexpr int kBinKeep = 1536;  // entries of 256 surfels that the emission keeps in LDS between its two steps
// Words of the count table up to which the emission scans it itself: 16
// loads a thread, about what the launch that it saves costs.
constexpr uint64_t kBinSmallTable = 4096;
constexpr int kChunk = kBinChunk;  // entries a wave expands at a time

// 256 surfels of the order, staged for the cell loops: their bands and
// rects, and the running number of their cell rows.  The unit of work is a
// (surfel, cell row) item, so that the nearest surfels, which span the
// image, are spread over the workgroup.
struct BinStage {
    double k0[256], k16[256], r[256], inv[256];
    uint2 rect[256];
    uint32_t id[256];
    uint32_t item[257];
    uint32_t wsum[4];
};

// Inclusive scan over the wave by DPP: within rows of 16 lanes, then the last
// lane of each row and of the lower half into what follows.
template <typename Add>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, Add&& sum) {
    const auto add = [&](uint32_t x) { v = sum(v, x); };
    add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false));  // row_shr:1
    add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false));
    add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false));
    add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false));
    add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return v;
}
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
    return wave_scan(v, [](uint32_t a, uint32_t b) { return a + b; });
}

// Sums of keys that stop at 2^32 - 1 (4097 surfels across a 16384x16384 image
// have more): such a frame is past any capacity, and reports that.
__device__ __forceinline__ uint32_t add_sat(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ uint32_t wave_scan_sat(uint32_t v) { return wave_scan(v, add_sat); }

// Exclusive scan over a 256-thread block (w4: 4 words of LDS, free again
// after the next barrier); *total gets the sum.
__device__ __forceinline__ uint32_t block_scan_256(uint32_t v, uint32_t* w4, uint32_t* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t x = wave_scan_u32(v);
    if (lane == 63) w4[w] = x;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t y = w4[q];
        before += q < w ? y : 0u;
        sum += y;
    }
    *total = sum;
    return before + x - v;
}

// The positions of the order that chunk c holds.
__device__ __forceinline__ void bin_chunk(const BinArgs& a, uint32_t c, int64_t* p0, int64_t* p1) {
    const bool fine = c < a.fine;
    const int64_t b = fine ? (int64_t)c * kBinFine : (int64_t)a.fine * kBinFine + (int64_t)(c - a.fine) * a.per;
    *p0 = min((int64_t)a.n, b);
    *p1 = min((int64_t)a.n, b + (fine ? kBinFine : a.per));
}

// Stages surfels order[p0 .. p0 + m) and returns the number of items.  Has
// block barriers; the stage may be read after it.  kGather (the counting
// kernel): rects and bands are gathered through the order, and kept in
// compositing order for the emission, which reads them from there (two
// gathers of a line each per surfel are a third of these kernels' time).
template <bool kGather>
__device__ __forceinline__ uint32_t bin_stage(const BinArgs& a, int64_t p0, int m, BinStage& s) {
    const int t = threadIdx.x;
    uint32_t rows = 0;
    if (t < m) {
        const uint32_t k = a.order[p0 + t];
        uint4 g = make_uint4(1u, 0u, 0u, 0u);  // rect, band direction and interval
        float2 mu = make_float2(0.f, 0.f);
        if (kGather) {
            const uint2 rc = a.rects[k];
            if (!(rc.x > rc.y) && (!a.mask.cells || rect_masked(a.mask, (int)(rc.x & 0xFFFFu), (int)(rc.x >> 16),
                                                                (int)(rc.y & 0xFFFFu), (int)(rc.y >> 16)))) {
                const SurfelRec& r = a.recs[k];
                g = make_uint4(rc.x, rc.y, __float_as_uint(r.c.w), __float_as_uint(r.d.w));
                mu = make_float2(r.a.x, r.a.y);
            }
            a.band[p0 + t] = g;
            a.mu[p0 + t] = mu;
        } else {
            g = a.band[p0 + t];
            mu = a.mu[p0 + t];
        }
        if (!(g.x > g.y)) {
            const BandRows br(mu.x, mu.y, g.z, g.w);
            s.k0[t] = br.k0;
            s.k16[t] = br.k16;
            s.r[t] = br.r;
            s.inv[t] = br.inv;
            s.rect[t] = make_uint2(g.x, g.y);
            s.id[t] = k;
            rows = (g.y >> 19) - (g.x >> 19) + 1;  // cell rows: tile row / 8
        }
    }
    uint32_t total;
    s.item[t] = block_scan_256(rows, s.wsum, &total);
    if (t == 0) s.item[256] = total;
    __syncthreads();
    return total;
}

// The band of surfel j of the stage.
__device__ __forceinline__ BandRows stage_band(const BinStage& s, int j) {
    return BandRows(s.k0[j], s.k16[j], s.r[j], s.inv[j]);
}

// f(cell column, mask) for every entry of surfel j in cell row cr.
template <typename F>
__device__ __forceinline__ void surfel_cells(const BinArgs& a, const BinStage& s, int j, int cr, F&& f) {
    const uint2 rc = s.rect[j];
    cell_masks(stage_band(s, j), rc.x & 0xFFFF, rc.x >> 16, rc.y & 0xFFFF, rc.y >> 16, cr, [&](int cx, uint64_t m) {
        if (a.mask.cells) m &= a.mask.cells[(uint32_t)(cr * a.cells_x + cx)];
        if (m) f(cx, m);
    });
}

// f(surfel of the stage, cell, mask) for every entry of item `it`.
template <typename F>
__device__ __forceinline__ void bin_item(const BinArgs& a, const BinStage& s, uint32_t it, F&& f) {
    int lo = 0, hi = 255;  // the last surfel whose first item is not past `it`
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s.item[mid] <= it) lo = mid;
        else hi = mid - 1;
    }
    const int cr = (int)(s.rect[lo].x >> 19) + (int)(it - s.item[lo]);
    surfel_cells(a, s, lo, cr, [&](int cx, uint64_t m) { f(lo, (uint32_t)(cr * a.cells_x + cx), m); });
}

// Entries per (cell, chunk of the order), and the keys and entries of each
// chunk (k_bin_scan makes the keys a running sum).  One workgroup per chunk.
__global__ __launch_bounds__(256) void k_bin_count(BinArgs a) {
    extern __shared__ uint32_t s_cnt[];  // a.n_cells words
    __shared__ BinStage s;
    __shared__ uint32_t s_keys[4];
    const int t = threadIdx.x;
    for (uint32_t c = t; c < a.n_cells; c += 256) s_cnt[c] = 0u;
    int64_t p0, p1;
    bin_chunk(a, blockIdx.x, &p0, &p1);
    uint32_t keys = 0;
    for (int64_t p = p0; p < p1; p += 256) {
        __syncthreads();
        const uint32_t items = bin_stage<true>(a, p, (int)min((int64_t)256, p1 - p), s);
        for (uint32_t it = t; it < items; it += 256)
            bin_item(a, s, it, [&](int, uint32_t cell, uint64_t m) {
                atomicAdd(&s_cnt[cell], 1u);
                keys = add_sat(keys, (uint32_t)__popcll(m));
            });
    }
    keys = wave_scan_sat(keys);
    if ((t & 63) == 63) s_keys[t >> 6] = keys;
    __syncthreads();
    for (uint32_t c = t; c < a.n_cells; c += 256) a.matrix[(size_t)c * a.chunks + blockIdx.x] = s_cnt[c];
    if (t == 0) {
        const uint32_t nk = add_sat(add_sat(s_keys[0], s_keys[1]), add_sat(s_keys[2], s_keys[3]));
        a.kpart[blockIdx.x] = make_uint2(nk, nk ? 1u : 0u);  // an entry has a key at least
    }
}

// The pass's key count (one thread) and the counters that a pass starts
// from.
__device__ __forceinline__ void bin_status(const BinArgs& a, DevStatus* st, int which, uint32_t total) {
    st->n_slots = 0;
    st->n_items = 0;
    st->n_keys = total;
    st->n_sort = total < a.cap ? total : a.cap;
    if (total > a.cap) st->overflow |= 1u;
    if (which == 0) st->n_keys_dom = total;
    else st->n_keys_roi = total;
}

// Block c < n_cells: exclusive scan of the cell's row of the matrix over the
// chunks, in place, and the cell's total.  The last block: the chunks' keys
// as an inclusive running sum, and the pass's key count into the status
// block.
__global__ __launch_bounds__(256) void k_bin_scan(BinArgs a, DevStatus* st, int which) {
    __shared__ uint32_t w4[4];
    const int t = threadIdx.x;
    constexpr int kPer = kBinMaxChunks / 256;
    uint32_t total;
    const uint32_t per = (a.chunks + 255) / 256, c0 = t * per;
    uint32_t v[kPer], sum = 0;
    if (blockIdx.x == a.n_cells) {
        uint64_t keys = 0;  // below 2^36: scanned in two parts
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            v[j] = ((uint32_t)j < per && c0 + j < a.chunks) ? a.kpart[c0 + j].x : 0u;
            keys += v[j];
        }
        uint32_t total_hi;
        const uint64_t lo = block_scan_256((uint32_t)keys & 0xFFFFFu, w4, &total);
        __syncthreads();
        uint64_t run = ((uint64_t)block_scan_256((uint32_t)(keys >> 20), w4, &total_hi) << 20) + lo;
        constexpr uint64_t kMost = 0xFFFFFFFFull;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            run += v[j];
            if ((uint32_t)j < per && c0 + j < a.chunks) a.kpart[c0 + j].x = (uint32_t)min(run, kMost);
        }
        if (t == 0) bin_status(a, st, which, (uint32_t)min(((uint64_t)total_hi << 20) + total, kMost));
        return;
    }
    uint32_t* row = a.matrix + (size_t)blockIdx.x * a.chunks;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        v[j] = ((uint32_t)j < per && c0 + j < a.chunks) ? row[c0 + j] : 0u;
        sum += v[j];
    }
    uint32_t run = block_scan_256(sum, w4, &total);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if ((uint32_t)j < per && c0 + j < a.chunks) row[c0 + j] = run;
        run += v[j];
    }
    if (t == 0) a.ctot[blockIdx.x] = total;
}

// Places the entries.  One workgroup per chunk of the order: 256 surfels at a
// time, a bitmap per cell of the surfels that have an entry there, from
// which an entry's rank follows, so that a cell's entries keep the
// compositing order without a sort.  The first workgroup also writes the
// cells' first entries and first expansion chunks.  A pass with more keys
// than the capacity reports the overflow and keeps the first of them, in
// compositing order and within a surfel in row order of its tiles: only
// surfels that keep a key are placed (every workgroup counts the chunk that
// the capacity cuts again for that), so that those in front keep theirs
// wherever their cells lie, and of the surfel that the capacity cuts the masks
// lose the bits past it.  kScan: a small count table is read whole by every
// workgroup, which takes what it needs of k_bin_scan's sums itself, so that
// small frames save that launch.
template <bool kScan>
__global__ __launch_bounds__(256) void k_bin_emit(BinArgs a, DevStatus* st, int which) {
    extern __shared__ uint32_t s_dyn[];
    __shared__ BinStage s;
    __shared__ uint64_t s_mask[kBinKeep];
    __shared__ uint32_t s_at[kBinKeep];  // cell << 8 | surfel of the stage
    __shared__ uint32_t s_n;
    __shared__ uint32_t s_kpos[257];  // past the capacity: the surfels' first keys
    uint32_t* s_base = s_dyn;              // n_cells
    uint32_t* s_bits = s_dyn + a.n_cells;  // min(n_cells, kBinWin) x 8 words
    const int t = threadIdx.x;
    if (blockIdx.x != 0 && a.kpart[blockIdx.x].y == 0) return;
    // ctot[c]: the entries of cell c; pre(c): those of earlier chunks.
    const uint32_t* ctot = a.ctot;
    uint32_t key0 = 0;  // the chunk's first key, counted through the order
    uint32_t all_keys;
    if (kScan) {
        uint32_t* s_tot = s_dyn + a.n_cells;  // the bitmap's words, not in use yet
        for (uint32_t c = t >> 6; c <= a.n_cells; c += 4) {  // the last: the chunks' keys
            const uint32_t* row = a.matrix + (size_t)c * a.chunks;
            uint32_t pre = 0, tot = 0;
            for (uint32_t q = t & 63; q < a.chunks; q += 64) {
                const uint32_t v = c < a.n_cells ? row[q] : a.kpart[q].x;
                pre = add_sat(pre, q < blockIdx.x ? v : 0u);
                tot = add_sat(tot, v);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                pre = add_sat(pre, (uint32_t)__shfl_xor((int)pre, off, 64));
                tot = add_sat(tot, (uint32_t)__shfl_xor((int)tot, off, 64));
            }
            if ((t & 63) == 0 && c < a.n_cells) {
                s_base[c] = pre;
                s_tot[c] = tot;
            } else if ((t & 63) == 0) {
                s_kpos[0] = pre;
                s_kpos[1] = tot;
            }
        }
        __syncthreads();
        ctot = s_tot;
        key0 = s_kpos[0];
        all_keys = s_kpos[1];
        if (blockIdx.x == 0 && t == 0) bin_status(a, st, which, all_keys);
    } else {
        if (blockIdx.x != 0) key0 = a.kpart[blockIdx.x - 1].x;
        all_keys = a.kpart[a.chunks - 1].x;
    }
    int64_t p0, p1;
    bool over = false;  // does the capacity cut this chunk?  (uniform)
    // Past the capacity: the first keys of the staged surfels, from `first` on,
    // into s_kpos; returns the key after them.
    const auto stage_keys = [&](uint32_t items, uint32_t first) {
        s_kpos[t] = 0u;
        __syncthreads();
        for (uint32_t it = t; it < items; it += 256)
            bin_item(a, s, it, [&](int j, uint32_t, uint64_t m) { atomicAdd(&s_kpos[j], (uint32_t)__popcll(m)); });
        __syncthreads();
        uint32_t total;
        const uint32_t at = add_sat(first, block_scan_256(s_kpos[t], s.wsum, &total));
        s_kpos[t] = at;
        if (t == 0) s_kpos[256] = add_sat(first, total);
        __syncthreads();
        return add_sat(first, total);
    };
    const uint32_t per = (a.n_cells + 255) / 256, c0 = min(a.n_cells, t * per), c1 = min(a.n_cells, c0 + per);
    if (all_keys > a.cap) {  // uniform over the grid
        // The chunk that the capacity cuts: the first that does not keep all of
        // its keys.  Later ones place nothing.
        const auto chunk_keys = [&](uint32_t q) {
            return a.kpart[q].x - (kScan || q == 0 ? 0u : a.kpart[q - 1].x);
        };
        const uint32_t run = (a.chunks + 255) / 256;
        uint32_t sum = 0;
        for (uint32_t j = 0; j < run; ++j) sum = add_sat(sum, t * run + j < a.chunks ? chunk_keys(t * run + j) : 0u);
        __syncthreads();  // key0 and all_keys have been read
        s_kpos[t] = sum;
        __syncthreads();
        if (t == 0) {
            uint32_t first = 0, i = 0;
            while (i < 255 && add_sat(first, s_kpos[i]) <= a.cap) first += s_kpos[i++];
            uint32_t q = min(i * run, a.chunks - 1);
            while (q + 1 < a.chunks && add_sat(first, chunk_keys(q)) <= a.cap) first += chunk_keys(q++);
            s_n = q;
            s_kpos[256] = first;
        }
        __syncthreads();
        const uint32_t cut = s_n;
        uint32_t key = s_kpos[256];
        if (blockIdx.x > cut) return;
        over = blockIdx.x == cut;
        // The cells' entries: all of the chunks before it, and of its surfels
        // those whose first key is kept.
        uint32_t* kept = kScan ? s_dyn + a.n_cells : s_base;
        if (kScan) {
            for (uint32_t c = t >> 6; c < a.n_cells; c += 4) {
                uint32_t v = 0;
                for (uint32_t q = t & 63; q < cut; q += 64) v += a.matrix[(size_t)c * a.chunks + q];
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
                if ((t & 63) == 0) kept[c] = v;
            }
        } else {
            for (uint32_t c = t; c < a.n_cells; c += 256) kept[c] = a.matrix[(size_t)c * a.chunks + cut];
        }
        bin_chunk(a, cut, &p0, &p1);
        for (int64_t p = p0; p < p1 && key < a.cap; p += 256) {
            __syncthreads();
            const uint32_t items = bin_stage<false>(a, p, (int)min((int64_t)256, p1 - p), s);
            if (items == 0) continue;  // uniform
            key = stage_keys(items, key);
            for (uint32_t it = t; it < items; it += 256)
                bin_item(a, s, it, [&](int j, uint32_t cell, uint64_t) {
                    if (s_kpos[j] < a.cap) atomicAdd(&kept[cell], 1u);
                });
        }
        __syncthreads();
        ctot = kept;
    }
    {
        uint32_t sum = 0, total;
        for (uint32_t c = c0; c < c1; ++c) sum += ctot[c];
        uint32_t run = block_scan_256(sum, s.wsum, &total);
        if (blockIdx.x == 0) {
            uint32_t at = run, nq = 0, all;
            for (uint32_t c = c0; c < c1; ++c) nq += (ctot[c] + kChunk - 1) / kChunk;
            __syncthreads();
            uint32_t q = block_scan_256(nq, s.wsum, &all);
            for (uint32_t c = c0; c < c1; ++c) {
                a.cstart[c] = at;
                a.cpre[c] = q;
                q += (ctot[c] + kChunk - 1) / kChunk;
                at += ctot[c];
            }
            if (t == 0) {
                a.cstart[a.n_cells] = total;
                a.cpre[a.n_cells] = all;
            }
        }
        for (uint32_t c = c0; c < c1; ++c) {
            const uint32_t v = ctot[c];  // may lie where the base goes
            s_base[c] = run + (kScan ? s_base[c] : a.matrix[(size_t)c * a.chunks + blockIdx.x]);
            run += v;
        }
    }
    bin_chunk(a, blockIdx.x, &p0, &p1);
    for (int64_t p = p0; p < p1; p += 256) {
        __syncthreads();
        const uint32_t items = bin_stage<false>(a, p, (int)min((int64_t)256, p1 - p), s);
        if (items == 0) continue;  // uniform
        if (over) {
            if (key0 >= a.cap) break;  // uniform
            key0 = stage_keys(items, key0);
        }
        for (uint32_t w0 = 0; w0 < a.n_cells; w0 += kBinWin) {
            const uint32_t nw = min((uint32_t)kBinWin, a.n_cells - w0);
            if (w0) __syncthreads();  // the last window's bits have been counted into s_base
            for (uint32_t i = t; i < 8 * nw; i += 256) s_bits[i] = 0u;
            if (t == 0) s_n = 0u;
            __syncthreads();
            for (uint32_t it = t; it < items; it += 256)
                bin_item(a, s, it, [&](int j, uint32_t cell, uint64_t m) {
                    if (cell - w0 >= nw) return;
                    atomicOr(&s_bits[8 * (cell - w0) + (j >> 5)], 1u << (j & 31));
                    const uint32_t e = atomicAdd(&s_n, 1u);
                    if (e < (uint32_t)kBinKeep) {
                        s_mask[e] = m;
                        s_at[e] = cell << 8 | (uint32_t)j;
                    }
                });
            __syncthreads();
            const auto place = [&](int j, uint32_t cell, uint64_t m) {
                const uint32_t* b = s_bits + 8 * (cell - w0);
                uint32_t pos = s_base[cell] + (uint32_t)__popc(b[j >> 5] & ((1u << (j & 31)) - 1u));
                for (int q = 0; q < (j >> 5); ++q) pos += (uint32_t)__popc(b[q]);
                if (over && s_kpos[j] >= a.cap) return;
                if (pos < a.ecap) {  // always true for consistent counts; keeps every write in bounds
                    a.emask[pos] = m;
                    a.eid[pos] = s.id[j];
                }
            };
            const uint32_t n = s_n;
            if (n <= (uint32_t)kBinKeep) {
                for (uint32_t e = t; e < n; e += 256) place((int)(s_at[e] & 255u), s_at[e] >> 8, s_mask[e]);
            } else {  // the nearest surfels: more entries than are kept, so their masks are formed again
                for (uint32_t it = t; it < items; it += 256)
                    bin_item(a, s, it, [&](int j, uint32_t cell, uint64_t m) {
                        if (cell - w0 < nw) place(j, cell, m);
                    });
            }
            __syncthreads();
            if (over) {  // the surfel that the capacity cuts, if it is staged
                if (t == 0) s_n = 256u;
                __syncthreads();
                if (s_kpos[t] < a.cap && s_kpos[t + 1] > a.cap) s_n = (uint32_t)t;
                __syncthreads();
                const int j = (int)s_n;
                uint32_t room = j < 256 ? a.cap - s_kpos[j] : 0u;
                for (int cr = (int)(s.rect[j & 255].x >> 19); j < 256 && cr <= (int)(s.rect[j].y >> 19); ++cr) {
                    // A row of its cells (at most 128: sides <= 16384 px), a thread each.
                    __syncthreads();
                    if (t < a.cells_x) s_mask[t] = 0ull;
                    __syncthreads();
                    if (t == 0) surfel_cells(a, s, j, cr, [&](int cx, uint64_t m) { s_mask[cx] = m; });
                    __syncthreads();
                    const uint64_t m = t < a.cells_x ? s_mask[t] : 0ull;
                    uint64_t kept = 0;
                    for (int y = 0; y < 8; ++y) {
                        uint32_t left = 0, row = 0;  // keys of this tile row: in the cells before, and all
                        for (int c = 0; c < a.cells_x; ++c) {
                            const uint32_t k = (uint32_t)__popc((uint32_t)(s_mask[c] >> (8 * y)) & 255u);
                            row += k;
                            left += c < t ? k : 0u;
                        }
                        uint32_t bits = (uint32_t)(m >> (8 * y)) & 255u;
                        for (; bits && left < room; bits &= bits - 1u, ++left)
                            kept |= (uint64_t)(bits & (0u - bits)) << (8 * y);
                        room -= min(room, row);
                    }
                    const uint32_t cell = (uint32_t)(cr * a.cells_x + t);
                    if (m && cell - w0 < nw) place(j, cell, kept);
                }
                __syncthreads();
            }
            if (p + 256 < p1)
                for (uint32_t c = t; c < nw; c += 256) {
                    uint32_t k = 0;
#pragma unroll
                    for (int q = 0; q < 8; ++q) k += (uint32_t)__popc(s_bits[8 * c + q]);
                    s_base[w0 + c] += k;
                }
        }
    }
}

// The cell that expansion chunk q belongs to: the last with cp[cell] <= q
// (cells without entries share their successor's and are never chosen).
__device__ __forceinline__ uint32_t chunk_cell(const uint32_t* cp, uint32_t n_cells, uint32_t q) {
    uint32_t lo = 0, hi = n_cells - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (cp[mid] <= q) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Expansion of a chunk of a cell's entries (lane = entry), in four quarters
// of two rows of the cell's tiles: the same 16 bits of every entry's mask.
// Where there are many chunks a wave takes a whole chunk; where there are
// few (small frames) the four waves of a workgroup take a quarter each,
// which is four times sooner done.  The chunks are taken grid-stride: their
// number is known only on the device.
constexpr uint32_t kManyChunks = 4096;

struct ExpandStage {
    uint32_t i0, i1, cell;
    uint64_t m[kChunk / 64];  // the masks of the lane's entries
};

struct ExpandPlan {
    uint32_t nq, q0, step;  // chunks, the wave's first, the stride
    int t0, t1;             // the wave's quarters
    __device__ __forceinline__ ExpandPlan(uint32_t n) : nq(n) {
        const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const bool many = nq > kManyChunks;
        q0 = many ? blockIdx.x * 4 + (uint32_t)w : blockIdx.x;
        step = many ? gridDim.x * 4 : gridDim.x;
        t0 = many ? 0 : w;
        t1 = many ? 4 : w + 1;
    }
};

__device__ __forceinline__ void expand_load(const BinArgs& a, const uint32_t* cp, uint32_t q, int lane, ExpandStage& s) {
    s.cell = chunk_cell(cp, a.n_cells, q);
    s.i0 = a.cstart[s.cell] + (q - cp[s.cell]) * kChunk;
    s.i1 = min(s.i0 + kChunk, a.cstart[s.cell + 1]);
#pragma unroll
    for (int g = 0; g < kChunk / 64; ++g) {
        const uint32_t e = s.i0 + 64 * g + lane;
        s.m[g] = e < s.i1 ? a.emask[e] : 0ull;
    }
}

__device__ __forceinline__ void expand_quarter(const ExpandStage& s, int t, uint32_t (&m)[kChunk / 64]) {
#pragma unroll
    for (int g = 0; g < kChunk / 64; ++g) m[g] = (uint32_t)(s.m[g] >> (16 * t));
}

// The lanes whose mask has bit l.
__device__ __forceinline__ uint64_t tile_lanes(uint32_t m, int l) { return __ballot((m & (1u << l)) != 0u); }

// Transposes the wave's 64x64 bit matrix (row = lane, column = bit of w):
// swaps of the off-diagonal blocks of 32, 16 .. 1, each a value of the lane
// across and, per 32-bit word, a rotation and a bit select.
struct BitTranspose {
    uint32_t keep[5], rot[5];  // for blocks of 16, 8, 4, 2, 1
    bool upper;                // lane >= 32
    __device__ __forceinline__ explicit BitTranspose(int lane) : upper(lane >= 32) {
        constexpr uint32_t low[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const bool set = (lane & (16 >> i)) != 0;
            keep[i] = set ? ~low[i] : low[i];
            rot[i] = set ? (uint32_t)(16 >> i) : 32u - (uint32_t)(16 >> i);  // right
        }
    }
    // The value of lane ^ (16 >> i).
    template <int i>
    static __device__ __forceinline__ uint32_t across(uint32_t x) {
        if (i == 0) return (uint32_t)__shfl_xor((int)x, 16, 64);
        if (i == 1) return dpp<0x128>(x);               // row_ror:8
        if (i == 2) return dpp<0x1B>(dpp<0x141>(x));    // ^ 7 (row_half_mirror), then ^ 3
        if (i == 3) return dpp<0x4E>(x);                // quad_perm [2, 3, 0, 1]
        return dpp<0xB1>(x);                            // quad_perm [1, 0, 3, 2]
    }
    template <int kCtrl>
    static __device__ __forceinline__ uint32_t dpp(uint32_t x) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xF, 0xF, true);
    }
    template <int i>
    __device__ __forceinline__ void step(uint32_t& x) const {
        const uint32_t y = across<i>(x);
        x = (x & keep[i]) | (__builtin_amdgcn_alignbit(y, y, rot[i]) & ~keep[i]);
    }
    __device__ __forceinline__ uint64_t operator()(uint64_t w) const {
        uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
        const uint32_t y = (uint32_t)__shfl_xor((int)(upper ? lo : hi), 32, 64);
        lo = upper ? y : lo;
        hi = upper ? hi : y;
        step<0>(lo), step<0>(hi);
        step<1>(lo), step<1>(hi);
        step<2>(lo), step<2>(hi);
        step<3>(lo), step<3>(hi);
        step<4>(lo), step<4>(hi);
        return (uint64_t)hi << 32 | lo;
    }
};

// Keys of each tile in each chunk: a wave per chunk.  The four masks of a
// lane are added as bit planes (the sum of a tile's four bits is 0 .. 4) and
// the planes are transposed, which leaves lane l the entries of tile l to
// count.  Bound by the reading of the masks; with a ballot per tile and mask
// it was bound by their instructions (1.2M surfels at 1920x1080: 34 us, now
// 10).
__global__ __launch_bounds__(256) void k_tile_count(BinArgs a) {
    static_assert(kChunk == 256, "four masks a lane");
    extern __shared__ uint32_t s_cp[];  // n_cells + 1 words
    const int lane = threadIdx.x & 63;
    const uint32_t nq = a.cpre[a.n_cells], q0 = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blockIdx.x * 4 >= nq) return;
    for (uint32_t c = threadIdx.x; c <= a.n_cells; c += 256) s_cp[c] = a.cpre[c];
    __syncthreads();
    const BitTranspose tr(lane);
    for (uint32_t q = q0; q < nq; q += gridDim.x * 4) {
        ExpandStage s;
        expand_load(a, s_cp, q, lane, s);
        const uint64_t x = s.m[0] ^ s.m[1], one = x ^ s.m[2], c0 = (s.m[0] & s.m[1]) | (x & s.m[2]);
        const uint64_t b0 = one ^ s.m[3], c1 = one & s.m[3], b1 = c0 ^ c1, b2 = c0 & c1;
        a.tcount[(size_t)q * 64 + lane] =
            (uint32_t)(__popcll(tr(b0)) + 2 * __popcll(tr(b1)) + 4 * __popcll(tr(b2)));
    }
}

__device__ __forceinline__ void write_tile_total(const BinArgs& a, uint32_t cell, int lane, uint32_t total) {
    const int tx = (int)(cell % a.cells_x) * 8 + (lane & 7), ty = (int)(cell / a.cells_x) * 8 + (lane >> 3);
    if (tx < a.tiles_x && ty < a.tiles_y) a.ttot[(int64_t)ty * a.tiles_x + tx] = total;
}

// One workgroup per cell: exclusive scan of its tiles' counts (lane = tile)
// over its chunks, in place (a wave takes eight chunks of 128 per round),
// and the tiles' totals.
__global__ __launch_bounds__(1024) void k_tile_scan(BinArgs a) {
    __shared__ uint32_t s_sum[2][16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t q0 = a.cpre[blockIdx.x], q1 = a.cpre[blockIdx.x + 1];
    uint32_t carry = 0;
    int buf = 0;
    for (uint32_t base = q0; base < q1; base += 128, buf ^= 1) {
        uint32_t v[8], sum = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t q = base + 8 * w + j;
            v[j] = q < q1 ? a.tcount[(size_t)q * 64 + lane] : 0u;
            sum += v[j];
        }
        s_sum[buf][w][lane] = sum;
        __syncthreads();  // two buffers: the next round's writes need no barrier of their own
        uint32_t run = carry;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t x = s_sum[buf][k][lane];
            run += k < w ? x : 0u;
            carry += x;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t q = base + 8 * w + j;
            if (q < q1) a.tcount[(size_t)q * 64 + lane] = run;
            run += v[j];
        }
    }
    if (w == 0) write_tile_total(a, blockIdx.x, lane, carry);
}

// The same for one cell by a single wave, without barriers.
__device__ __forceinline__ void tile_scan_wave(const BinArgs& a, uint32_t cell, int lane) {
    const uint32_t q0 = a.cpre[cell], q1 = a.cpre[cell + 1];
    uint32_t run = 0;
    for (uint32_t base = q0; base < q1; base += 16) {
        uint32_t v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = base + j < q1 ? a.tcount[(size_t)(base + j) * 64 + lane] : 0u;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (base + j < q1) a.tcount[(size_t)(base + j) * 64 + lane] = run;
            run += v[j];
        }
    }
    write_tile_total(a, cell, lane, run);
}

// The plan scans the cells itself, one wave each, up to this many cells and
// surfels (so at most 64 chunks of a cell): small frames save a launch.
constexpr uint32_t kPlanCells = 16;
constexpr int kPlanSurfels = 16384;

// Tile order for the blend: tiles by decreasing key count, bucketed by the
// leading bit and the next four bits of the count (about 6% resolution), so
// that the heaviest tiles are dispatched first and spread over all CUs.
// The order only decides which block renders which tile; every tile's
// pixels are computed the same way whatever the order.
constexpr int kOrderBuckets = 32 * 16 + 1;  // (octave, 4 mantissa bits), then empty tiles

__device__ __forceinline__ uint32_t order_bucket(uint32_t len) {
    if (len == 0) return kOrderBuckets - 1;
    const uint32_t e = 31u - (uint32_t)__clz((int)len);
    const uint32_t m = e >= 4 ? (len >> (e - 4)) & 15u : (len << (4 - e)) & 15u;
    return (31u - e) * 16u + (15u - m);
}

// One workgroup: the tiles' list ranges (their totals scanned in tile order,
// clamped to the capacity), and the dispatch order of the live tiles (the
// masked ones with a mask, whose number goes to the status block).  Latency
// bound: up to kPlanHeld tiles are read once and kept in registers, and
// every bucket has kPlanSub counters, taken by lane, because the returning
// LDS atomics of a wave on one counter run one after the other.
constexpr int kPlanSub = 8;
constexpr int kPlanCounters = kOrderBuckets * kPlanSub;

template <int kPlanRegs, bool kScan>
__global__ __launch_bounds__(1024) void k_tile_plan(BinArgs a, uint32_t n_tiles, uint2* __restrict__ ranges,
                                                    uint32_t* __restrict__ order, DevStatus* st) {
    constexpr int kPlanHeld = 1024 * kPlanRegs;
    constexpr int kPer = (kPlanCounters + 1023) / 1024;  // counters per thread of their scan
    __shared__ uint32_t hist[1024 * kPer];
    __shared__ uint16_t s_order[kPlanHeld];  // gathered here, written in order
    __shared__ uint32_t wsum[2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t sub = (uint32_t)tid & (kPlanSub - 1);
    for (int i = tid; i < 1024 * kPer; i += 1024) hist[i] = 0;
    if (kScan && (uint32_t)wave < a.n_cells) tile_scan_wave(a, (uint32_t)wave, lane);  // the barrier below publishes it
    const auto live = [&](uint32_t t) {
        if (t >= n_tiles) return false;
        if (!a.mask.cells) return true;
        const uint32_t ty = t / (uint32_t)a.tiles_x, tx = t - ty * (uint32_t)a.tiles_x;
        return ((a.mask.cells[(ty >> 3) * a.cells_x + (tx >> 3)] >> (8 * (ty & 7) + (tx & 7))) & 1ull) != 0;
    };
    uint32_t bk[kPlanRegs];  // the order bucket of each held tile, or none
    uint32_t carry = 0;
    int buf = 0;
    __syncthreads();
    for (uint32_t base = 0; base < n_tiles; base += kPlanHeld, buf ^= 1) {
        // A wave takes consecutive tiles, 64 at a time, so that what it reads
        // and writes is contiguous.
        uint32_t v[kPlanRegs], x[kPlanRegs], sum = 0;
        const uint32_t t0 = base + (uint32_t)wave * (64 * kPlanRegs) + (uint32_t)lane;
#pragma unroll
        for (int u = 0; u < kPlanRegs; ++u) v[u] = t0 + 64 * u < n_tiles ? a.ttot[t0 + 64 * u] : 0u;
#pragma unroll
        for (int u = 0; u < kPlanRegs; ++u) {
            x[u] = sum + wave_scan_u32(v[u]);
            sum = (uint32_t)__builtin_amdgcn_readlane((int)x[u], 63);
        }
        if (lane == 0) wsum[buf][wave] = sum;
        __syncthreads();
        uint32_t before = carry;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t y = wsum[buf][w];
            before += w < wave ? y : 0u;
            carry += y;
        }
#pragma unroll
        for (int u = 0; u < kPlanRegs; ++u) {
            const uint32_t t = t0 + 64 * u, end = before + x[u];
            const uint32_t r0 = min(end - v[u], a.cap), r1 = min(end, a.cap);
            bk[u] = 0xFFFFFFFFu;
            if (t < n_tiles) {
                ranges[t] = make_uint2(r0, r1);
                if (live(t)) {
                    bk[u] = order_bucket(r1 - r0) * kPlanSub + sub;
                    atomicAdd(&hist[bk[u]], 1u);
                }
            }
        }
    }
    __syncthreads();
    // Exclusive scan of the counters.
    uint32_t hv[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        hv[j] = hist[tid * kPer + j];
        sum += hv[j];
    }
    const uint32_t x = wave_scan_u32(sum);
    if (lane == 63) wsum[buf][wave] = x;
    __syncthreads();
    uint32_t before = x - sum, n_live = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const uint32_t y = wsum[buf][w];
        before += w < wave ? y : 0u;
        n_live += y;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        hist[tid * kPer + j] = before;
        before += hv[j];
    }
    if (tid == 0 && a.mask.cells) {
        st->n_masked = n_live;
        st->n_roi_tiles = n_live;
    }
    __syncthreads();
    if (n_tiles <= (uint32_t)kPlanHeld) {
#pragma unroll
        for (int u = 0; u < kPlanRegs; ++u)
            if (bk[u] != 0xFFFFFFFFu)
                s_order[atomicAdd(&hist[bk[u]], 1u)] = (uint16_t)(wave * (64 * kPlanRegs) + 64 * u + lane);
        __syncthreads();
        for (uint32_t i = tid; i < n_live; i += 1024) order[i] = s_order[i];
    } else {
        // The counter of a tile is that of the thread that counted it.
        for (uint32_t base = 0; base < n_tiles; base += kPlanHeld)
            for (int u = 0; u < kPlanRegs; ++u) {
                const uint32_t t = base + (uint32_t)wave * (64 * kPlanRegs) + 64 * u + (uint32_t)lane;
                if (!live(t)) continue;
                const uint2 r = ranges[t];  // written above by this thread
                order[atomicAdd(&hist[order_bucket(r.y - r.x) * kPlanSub + sub], 1u)] = t;
            }
    }
}

// Writes the tile lists.  A tile's lanes are a ballot of its mask bit; they
// store their surfels at consecutive places of the tile's list, so a store
// leaves as one run of a line or two, without a pass through LDS (appending
// through an LDS buffer, 17 KiB a wave, took 242 us where this takes 77, on
// 8.3e7 keys of a 1920x1080 frame: 4.3 TB/s written).
__global__ __launch_bounds__(256) void k_tile_write(BinArgs a, const uint2* __restrict__ ranges) {
    extern __shared__ uint32_t s_cp[];  // n_cells + 1 words
    const int lane = threadIdx.x & 63;
    const ExpandPlan pl(a.cpre[a.n_cells]);
    if (blockIdx.x >= pl.nq) return;
    for (uint32_t c = threadIdx.x; c <= a.n_cells; c += 256) s_cp[c] = a.cpre[c];
    __syncthreads();
    for (uint32_t q = pl.q0; q < pl.nq; q += pl.step) {
        ExpandStage s;
        expand_load(a, s_cp, q, lane, s);
        uint32_t id[kChunk / 64];
#pragma unroll
        for (int g = 0; g < kChunk / 64; ++g) {
            const uint32_t e = s.i0 + 64 * g + lane;
            id[g] = e < s.i1 ? a.eid[e] : 0u;
        }
        // Lane = tile: where the chunk's run of its list begins.
        const int tx = (int)(s.cell % a.cells_x) * 8 + (lane & 7), ty = (int)(s.cell / a.cells_x) * 8 + (lane >> 3);
        const bool in = tx < a.tiles_x && ty < a.tiles_y;
        const uint32_t base = in ? ranges[(int64_t)ty * a.tiles_x + tx].x + a.tcount[(size_t)q * 64 + lane] : 0u;
        for (int t = pl.t0; t < pl.t1; ++t) {
            uint32_t m[kChunk / 64];
            expand_quarter(s, t, m);
#pragma unroll
            for (int l = 0; l < 16; ++l) {
                uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)base, 16 * t + l);
#pragma unroll
                for (int g = 0; g < kChunk / 64; ++g) {
                    const uint64_t has = tile_lanes(m[g], l);
                    if (has) {  // uniform
                        const uint32_t pos = b + __builtin_amdgcn_mbcnt_hi(
                                                     (uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
                        if (__builtin_amdgcn_inverse_ballot_w64(has) && pos < a.cap) a.vals[pos] = id[g];
                        b += (uint32_t)__popcll(has);
                    }
                }
            }
        }
    }
}

// The masked tiles of each cell, from an ROI tile mask of T x T pixel tiles
// (a 16-pixel tile is masked iff it overlaps a masked T-tile).  A wave per
// cell, a lane per tile.
__global__ __launch_bounds__(256) void k_cell_masks(const uint8_t* __restrict__ tm, int T, int tw, int th, int tiles_x,
                                                    int tiles_y, int cells_x, int n_cells,
                                                    uint64_t* __restrict__ cells) {
    const int lane = threadIdx.x & 63, cell = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (cell >= n_cells) return;  // whole wave
    const int tx = cell % cells_x * 8 + (lane & 7), ty = cell / cells_x * 8 + (lane >> 3);
    bool v = false;
    if (tx < tiles_x && ty < tiles_y) {
        if (T == 16) {
            v = tm[ty * tw + tx] != 0;
        } else if (T == 32) {
            v = tm[(ty >> 1) * tw + (tx >> 1)] != 0;
        } else {  // T == 8: any of the (up to) four 8x8 tiles of this 16x16 tile
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int qx = 2 * tx + (u & 1), qy = 2 * ty + (u >> 1);
                v = v || (qx < tw && qy < th && tm[qy * tw + qx] != 0);
            }
        }
    }
    const uint64_t m = __ballot(v);
    if (lane == 0) cells[cell] = m;
}

// ---------------------------------------------------------------------------
// Blend.  One 256-thread block per 16x16 tile; wave w owns the 8x8 quadrant
// (w & 1, w >> 1) of the tile.  walk_range composites the records [b, e)
// of the tile's sorted list into the block's pixels: batches of 256 records
// are fetched by all threads with vector loads (the next batch while the
// current one is composited) and put in LDS; each wave tests the whole
// batch against its region (the record's strip band) in one vector pass and
// writes the byte offsets of the records that can touch it, in list order,
// to its own LDS list, padded with an all-zero
// record that never contributes.  It then takes kTrip records per trip: their
// alphas are independent and computed together, and only the short
// transmittance chain runs in sequence.  The walk ends at the first batch
// boundary where all 256 pixels are done.  Every thread of the block must
// call it (it has block barriers).
// ---------------------------------------------------------------------------
constexpr int kBatch = 256;
constexpr int kTrip = 4;                // records per trip of the walk
constexpr int kDummy = kBatch;          // LDS record index of the zero record
// Staged records lie in four planes, a float4 of each record apiece: a wave
// stages and tests neighbouring records, which at their 64-byte stride would
// meet in a quarter of the LDS banks.  (1.2M surfels at 1920x1080: 448 ->
// 392 us.)
constexpr int kPlaneRecs = kBatch + 1;
constexpr int kListLen = kBatch + 8;    // per-wave hit list, with padding and the trip after it
// Continuation segments are walked in kRounds rounds: round r takes the
// segments [round_lo(r), round_lo(r + 1)) of every continued tile.  One
// round: a second one (the later segments walked from the exact
// transmittance after the first four) saved speculative work but cost a
// launch of latency (800x600 frames: 1.5% slower, 256x256 2%).
constexpr int kRounds = 1;
__host__ __device__ constexpr uint32_t round_lo(int r) { return r <= 0 ? 0u : kContMaxSeg; }
static_assert(round_lo(kRounds) == kContMaxSeg, "the rounds cover every segment");
constexpr uint32_t kChainBatch = 8;     // earlier segments' parts loaded together when chaining


// A pixel's compositing state.  A pixel that has stopped, or that takes no
// part in a walk, has T = 0: every later pair then adds nothing, so no
// separate flag is needed.  The background weight of a stopped pixel is its
// transmittance at the stop, which equals 1 - A (A is the sum of the
// weights alpha * T, and each step lowers T by exactly its weight).
struct PixelState {
    float T, c0, c1, c2, D, A;
    float x0, x1, x2;  // view-colour transfer only: the affiliated eye's colours, same weights
};

__device__ __forceinline__ bool live(const PixelState& p) { return p.T > 0.f; }

struct WalkCounts {
    uint32_t eval, used, walk, test;
};

struct TileGeom {
    int tid, lane;
    float fpx, fpy;
    float scx, scy;  // centre of the wave's 8x8 region
};

// Alpha of one (pixel, surfel) pair (Eq. 2 with the plane homography of the
// record): alpha = min(alpha_max, o * max(G3, G2)), and the depth the pair
// adds to the proxy (the ray-plane depth where G3 wins, else the centre
// depth).  kPlane: of a pair whose record is plane-only in the wave's region
// (record_in_region), which leaves out what cannot matter there.
template <bool kPlane>
__device__ __forceinline__ void pair_alpha(const float4& r0, const float4& r1, const float4& r2, float fpx, float fpy,
                                           const BlendArgs& a, float& al, float& dsel) {
    const float dx = fpx - r0.x, dy = fpy - r0.y;
    const float den = fmaf(r1.z, dx, fmaf(r1.w, dy, 1.f));
    const float w = __builtin_amdgcn_rcpf(den);
    const float u = fmaf(r0.z, dx, r0.w * dy) * w;
    const float v = fmaf(r1.x, dx, r1.y * dy) * w;
    const float lam = r2.x * w;
    // lam <= z_near covers hits behind the camera and edge-on records; a
    // non-finite u, v near the plane's horizon gives -inf or NaN, and
    // fmaxf then keeps the low-pass term.
    // The record's u and v coefficients carry a factor sqrt(1/2), so
    // -(u^2 + v^2) here is the G3 exponent -(u^2 + v^2) / 2 of the plane.
    const float eq = -fmaf(u, u, v * v);
    if (kPlane) {
        al = fminf(a.alpha_max, r2.z * __expf(eq));
        dsel = lam;
        return;
    }
    const float e3 = lam > a.z_near ? eq : -INFINITY;
    const float e2 = a.lowpass ? -fmaf(dx, dx, dy * dy) : -INFINITY;
    al = fminf(a.alpha_max, r2.z * __expf(fmaxf(e3, e2)));
    dsel = (e3 >= e2) ? lam : r2.y;
}

// One front-to-back compositing step: a pair below alpha_min is skipped;
// the pixel stops before the surfel that would take T below t_min;
// otherwise RGB, the depth proxy D and A accumulate with the same weight
// w = alpha * T, and T drops by w.
template <bool kXfer>
__device__ __forceinline__ void accumulate(float al, float dsel, const float4& r3, const float4& xc, const BlendArgs& a,
                                           PixelState& p, WalkCounts& wc, bool count, bool valid) {
    float wt = (al >= a.alpha_min ? al : 0.f) * p.T;
    const float Tn = p.T - wt;
    const bool stop = Tn < a.t_min;  // also for a pixel already stopped (T = 0)
    wt = stop ? 0.f : wt;
    if (count && valid) {
        wc.eval += p.T > 0.f ? 1u : 0u;
        wc.used += wt > 0.f ? 1u : 0u;
    }
    p.c0 = fmaf(wt, r3.x, p.c0);
    p.c1 = fmaf(wt, r3.y, p.c1);
    p.c2 = fmaf(wt, r3.z, p.c2);
    p.D = fmaf(wt, dsel, p.D);
    p.A += wt;
    p.T = stop ? 0.f : Tn;
    if (kXfer) {
        p.x0 = fmaf(wt, xc.x, p.x0);
        p.x1 = fmaf(wt, xc.y, p.x1);
        p.x2 = fmaf(wt, xc.z, p.x2);
    }
}

// What a record whose band meets the wave's 8x8 region (centre offset dx, dy
// from the projected centre) can do there.
//
// kMisses: nothing at any pixel.  The band bounds the footprint across its
// narrowest direction only; along the others the region may lie past the
// footprint's end.  In plane coordinates (u, v) = (nu, nv) / den the
// footprint is the disc u^2 + v^2 <= ln(o / alpha_min); over the region
// |(nu, nv)| falls below its value at the centre by at most the larger half
// diagonal of the region's image, and den rises by at most
// 3.5 (|N1| + |N2|).  The low-pass disc must be missed too.
//
// kPlane: the low-pass disc is missed, so at every pixel where the pair counts
// (alpha >= alpha_min) G3 is the larger term and gives the depth, and the
// plane is in front of z_near all over the region: the walk then needs
// neither the low-pass term nor the selections between the two, nor the
// test against z_near.  den is bounded away from 0, so that the depth is
// finite also where the pair does not count and enters with weight 0; u and v
// are numbers, since the coefficients of a record that is not edge-on are
// finite with room to spare.  Most
// (record, region) pairs of surfels larger than a tile are of this kind.
//
// Every bound is widened far beyond the rounding of these sums and of
// pair_alpha's, so neither case changes a bit of the image.  (One lane
// tests one record, so this costs each wave less than one of the evaluations
// it saves.)
enum { kMisses, kPlane, kGeneral };
__device__ __forceinline__ int record_in_region(const float4& r0, const float4& r1, const float4& r2, float dx, float dy,
                                                const BlendArgs& a) {
    const float lr = __logf(r2.z * __builtin_amdgcn_rcpf(a.alpha_min)) + 1e-3f;
    const float cx = r0.z * dx, cy = r0.w * dy, ex = r1.x * dx, ey = r1.y * dy, nx = r1.z * dx, ny = r1.w * dy;
    const float nu = cx + cy, nv = ex + ey;
    const float dden = 3.5f * (fabsf(r1.z) + fabsf(r1.w)) + 1e-5f * (1.f + fabsf(nx) + fabsf(ny));
    const float den = 1.f + nx + ny;
    const float pu = r0.z + r0.w, pv = r1.x + r1.y, qu = r0.z - r0.w, qv = r1.x - r1.y;
    const float reach = 3.5f * __builtin_amdgcn_sqrtf(fmaxf(fmaf(pu, pu, pv * pv), fmaf(qu, qu, qv * qv))) * 1.0001f +
                        1e-5f * (fabsf(cx) + fabsf(cy) + fabsf(ex) + fabsf(ey));
    const float rest = __builtin_amdgcn_sqrtf(fmaf(nu, nu, nv * nv)) * 0.9999f - reach, far = den + dden;
    const float lx = fmaxf(fabsf(dx) - 3.5f, 0.f), ly = fmaxf(fabsf(dy) - 3.5f, 0.f);
    const bool plane = den > 2.f * dden && !(a.lowpass && !(fmaf(lx, lx, ly * ly) * 0.9999f > lr));
    const bool misses = rest > 0.f && rest * rest * 0.9999f > lr * far * far;
    return !plane ? kGeneral : misses ? kMisses : r2.x * 0.9999f > a.z_near * far ? kPlane : kGeneral;
}

// One trip of the walk: the records at the LDS offsets off.
template <bool kPlane, bool kCount, bool kXfer>
__device__ __forceinline__ void walk_trip(const char* s_bytes, const uint32_t (&off)[kTrip], const float4* s_xc,
                                          uint32_t nvalid, const TileGeom& g, const BlendArgs& a, PixelState& p,
                                          WalkCounts& wc) {
    float al[kTrip], ds[kTrip];
#pragma unroll
    for (int i = 0; i < kTrip; ++i) {
        const float4* r = reinterpret_cast<const float4*>(s_bytes + off[i]);
        pair_alpha<kPlane>(r[0], r[kPlaneRecs], r[2 * kPlaneRecs], g.fpx, g.fpy, a, al[i], ds[i]);
    }
#pragma unroll
    for (int i = 0; i < kTrip; ++i) {
        const float4* r = reinterpret_cast<const float4*>(s_bytes + off[i]);
        const float4 xc = kXfer ? s_xc[off[i] >> 4] : make_float4(0.f, 0.f, 0.f, 0.f);
        accumulate<kXfer>(al[i], ds[i], r[3 * kPlaneRecs], xc, a, p, wc, kCount, (uint32_t)i < nvalid);
    }
}

// Region test, compaction and compositing of one staged batch of nb records
// by one wave (no block barriers).  A list entry is a record's LDS offset,
// and its top bit is set unless the record is plane-only in the region; a
// trip of plane-only records takes the shorter evaluation.
constexpr uint32_t kGeneralBit = 0x8000u;
static_assert(kDummy * 16 < (int)kGeneralBit, "offsets leave the top bit free");
// kAhead: for launches of few waves, where nothing else hides a wave's own
// latencies: the next trip's entries are read during this one, and the four
// tests of a batch run side by side without branches (10k surfels at 256x256:
// 36.2 -> 33.5 us; 50k at 120x150: 148 -> 135).  The registers that this
// takes cost more where waves are many (1.2M at 1920x1080: 374 -> 383 us; the
// continuation of 800x600: 53 -> 60).
template <bool kCount, bool kXfer = false, bool kAhead = false>
__device__ __forceinline__ void walk_batch(const float4* s_rec, uint32_t nb, uint16_t* s_list, const TileGeom& g,
                                           const BlendArgs& a, PixelState& p, WalkCounts& wc,
                                           const float4* s_xc = nullptr) {
    const char* s_bytes = reinterpret_cast<const char*>(s_rec);
    uint32_t nhit = 0;
    const auto kind = [&](uint32_t j) {
        const uint32_t nq = __float_as_uint(s_rec[2 * kPlaneRecs + j].w), bq = __float_as_uint(s_rec[3 * kPlaneRecs + j].w);
        const float nx = snorm16_value((int)(int16_t)(nq & 0xFFFFu));
        const float ny = snorm16_value((int)(int16_t)(nq >> 16));
        const float4 r0 = s_rec[j];
        const float pr = fmaf(nx, g.scx - r0.x, ny * (g.scy - r0.y)) - half_value(bq);
        const bool band = fabsf(pr) <= half_value(bq >> 16) + 3.5f * (fabsf(nx) + fabsf(ny));
        if (!kAhead && !band) return (int)kMisses;
        const int c = record_in_region(r0, s_rec[kPlaneRecs + j], s_rec[2 * kPlaneRecs + j], g.scx - r0.x,
                                       g.scy - r0.y, a);
        return band ? c : (int)kMisses;
    };
    int ahead[kBatch / 64];  // few waves: the four tests side by side, without branches
    if (kAhead) {
#pragma unroll
        for (int q = 0; q < kBatch / 64; ++q) ahead[q] = kind((uint32_t)(q * 64 + g.lane));
    }
#pragma unroll
    for (int q = 0; q < kBatch / 64; ++q) {
        const uint32_t j = (uint32_t)(q * 64 + g.lane);
        const int c = j >= nb ? (int)kMisses : kAhead ? ahead[q] : kind(j);
        const bool h = c != kMisses;
        const uint32_t entry = j * 16u | (c == kGeneral ? kGeneralBit : 0u);
        const uint64_t m = __ballot(h);
        if (h) {
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            s_list[nhit + below] = (uint16_t)entry;
        }
        nhit += (uint32_t)__popcll(m);
    }
    if (g.lane < kTrip) s_list[nhit + g.lane] = (uint16_t)(kDummy * 16);
    // The list is written and read by this wave only.
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (kCount) {
        wc.walk += nb;
        wc.test += nhit;
    }
    static_assert(kTrip == 4, "a trip's entries are one 8-byte read");
    uint2 next = make_uint2(0u, 0u);
    if (kAhead) next = *reinterpret_cast<const uint2*>(s_list);
    for (uint32_t k = 0; k < nhit; k += kTrip) {
        if (__ballot(live(p)) == 0ull) break;
        const uint2 o = kAhead ? next : *reinterpret_cast<const uint2*>(s_list + k);
        if (kAhead) next = *reinterpret_cast<const uint2*>(s_list + k + kTrip);
        const uint32_t off[kTrip] = {o.x & 0x7FFFu, (o.x >> 16) & 0x7FFFu, o.y & 0x7FFFu, (o.y >> 16) & 0x7FFFu};
        if (__ballot((((o.x | o.y) & (kGeneralBit << 16 | kGeneralBit)) != 0u)) == 0ull)
            walk_trip<true, kCount, kXfer>(s_bytes, off, s_xc, nhit - k, g, a, p, wc);
        else
            walk_trip<false, kCount, kXfer>(s_bytes, off, s_xc, nhit - k, g, a, p, wc);
    }
}

__device__ __forceinline__ void load_rec(const SurfelRec* __restrict__ recs, const uint32_t* __restrict__ vals,
                                         uint32_t pos, float4& q0, float4& q1, float4& q2,
                                         float4& q3) {
    const SurfelRec* r = recs + vals[pos];
    q0 = r->a;
    q1 = r->b;
    q2 = r->c;
    q3 = r->d;
}

// The same, and with the transfer the surfel's colour seen from the other
// eye (the last float4 of its record there).
template <bool kXfer>
__device__ __forceinline__ void load_rec(const SurfelRec* __restrict__ recs, const uint32_t* __restrict__ vals,
                                         uint32_t pos, const BlendArgs& a, float4& q0, float4& q1, float4& q2,
                                         float4& q3, float4& qx) {
    const uint32_t k = vals[pos];
    const SurfelRec* r = recs + k;
    q0 = r->a;
    q1 = r->b;
    q2 = r->c;
    q3 = r->d;
    if (kXfer) qx = a.xrecs[k].d;
}

__device__ __forceinline__ void stage_rec(float4* s_rec, int t, const float4& q0, const float4& q1, const float4& q2,
                                          const float4& q3) {
    s_rec[t] = q0;
    s_rec[kPlaneRecs + t] = q1;
    s_rec[2 * kPlaneRecs + t] = q2;
    s_rec[3 * kPlaneRecs + t] = q3;
}

template <bool kCount>
__device__ __forceinline__ void walk_range(const SurfelRec* __restrict__ recs, const uint32_t* __restrict__ vals,
                                           uint32_t b, uint32_t e, float4* s_rec, uint16_t* s_list,
                                           const TileGeom& g, const BlendArgs& a, PixelState& p, WalkCounts& wc) {
    float4 q0, q1, q2, q3;
    if (b + g.tid < e) load_rec(recs, vals, b + g.tid, q0, q1, q2, q3);
    for (uint32_t base = b; base < e; base += kBatch) {
        const uint32_t nb = min((uint32_t)kBatch, e - base);
        __syncthreads();
        if ((uint32_t)g.tid < nb) stage_rec(s_rec, g.tid, q0, q1, q2, q3);
        __syncthreads();
        if (base + kBatch + g.tid < e) load_rec(recs, vals, base + kBatch + g.tid, q0, q1, q2, q3);
        walk_batch<kCount>(s_rec, nb, s_list, g, a, p, wc);
        if (__syncthreads_count(live(p)) == 0) break;
    }
}

__device__ __forceinline__ TileGeom tile_geom(uint32_t tile, int tid, const BlendArgs& a, bool* inside, int* px,
                                              int* py) {
    TileGeom g;
    const int tx = (int)(tile % (uint32_t)a.tiles_x), ty = (int)(tile / (uint32_t)a.tiles_x);
    g.tid = tid;
    g.lane = g.tid & 63;
    const int wave = g.tid >> 6;
    *px = tx * kTile + (wave & 1) * 8 + (g.lane & 7);
    *py = ty * kTile + (wave >> 1) * 8 + (g.lane >> 3);
    *inside = *px < a.W && *py < a.H &&
              (!a.qmask || a.qmask[(int64_t)(2 * ty + (wave >> 1)) * a.qmask_w + 2 * tx + (wave & 1)] != 0);
    g.fpx = (float)*px;
    g.fpy = (float)*py;
    g.scx = (float)(tx * kTile + (wave & 1) * 8) + 3.5f;
    g.scy = (float)(ty * kTile + (wave >> 1) * 8) + 3.5f;
    return g;
}

template <bool kPatch, bool kXfer = false>
__device__ __forceinline__ void write_pixel(const PixelState& p, int px, int py, const BlendArgs& a,
                                            float* __restrict__ rgb, float* __restrict__ dz, float* __restrict__ alpha,
                                            uint8_t* __restrict__ cls) {
    const int64_t hw = (int64_t)a.W * a.H;
    const int64_t q = (int64_t)py * a.W + px;
    const float tb = p.T > 0.f ? p.T : 1.f - p.A;  // background weight
    rgb[q] = fmaf(tb, a.bg0, p.c0);
    rgb[hw + q] = fmaf(tb, a.bg1, p.c1);
    rgb[2 * hw + q] = fmaf(tb, a.bg2, p.c2);
    if (kXfer) {
        a.xrgb[q] = fmaf(tb, a.bg0, p.x0);
        a.xrgb[hw + q] = fmaf(tb, a.bg1, p.x1);
        a.xrgb[2 * hw + q] = fmaf(tb, a.bg2, p.x2);
    }
    alpha[q] = p.A;
    if (!kPatch) {
        dz[q] = p.D;
    } else {
        dz[q] = p.A >= a.a_min ? p.D / p.A : INFINITY;
        cls[q] = (uint8_t)BGS_CLS_ROI;
    }
}

__device__ __forceinline__ void count_flush(const WalkCounts& wc, int lane, int wave, uint32_t len,
                                            unsigned long long* pair_counts, uint32_t* s_walk) {
    unsigned long long e = wc.eval, u = wc.used;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        e += __shfl_xor(e, off, 64);
        u += __shfl_xor(u, off, 64);
    }
    if (lane == 0) {
        // walk / test are wave-uniform: records walked by this wave and
        // records that passed its strip test.
        atomicAdd(&pair_counts[0], e);
        atomicAdd(&pair_counts[1], u);
        atomicAdd(&pair_counts[2], (unsigned long long)wc.walk);
        atomicAdd(&pair_counts[3], (unsigned long long)wc.test);
        atomicMax(&pair_counts[4], (unsigned long long)wc.walk);
        if (wave == 0) atomicMax(&pair_counts[5], (unsigned long long)len);
        if (s_walk) s_walk[wave] = wc.test;
    }
}

// One block per tile (taken in the order given, heaviest lists first): composite the whole list, then write the pixels.  kPatch:
// ROI patch of the affiliated eye (writes the depth proxy and the class).
// kMany: registers (80) for six workgroups a CU, where there are as many tiles
// (1.2M surfels at 1920x1080: 392 -> 374 us; for seven and eight, which
// spill, 380 and 403).  With fewer tiles than five a CU all run at once
// anyway, the wave that walks the longest list decides, and it is faster
// unconstrained (109; 10k surfels at 256x256: 42 -> 36 us).  The host knows
// the image's tiles only, so an ROI patch takes its image's form.  Against the
// other form, 1M surfels: 300 to 680 live tiles at 1600x1064, 19.0, 39.6, 31.4
// and 32.7 us (18.1, 38.0, 31.6, 32.8); 1656 and 1986 at 2064x2208, 37.9 and
// 25.0 (41.3, 28.5); 11166 there, 225 (249); but 1972 tiles of a 300k shell's
// silhouette at 1600x1064, 192 (185).  The view-colour transfer has the
// unconstrained form only: 463 us at 800x600, 183 at 1600x1064, 429 at
// 2064x2208 (with registers for six: 504, 167, 386).
constexpr int kManyTiles = 5 * 256;
template <bool kCount, bool kPatch, bool kXfer = false, bool kMany = false>
__global__ __launch_bounds__(256, kMany ? 6 : 1) void k_blend(const SurfelRec* __restrict__ recs, const uint32_t* __restrict__ vals,
                                               const uint2* __restrict__ ranges, const uint32_t* __restrict__ order,
                                               const uint32_t* __restrict__ n_live, BlendArgs a, ContArgs ca,
                                               float* __restrict__ rgb, float* __restrict__ dz,
                                               float* __restrict__ alpha, uint8_t* __restrict__ cls,
                                               unsigned long long* __restrict__ pair_counts,
                                               long long* __restrict__ trace) {
    __shared__ float4 s_rec[4 * kPlaneRecs];
    __shared__ float4 s_xc[kXfer ? kBatch + 1 : 1];  // transfer colours, one per staged record
    __shared__ __align__(8) uint16_t s_list[4 * kListLen];
    __shared__ uint32_t s_walk[4];
    __shared__ uint32_t s_slot, s_ibase, s_nseg;
    __shared__ float s_far[4];
    const long long t_begin = kCount ? wall_clock64() : 0;
    const uint32_t blk = blockIdx.x;
    if (n_live && blk >= *n_live) return;
    const uint32_t tile = order[blk];
    bool inside;
    int px, py;
    const TileGeom g = tile_geom(tile, (int)threadIdx.x, a, &inside, &px, &py);
    const uint2 rg = ranges[tile];
    PixelState p{inside ? 1.f : 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    WalkCounts wc{0, 0, 0, 0};
    if (g.tid < 4) s_rec[g.tid * kPlaneRecs + kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (kXfer && g.tid == 0) s_xc[kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    uint16_t* my_list = s_list + (g.tid >> 6) * kListLen;
    // The transfer keeps three more sums per pixel, which the continuation
    // does not carry: such a walk never hands over.
    const uint32_t cap_end = (!kXfer && ca.cap && ca.max_slots && rg.y - rg.x > ca.cap) ? rg.x + ca.cap : rg.y;
    // A capped walk also breaks its batches at its midpoint, where the
    // transmittance is sampled for the hand-over decision.
    const uint32_t mid = cap_end < rg.y ? rg.x + (cap_end - rg.x) / 2 : rg.y;
    float t_half = 1.f;
    uint32_t at_half = rg.x;  // records walked when t_half was taken
    bool half_taken = false, handed = false;
    // One batch loop over the whole list; batches stop at the cap, where the
    // tile decides once whether to hand the rest over (then it leaves the
    // loop) or to walk on.
    float4 q0, q1, q2, q3, qx;
    if (rg.x + g.tid < rg.y) load_rec<kXfer>(recs, vals, rg.x + g.tid, a, q0, q1, q2, q3, qx);
    for (uint32_t base = rg.x; base < rg.y;) {
        const uint32_t lim = base < mid ? mid : base < cap_end ? cap_end : rg.y;
        const uint32_t nb = min((uint32_t)kBatch, lim - base);
        __syncthreads();
        if ((uint32_t)g.tid < nb) {
            stage_rec(s_rec, g.tid, q0, q1, q2, q3);
            if (kXfer) s_xc[g.tid] = qx;
        }
        __syncthreads();
        if (base + nb + g.tid < rg.y) load_rec<kXfer>(recs, vals, base + nb + g.tid, a, q0, q1, q2, q3, qx);
        walk_batch<kCount, kXfer, !kMany>(s_rec, nb, my_list, g, a, p, wc, s_xc);
        base += nb;
        if (!half_taken && base >= mid) {
            half_taken = true;
            t_half = p.T;
            at_half = base;
        }
        const int n_live_px = __syncthreads_count(live(p));
        if (n_live_px == 0) break;
        if (base != cap_end || cap_end == rg.y) continue;
        // Pixels still compositing past the cap: hand the rest of the list
        // to continuation segments if a slot is free and the split pays,
        // else walk on.  It pays when some pixel is expected to walk far:
        // extrapolating the transmittance's decay over the second half of
        // the capped walk, a pixel needs about ln(T / t_min) / (decay per
        // record) more records.  Segments started for pixels that will stop
        // soon would mostly be walked in vain.
        float far = 0.f;
        if (live(p)) {
            const float drop = t_half > p.T ? __logf(t_half / p.T) : 0.f;
            const float need = __logf(p.T / a.t_min) * (float)(cap_end - at_half);
            far = need >= 1e30f * drop ? 1e30f : need / drop;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) far = fmaxf(far, __shfl_xor(far, off, 64));
        if (g.lane == 0) s_far[g.tid >> 6] = far;
        __syncthreads();
        const float far_max = fmaxf(fmaxf(s_far[0], s_far[1]), fmaxf(s_far[2], s_far[3]));
        const uint32_t rem = rg.y - cap_end;
        if (g.tid == 0) {
            s_slot = 0xFFFFFFFFu;
            if (far_max >= (float)ca.min_far && rem >= 2 * ca.seg_len) {
                const uint32_t slot = atomicAdd(ca.n_slots, 1u);
                if (slot < ca.max_slots) {
                    const uint32_t nseg = min(kContMaxSeg, max(1u, (rem + ca.seg_len - 1) / ca.seg_len));
                    const uint32_t ibase = atomicAdd(ca.n_items, nseg);
                    ca.slot_desc[slot] = make_uint4(tile, cap_end, rg.y, ibase | (nseg << kContSegShift));
                    s_slot = slot;
                    s_ibase = ibase;
                    s_nseg = nseg;
                }
            }
        }
        __syncthreads();
        const uint32_t slot = s_slot;
        if (slot != 0xFFFFFFFFu) {
            if ((uint32_t)g.tid < s_nseg) ca.item_slot[s_ibase + g.tid] = slot;
            float4* st = ca.st1 + (size_t)slot * 512;
            st[2 * g.tid] = make_float4(p.c0, p.c1, p.c2, p.D);
            st[2 * g.tid + 1] = make_float4(p.A, p.T, live(p) ? 1.f : 0.f, 0.f);
            handed = live(p);  // pixels already done are final now
            break;
        }
    }
    if (kCount) {
        count_flush(wc, g.lane, g.tid >> 6, rg.y - rg.x, pair_counts, s_walk);
        __syncthreads();
        if (trace && g.tid == 0) {
            // Per tile: id, list length, most records one wave evaluated, CU,
            // start, end.
            long long* t = trace + 6 * (long long)blk;
            t[0] = tile;
            t[1] = rg.y - rg.x;
            t[2] = max(max(s_walk[0], s_walk[1]), max(s_walk[2], s_walk[3]));
            t[3] = __smid();
            t[4] = t_begin;
            t[5] = wall_clock64();
        }
    }
    if (inside && !handed) write_pixel<kPatch, kXfer>(p, px, py, a, rgb, dz, alpha, cls);
}

// ---------------------------------------------------------------------------
// Continuation of the lists handed over by k_blend.  Segment k of a slot's
// remaining records is walked by k_blend_seg from an upper bound of the
// true transmittance at the segment's start: its sums divided by that bound
// are the segment's contribution per unit of incoming transmittance, which
// chains exactly while no pixel would stop inside the segment, and a pixel
// that stops in this walk stops at or before the same record in the true
// one.
// k_blend_chain chains a slot's segments for every pixel and writes the
// pixels that never stop; a pixel whose transmittance would cross t_min
// inside a segment (or that stopped in the speculative walk) is composited
// again over that segment, in order, from its exact state, by k_blend_fix,
// and written there.  k_blend writes the pixels already done when it hands
// a tile over, so every pixel is written once.
// ---------------------------------------------------------------------------
struct Chain {
    float T, c0, c1, c2, D, A;
};

// One segment of the chain.  Returns false where the pixel stops inside the
// segment (nothing is added then).
// One segment of the chain; the segment's sums are stored per unit of the
// transmittance its walk started from.  Returns false where the pixel stops
// inside the segment, or the segment was not walked for it (nothing is added
// then).
__device__ __forceinline__ bool chain_step(const float4& x0, const float4& x1, float t_min, Chain& c) {
    if (x1.z != 0.f || c.T * x1.y < t_min) return false;
    c.c0 = fmaf(c.T, x0.x, c.c0);
    c.c1 = fmaf(c.T, x0.y, c.c1);
    c.c2 = fmaf(c.T, x0.z, c.c2);
    c.D = fmaf(c.T, x0.w, c.D);
    c.A = fmaf(c.T, x1.x, c.A);
    c.T *= x1.y;
    return true;
}

__device__ __forceinline__ void item_segment(const uint4& d, uint32_t k, uint32_t* sb, uint32_t* se) {
    const uint32_t nseg = d.w >> kContSegShift;
    const uint64_t rem = d.z - d.y;
    *sb = d.y + (uint32_t)(rem * k / nseg);
    *se = d.y + (uint32_t)(rem * (k + 1) / nseg);
}

// Round 0 walks the first segments of every continued tile from the
// transmittance T1 after the capped walk.  Each later round (if kRounds > 1)
// walks its segments from every pixel's exact transmittance after the
// segments of the rounds before (a tighter bound than T1), and only for the
// pixels that get through them.
template <bool kCount>
__global__ __launch_bounds__(256) void k_blend_seg(const SurfelRec* __restrict__ recs,
                                                   const uint32_t* __restrict__ vals,
                                                   BlendArgs a, ContArgs ca,
                                                   int round, unsigned long long* __restrict__ pair_counts) {
    __shared__ float4 s_rec[4 * kPlaneRecs];
    __shared__ __align__(8) uint16_t s_list[4 * kListLen];
    const uint32_t n_items = min(*ca.n_items, ca.max_slots * kContMaxSeg);
    if (blockIdx.x >= n_items) return;
    const int tid = (int)threadIdx.x;
    if (tid < 4) s_rec[tid * kPlaneRecs + kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    WalkCounts wc{0, 0, 0, 0};
    for (uint32_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const uint32_t slot = ca.item_slot[item];
        const uint4 d = ca.slot_desc[slot];
        const uint32_t ibase = d.w & ((1u << kContSegShift) - 1u), k = item - ibase;
        const uint32_t lo = round_lo(round);
        if (k < lo || k >= round_lo(round + 1)) continue;
        uint32_t sb, se;
        item_segment(d, k, &sb, &se);
        bool inside;
        int px, py;
        const TileGeom g = tile_geom(d.x, tid, a, &inside, &px, &py);
        const float4 s1 = ca.st1[(size_t)slot * 512 + 2 * tid + 1];
        Chain c{s1.y, 0.f, 0.f, 0.f, 0.f, 0.f};
        bool live = s1.z != 0.f;
        // Chain the lo segments of the earlier rounds, four parts loaded
        // together at a time.
        const float4* xb = ca.part + (size_t)ibase * 512 + 2 * tid;
        for (uint32_t j0 = 0; j0 < lo && live; j0 += 4) {
            float4 x0[4], x1[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                if (j0 + u < lo) {
                    x0[u] = xb[(size_t)(j0 + u) * 512];
                    x1[u] = xb[(size_t)(j0 + u) * 512 + 1];
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u)
                if (j0 + u < lo && live) live = chain_step(x0[u], x1[u], a.t_min, c);
        }
        const float ts = c.T;
        PixelState p{live ? ts : 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (__syncthreads_or(live))
            walk_range<kCount>(recs, vals, sb, se, s_rec, s_list + (tid >> 6) * kListLen, g, a, p, wc);
        const float inv = live ? 1.f / ts : 0.f;
        float4* o = ca.part + (size_t)item * 512;
        o[2 * tid] = make_float4(p.c0 * inv, p.c1 * inv, p.c2 * inv, p.D * inv);
        o[2 * tid + 1] = make_float4(p.A * inv, p.T * inv, live ? (p.T > 0.f ? 0.f : 1.f) : 3.f, 0.f);
    }
    if (kCount) count_flush(wc, tid & 63, tid >> 6, 0, pair_counts, nullptr);
}

// After all segment rounds, one workgroup per slot chains the segments of
// every pixel from the state after the capped walk.  A pixel that never
// stops is written here, and so is one that stops in a segment walked from
// its exact transmittance; for one that stops inside any other segment j
// (or stopped in its speculative walk), the exact state at the start of
// segment j and j + 1 replace the slot's state after the capped walk, for
// k_blend_fix.
template <bool kPatch>
__global__ __launch_bounds__(256) void k_blend_chain(BlendArgs a, ContArgs ca,
                                                     float* __restrict__ rgb, float* __restrict__ dz,
                                                     float* __restrict__ alpha, uint8_t* __restrict__ cls) {
    const uint32_t n_slots = min(*ca.n_slots, ca.max_slots);
    const int tid = (int)threadIdx.x;
    for (uint32_t slot = blockIdx.x; slot < n_slots; slot += gridDim.x) {
        const uint4 d = ca.slot_desc[slot];
        const uint32_t ibase = d.w & ((1u << kContSegShift) - 1u), nseg = d.w >> kContSegShift;
        bool inside;
        int px, py;
        (void)tile_geom(d.x, tid, a, &inside, &px, &py);
        float4* st = ca.st1 + (size_t)slot * 512 + 2 * tid;
        const float4 s0 = st[0], s1 = st[1];
        if (s1.z == 0.f) continue;  // done before the cap and written then
        Chain c{s1.y, s0.x, s0.y, s0.z, s0.w, s1.x};
        uint32_t stop = nseg;
        bool exact = false;
        const float4* xb = ca.part + (size_t)ibase * 512 + 2 * tid;
        for (uint32_t j0 = 0; j0 < nseg && stop == nseg; j0 += kChainBatch) {
            float4 x0[kChainBatch], x1[kChainBatch];
#pragma unroll
            for (uint32_t u = 0; u < kChainBatch; ++u) {
                if (j0 + u < nseg) {
                    x0[u] = xb[(size_t)(j0 + u) * 512];
                    x1[u] = xb[(size_t)(j0 + u) * 512 + 1];
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < kChainBatch; ++u) {
                const uint32_t j = j0 + u;
                if (j < nseg && stop == nseg && !chain_step(x0[u], x1[u], a.t_min, c)) {
                    stop = j;
                    // The first segment of each round was walked from the
                    // pixel's exact transmittance: where the pixel stopped
                    // in that walk, the walk is the true one and needs no
                    // repeat.
                    if (x1[u].z == 1.f && (j == round_lo(0) || j == round_lo(1))) {
                        c.c0 = fmaf(c.T, x0[u].x, c.c0);
                        c.c1 = fmaf(c.T, x0[u].y, c.c1);
                        c.c2 = fmaf(c.T, x0[u].z, c.c2);
                        c.D = fmaf(c.T, x0[u].w, c.D);
                        c.A = fmaf(c.T, x1[u].x, c.A);
                        c.T = 0.f;
                        exact = true;
                    }
                }
            }
        }
        if (stop == nseg || exact) {
            if (inside) write_pixel<kPatch>(PixelState{c.T, c.c0, c.c1, c.c2, c.D, c.A}, px, py, a, rgb, dz, alpha, cls);
            st[1] = make_float4(c.A, c.T, 0.f, 0.f);
        } else {
            st[0] = make_float4(c.c0, c.c1, c.c2, c.D);
            st[1] = make_float4(c.A, c.T, (float)(stop + 1), 0.f);
        }
    }
}

// Item k of a slot composites segment k again, in order, from the exact
// state k_blend_chain recorded, for the pixels that stop inside it, and
// writes them.
template <bool kCount, bool kPatch>
__global__ __launch_bounds__(256) void k_blend_fix(const SurfelRec* __restrict__ recs,
                                                   const uint32_t* __restrict__ vals,
                                                   BlendArgs a, ContArgs ca,
                                                   float* __restrict__ rgb, float* __restrict__ dz,
                                                   float* __restrict__ alpha, uint8_t* __restrict__ cls,
                                                   unsigned long long* __restrict__ pair_counts) {
    __shared__ float4 s_rec[4 * kPlaneRecs];
    __shared__ __align__(8) uint16_t s_list[4 * kListLen];
    const uint32_t n_items = min(*ca.n_items, ca.max_slots * kContMaxSeg);
    if (blockIdx.x >= n_items) return;
    const int tid = (int)threadIdx.x;
    if (tid < 4) s_rec[tid * kPlaneRecs + kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    WalkCounts wc{0, 0, 0, 0};
    for (uint32_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const uint32_t slot = ca.item_slot[item];
        const uint4 d = ca.slot_desc[slot];
        const uint32_t k = item - (d.w & ((1u << kContSegShift) - 1u));
        const float4 s0 = ca.st1[(size_t)slot * 512 + 2 * tid], s1 = ca.st1[(size_t)slot * 512 + 2 * tid + 1];
        const bool need = s1.z == (float)(k + 1);
        if (!__syncthreads_or(need)) continue;
        uint32_t sb, se;
        item_segment(d, k, &sb, &se);
        bool inside;
        int px, py;
        const TileGeom g = tile_geom(d.x, tid, a, &inside, &px, &py);
        PixelState q{need ? s1.y : 0.f, s0.x, s0.y, s0.z, s0.w, s1.x};
        walk_range<kCount>(recs, vals, sb, se, s_rec, s_list + (tid >> 6) * kListLen, g, a, q, wc);
        // A pixel still compositing at the segment's end (whose crossing of
        // t_min the chained product placed in this segment by rounding) walks
        // on, in order, to its stop or the end of the list.
        if (__syncthreads_or(live(q)))
            walk_range<kCount>(recs, vals, se, d.z, s_rec, s_list + (tid >> 6) * kListLen, g, a, q, wc);
        if (inside && need) write_pixel<kPatch>(q, px, py, a, rgb, dz, alpha, cls);
    }
    if (kCount) count_flush(wc, tid & 63, tid >> 6, 0, pair_counts, nullptr);
}

}  // namespace

hipError_t launch_preprocess(const SceneArgs& sc, const PreCam& cam, float alpha_min, int lowpass,
                             const CellMask& mask, SurfelRec* recs, uint32_t* zkeys, uint2* rects,
                             uint32_t* counts, const PreCam* cam2, SurfelRec* recs2, uint32_t* zkeys2,
                             uint2* rects2, hipStream_t s) {
    if (sc.n <= 0) return hipSuccess;
    const dim3 g((sc.n + 255) / 256);
    if (cam2 && counts) return hipErrorInvalidValue;  // counts are of a single camera
    if (cam2)
        hipLaunchKernelGGL((k_preprocess<true, false>), g, dim3(256), 0, s, sc, cam, *cam2, alpha_min, lowpass, mask,
                           recs, zkeys, rects, nullptr, recs2, zkeys2, rects2);
    else if (counts)
        hipLaunchKernelGGL((k_preprocess<false, true>), g, dim3(256), 0, s, sc, cam, cam, alpha_min, lowpass, mask,
                           recs, zkeys, rects, counts, nullptr, nullptr, nullptr);
    else
        hipLaunchKernelGGL((k_preprocess<false, false>), g, dim3(256), 0, s, sc, cam, cam, alpha_min, lowpass, mask,
                           recs, zkeys, rects, nullptr, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_cell_masks(const uint8_t* tmask, int T, int W, int H, uint64_t* cells, hipStream_t s) {
    if (T != 8 && T != 16 && T != 32) return hipErrorInvalidValue;
    const int tiles_x = (W + kTile - 1) / kTile, tiles_y = (H + kTile - 1) / kTile;
    const int cells_x = (tiles_x + 7) / 8, n_cells = cells_x * ((tiles_y + 7) / 8);
    hipLaunchKernelGGL(k_cell_masks, dim3((unsigned)((n_cells + 3) / 4)), dim3(256), 0, s, tmask, T, (W + T - 1) / T,
                       (H + T - 1) / T, tiles_x, tiles_y, cells_x, n_cells, cells);
    return hipGetLastError();
}

hipError_t launch_bin_entries(const BinArgs& a, DevStatus* st, int which, hipStream_t s) {
    // One workgroup per chunk of the order; the LDS holds a word per cell
    // (64 KiB at 16384x16384) and the emission's bitmap window.
    const size_t cells = 4 * (size_t)a.n_cells;
    const size_t bits = 32 * (size_t)std::min<uint32_t>(a.n_cells, kBinWin);
    if (a.chunks < 1 || a.chunks > (uint32_t)kBinMaxChunks || a.fine > a.chunks || a.per < 256 || a.per % 256) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_bin_count, dim3(a.chunks), dim3(256), cells, s, a);
    if ((uint64_t)a.n_cells * a.chunks <= kBinSmallTable) {
        hipLaunchKernelGGL(k_bin_emit<true>, dim3(a.chunks), dim3(256), cells + bits, s, a, st, which);
    } else {
        hipLaunchKernelGGL(k_bin_scan, dim3(a.n_cells + 1), dim3(256), 0, s, a, st, which);
        hipLaunchKernelGGL(k_bin_emit<false>, dim3(a.chunks), dim3(256), cells + bits, s, a, st, which);
    }
    return hipGetLastError();
}

// Grid of the chunk-strided kernels: enough workgroups for the chunks that
// the key capacity allows, at most eight per CU.
static unsigned expand_grid(const BinArgs& a) {
    return (unsigned)std::min<uint64_t>(2048, bin_max_expand_chunks(a.ecap, a.n_cells));
}

hipError_t launch_tile_plan(const BinArgs& a, uint2* ranges, uint32_t* order, DevStatus* st, hipStream_t s) {
    const size_t cp = 4 * ((size_t)a.n_cells + 1);
    hipLaunchKernelGGL(k_tile_count, dim3(expand_grid(a)), dim3(256), cp, s, a);
    const uint32_t n_tiles = (uint32_t)(a.tiles_x * a.tiles_y);
    const dim3 one(1), wg(1024);
    if (a.n_cells <= kPlanCells && a.n <= kPlanSurfels) {  // at most 1024 tiles
        hipLaunchKernelGGL((k_tile_plan<1, true>), one, wg, 0, s, a, n_tiles, ranges, order, st);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_tile_scan, dim3(a.n_cells), dim3(1024), 0, s, a);
    if (n_tiles <= 4 * 1024)
        hipLaunchKernelGGL((k_tile_plan<4, false>), one, wg, 0, s, a, n_tiles, ranges, order, st);
    else if (n_tiles <= 8 * 1024)
        hipLaunchKernelGGL((k_tile_plan<8, false>), one, wg, 0, s, a, n_tiles, ranges, order, st);
    else
        hipLaunchKernelGGL((k_tile_plan<20, false>), one, wg, 0, s, a, n_tiles, ranges, order, st);
    return hipGetLastError();
}

hipError_t launch_tile_write(const BinArgs& a, const uint2* ranges, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_write, dim3(expand_grid(a)), dim3(256), 4 * ((size_t)a.n_cells + 1), s, a, ranges);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched blend: one persistent launch over the tiles of many frames.  Each
// workgroup takes the next (frame, compact tile) item from a queue counter,
// composites the tile's whole list (no continuation: the batch itself keeps
// the GPU full) and writes its pixels, until the queue is empty.  Items go
// frame by frame, each frame's tiles heaviest first.  Workgroups never wait
// for one another, so every workgroup reaches the end of the queue.
// ---------------------------------------------------------------------------
__global__ void k_put_desc(BatchBlendDesc d, BatchBlendDesc* dst) {
    if (threadIdx.x == 0) *dst = d;
}

hipError_t launch_put_desc(const BatchBlendDesc& d, BatchBlendDesc* dst, hipStream_t s) {
    hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(64), 0, s, d, dst);
    return hipGetLastError();
}

__global__ void k_batch_prefix(const BatchBlendDesc* __restrict__ descs, int n, uint32_t* __restrict__ prefix,
                               uint32_t* __restrict__ counter) {
    if (threadIdx.x != 0) return;
    uint32_t run = 0;
    for (int f = 0; f < n; ++f) {
        prefix[f] = run;
        run += descs[f].n_live ? min(*descs[f].n_live, descs[f].n_tiles) : descs[f].n_tiles;
    }
    prefix[n] = run;
    *counter = 0u;
}

template <bool kPatch>
__global__ __launch_bounds__(256, 6) void k_blend_batch(const BatchBlendDesc* __restrict__ descs, int n,
                                                     const uint32_t* __restrict__ prefix, uint32_t* counter) {
    __shared__ float4 s_rec[4 * kPlaneRecs];
    __shared__ __align__(8) uint16_t s_list[4 * kListLen];
    __shared__ uint32_t s_item;
    const int tid = (int)threadIdx.x;
    if (tid < 4) s_rec[tid * kPlaneRecs + kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    const uint32_t total = prefix[n];
    WalkCounts wc{0, 0, 0, 0};
    for (;;) {
        __syncthreads();  // the previous item's use of s_item and the LDS batches is over
        if (tid == 0) s_item = atomicAdd(counter, 1u);
        __syncthreads();
        const uint32_t item = s_item;
        if (item >= total) break;
        // The frame: the last f with prefix[f] <= item (a frame with no item
        // shares its prefix with the next one and is never chosen).
        int lo = 0, hi = n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (prefix[mid] <= item) lo = mid;
            else hi = mid - 1;
        }
        const BatchBlendDesc d = descs[lo];
        const uint32_t blk = item - prefix[lo];
        const uint32_t tile = d.order[blk];
        bool inside;
        int px, py;
        const TileGeom g = tile_geom(tile, tid, d.a, &inside, &px, &py);
        const uint2 rg = d.ranges[tile];
        PixelState p{inside ? 1.f : 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        walk_range<false>(d.recs, d.vals, rg.x, rg.y, s_rec, s_list + (tid >> 6) * kListLen, g, d.a, p, wc);
        if (inside) write_pixel<kPatch>(p, px, py, d.a, d.rgb, d.dz, d.alpha, d.cls);
    }
}

hipError_t launch_blend_batch(const BatchBlendDesc* descs, int n, uint32_t* scratch, int grid, bool patch,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    uint32_t* prefix = scratch;
    uint32_t* counter = scratch + n + 1;
    hipLaunchKernelGGL(k_batch_prefix, dim3(1), dim3(64), 0, s, descs, n, prefix, counter);
    if (patch)
        hipLaunchKernelGGL((k_blend_batch<true>), dim3(grid), dim3(256), 0, s, descs, n, prefix, counter);
    else
        hipLaunchKernelGGL((k_blend_batch<false>), dim3(grid), dim3(256), 0, s, descs, n, prefix, counter);
    return hipGetLastError();
}

hipError_t launch_blend(const SurfelRec* recs, const uint32_t* vals, const uint2* ranges, const uint32_t* order, const uint32_t* n_live, int n_blocks, const BlendArgs& a,
                        const ContArgs& ca, float* rgb, float* d_or_z, float* alpha, uint8_t* cls,
                        unsigned long long* pair_counts, long long* trace, hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    const dim3 g(n_blocks), b(256);
    const bool cont = ca.cap != 0 && ca.max_slots != 0, many = n_blocks > kManyTiles;
    const dim3 gc(min(ca.max_slots * kContMaxSeg, 4096u)), gs(ca.max_slots);
    if (a.patch && a.xrecs) return hipErrorInvalidValue;  // the transfer belongs to the dominant eye
    if (a.patch) {
        if (pair_counts) {
            hipLaunchKernelGGL((k_blend<true, true>), g, b, 0, s, recs, vals, ranges, order, n_live, a, ca,
                               rgb, d_or_z, alpha, cls, pair_counts, trace);
            if (cont) {
                for (int round = 0; round < kRounds; ++round)
                    hipLaunchKernelGGL((k_blend_seg<true>), gc, b, 0, s, recs, vals, a, ca, round,
                                       pair_counts);
                hipLaunchKernelGGL((k_blend_chain<true>), gs, b, 0, s, a, ca, rgb, d_or_z, alpha, cls);
                hipLaunchKernelGGL((k_blend_fix<true, true>), gc, b, 0, s, recs, vals, a, ca, rgb, d_or_z,
                                   alpha, cls, pair_counts);
            }
        } else {
            const auto kernel = many ? k_blend<false, true, false, true> : k_blend<false, true, false, false>;
            hipLaunchKernelGGL(kernel, g, b, 0, s, recs, vals, ranges, order, n_live, a, ca, rgb, d_or_z, alpha, cls, pair_counts,
                               (long long*)nullptr);
            if (cont) {
                for (int round = 0; round < kRounds; ++round)
                    hipLaunchKernelGGL((k_blend_seg<false>), gc, b, 0, s, recs, vals, a, ca, round,
                                       pair_counts);
                hipLaunchKernelGGL((k_blend_chain<true>), gs, b, 0, s, a, ca, rgb, d_or_z, alpha, cls);
                hipLaunchKernelGGL((k_blend_fix<false, true>), gc, b, 0, s, recs, vals, a, ca, rgb, d_or_z,
                                   alpha, cls, pair_counts);
            }
        }
    } else {
        if (pair_counts && a.xrecs) {
            hipLaunchKernelGGL((k_blend<true, false, true>), g, b, 0, s, recs, vals, ranges, order, n_live,
                               a, ca, rgb, d_or_z, alpha, cls, pair_counts, trace);
        } else if (pair_counts) {
            hipLaunchKernelGGL((k_blend<true, false>), g, b, 0, s, recs, vals, ranges, order, n_live, a, ca,
                               rgb, d_or_z, alpha, cls, pair_counts, trace);
            if (cont) {
                for (int round = 0; round < kRounds; ++round)
                    hipLaunchKernelGGL((k_blend_seg<true>), gc, b, 0, s, recs, vals, a, ca, round,
                                       pair_counts);
                hipLaunchKernelGGL((k_blend_chain<false>), gs, b, 0, s, a, ca, rgb, d_or_z, alpha, cls);
                hipLaunchKernelGGL((k_blend_fix<true, false>), gc, b, 0, s, recs, vals, a, ca, rgb, d_or_z,
                                   alpha, cls, pair_counts);
            }
        } else if (a.xrecs) {
            // View-colour transfer: never continued.
            hipLaunchKernelGGL((k_blend<false, false, true>), g, b, 0, s, recs, vals, ranges, order, n_live,
                               a, ca, rgb, d_or_z, alpha, cls, pair_counts, (long long*)nullptr);
        } else {
            const auto kernel = many ? k_blend<false, false, false, true> : k_blend<false, false, false, false>;
            hipLaunchKernelGGL(kernel, g, b, 0, s, recs, vals, ranges, order, n_live, a, ca, rgb, d_or_z, alpha, cls, pair_counts,
                               (long long*)nullptr);
            if (cont) {
                for (int round = 0; round < kRounds; ++round)
                    hipLaunchKernelGGL((k_blend_seg<false>), gc, b, 0, s, recs, vals, a, ca, round,
                                       pair_counts);
                hipLaunchKernelGGL((k_blend_chain<false>), gs, b, 0, s, a, ca, rgb, d_or_z, alpha, cls);
                hipLaunchKernelGGL((k_blend_fix<false, false>), gc, b, 0, s, recs, vals, a, ca, rgb,
                                   d_or_z, alpha, cls, pair_counts);
            }
        }
    }
    return hipGetLastError();
}

}  // namespace bgs
