// HIP kernels of the gamma index (section 2.2.3) and the array maximum it
// normalises by, for gfx950.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sde_internal.hpp"

namespace sde {
namespace {

__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Trilinear value of grid g at (fx, fy, fz) in voxel units; false outside
// [0, n - 1] on an axis.  The expression and the order of its operations are
// those of the definition, with no fused multiply-adds, so that the pass
// decision below is the same, bit for bit, as a double-precision evaluation
// of the definition.
__device__ __forceinline__ bool trilinear(const double* g, int nx, int ny, int nz, double fx,
                                          double fy, double fz, double& v) {
#pragma clang fp contract(off)
    if (fx < 0.0 || fy < 0.0 || fz < 0.0 || fx > nx - 1 || fy > ny - 1 || fz > nz - 1)
        return false;
    int x0 = (int)floor(fx), y0 = (int)floor(fy), z0 = (int)floor(fz);
    if (x0 > nx - 2) x0 = nx > 1 ? nx - 2 : 0;
    if (y0 > ny - 2) y0 = ny > 1 ? ny - 2 : 0;
    if (z0 > nz - 2) z0 = nz > 1 ? nz - 2 : 0;
    const double tx = fx - x0, ty = fy - y0, tz = fz - z0;
    const int x1 = nx > 1 ? x0 + 1 : x0, y1 = ny > 1 ? y0 + 1 : y0, z1 = nz > 1 ? z0 + 1 : z0;
    const double* p00 = g + ((size_t)z0 * ny + y0) * nx;
    const double* p10 = g + ((size_t)z0 * ny + y1) * nx;
    const double* p01 = g + ((size_t)z1 * ny + y0) * nx;
    const double* p11 = g + ((size_t)z1 * ny + y1) * nx;
    const double c00 = p00[x0] * (1 - tx) + p00[x1] * tx;
    const double c10 = p10[x0] * (1 - tx) + p10[x1] * tx;
    const double c01 = p01[x0] * (1 - tx) + p01[x1] * tx;
    const double c11 = p11[x0] * (1 - tx) + p11[x1] * tx;
    const double c0 = c00 * (1 - ty) + c10 * ty, c1 = c01 * (1 - ty) + c11 * ty;
    v = c0 * (1 - tz) + c1 * tz;
    return true;
}

constexpr int kMaxK = 50;   // largest interp (offsets per dta per axis)

// Everything the two gamma kernels read.
struct GammaArgs {
    const double* ref;
    const double* ev;
    int nx, ny, nz, K;
    double st, dta, dx, dy, dz;      // lattice spacing dta / K, dta, voxel size (cm)
    double dd, thresh, inv_dta2;
    int local, use_bound;
    double inv_nx, inv_ny;           // index decoding (with a correction by one)
    size_t v0;                       // first voxel of this pass (list entries count from it)
    unsigned nv;                     // voxels of this pass
    int n_max;                       // partial maxima of the reference
    unsigned long long* buf;         // the counters (GammaCounters)
    unsigned* list;
};

// The counters, one 128-byte line each so that their atomics (one per
// workgroup; same-address ones take 12 ns each) do not queue up behind one
// another: [0] list length, [1] maximum bits, then kSlots lines {evaluated,
// passed}, then the partial maxima of k_max.
constexpr int kLine = 16;                                // 128 bytes
constexpr int kSlots = kGammaSlots;
constexpr int kCountWords = kLine * (1 + kSlots);
static_assert(kCountWords + kGammaMaxParts <= kGammaWords, "counters and partial maxima");

// Per axis and lattice index a in [-K, K]: a st (cm) and a st / d (voxels),
// in LDS.
struct GammaLattice {
    double cm[3][2 * kMaxK + 1];
    double vx[3][2 * kMaxK + 1];
};

__device__ __forceinline__ void fill_lattice(const GammaArgs& A, GammaLattice& L) {
    const int nl = 2 * A.K + 1;
    for (int t = threadIdx.x; t < 3 * nl; t += blockDim.x) {
        const int ax = t / nl, a = t % nl - A.K;
        const double v = a * A.st;
        L.cm[ax][a + A.K] = v;
        L.vx[ax][a + A.K] = v / (ax == 0 ? A.dx : ax == 1 ? A.dy : A.dz);
    }
    __syncthreads();
}

// q = i / n and the remainder (i below 2^53; inv = 1 / n): the product may be
// off by one, which the remainder's sign and size show.
__device__ __forceinline__ unsigned long long div_rem(unsigned long long i, int n, double inv,
                                                      int& rem) {
    unsigned long long q = (unsigned long long)((double)i * inv);
    long long r = (long long)(i - q * (unsigned long long)n);
    if (r < 0) {
        --q;
        r += n;
    } else if (r >= n) {
        ++q;
        r -= n;
    }
    rem = (int)r;
    return q;
}

__device__ __forceinline__ void voxel_of(const GammaArgs& A, size_t i, int& ix, int& iy, int& iz) {
    const unsigned long long row = div_rem(i, A.nx, A.inv_nx, ix);
    iz = (int)div_rem(row, A.ny, A.inv_ny, iy);
}

__device__ __forceinline__ double norm_of(const GammaArgs& A, double dr) {
    return A.dd * (A.local ? dr : __longlong_as_double((long long)A.buf[1]));
}

// The test of one offset of the definition: r2 = |o|^2, v the evaluated map
// there.  Screened with multiplications by reciprocals; within 1e-12 of the
// boundary decided by the definition's divisions, so that the decision is the
// same, bit for bit, as a double-precision evaluation of the definition.
__device__ __forceinline__ bool offset_passes(const GammaArgs& A, double r2, double v, double dr,
                                              double norm2, double inv_n2, double& gf) {
#pragma clang fp contract(off)
    const double diff = v - dr;
    gf = r2 * A.inv_dta2 + diff * diff * inv_n2;
    if (gf > 1.0 + 1e-12) return false;
    return gf < 1.0 - 1e-12 || r2 / (A.dta * A.dta) + diff * diff / norm2 <= 1.0;
}

// The offset (a, b, c) of voxel (ix, iy, iz), by the definition.
__device__ __forceinline__ bool offset_test(const GammaArgs& A, const GammaLattice& L, int ix,
                                            int iy, int iz, int a, int b, int c, double dr,
                                            double norm2, double inv_n2) {
#pragma clang fp contract(off)
    const int K = A.K;
    double v, gf;
    if (!trilinear(A.ev, A.nx, A.ny, A.nz, ix + L.vx[0][a + K], iy + L.vx[1][b + K],
                   iz + L.vx[2][c + K], v))
        return false;
    const double r2 = L.cm[0][a + K] * L.cm[0][a + K] + L.cm[1][b + K] * L.cm[1][b + K] +
                      L.cm[2][c + K] * L.cm[2][c + K];
    return offset_passes(A, r2, v, dr, norm2, inv_n2, gf);
}

// One octant of a voxel's offsets: the sign pattern s = 0 takes a >= 0 (cell
// [i, i + 1]), s = 1 takes a < 0 (cell [i - 1, i]); v[x + 2 y + 4 z]: the cell's
// corners.
struct Octant {
    int ix, iy, iz, x0, y0, z0, sx, sy, sz;
    double dr, norm2, inv_n2;
    double v[8];
    int nmax;   // a^2 + b^2 + c^2 of a passing offset is at most this
};

// Smallest value over the rectangle [a0, a1] x [b0, b1] of s times the bilinear
// function with corner values e00, e10, e01, e11.
__device__ __forceinline__ double bilinear_min(double e00, double e10, double e01, double e11,
                                               double a0, double a1, double b0, double b1,
                                               double s) {
    const double p0 = e00 + a0 * (e10 - e00), p1 = e00 + a1 * (e10 - e00);
    const double q0 = e01 + a0 * (e11 - e01), q1 = e01 + a1 * (e11 - e01);
    return fmin(fmin(s * (p0 + b0 * (q0 - p0)), s * (p0 + b1 * (q0 - p0))),
                fmin(s * (p1 + b0 * (q1 - p1)), s * (p1 + b1 * (q1 - p1))));
}

// What the values of a cell say about an octant (dta at most a voxel on
// every axis): false when no offset of it can pass; else O.nmax, and in
// (ca, cb, cc) the lattice offset nearest the minimum of the linearised test
// function (all zero if that minimum exceeds 1).
//
// The evaluated map is trilinear in the cell, so its slope along an axis is
// bilinear in the other two and takes its extremes over the octant's box at
// the box's corners.  With g_i >= 0 the steepest approach to dr along axis i
// in the octant's direction and d = |v(0) - dr|, |v(o) - dr| >= d - g . |o|,
// and the smallest value of |o|^2 / dta^2 + max(0, d - g . |o|)^2 / norm^2 over all
// o is d^2 / (norm^2 + |g|^2 dta^2): above 1, by 1e-9 (far beyond rounding),
// nothing passes.  With an infinite or NaN corner the slopes mean nothing (and
// the offsets on a face towards the next cell, which dta equal to a voxel
// reaches, are that cell's): the rows decide.
__device__ __forceinline__ bool octant_open(const GammaArgs& A, const GammaLattice& L, Octant& O,
                                            int& ca, int& cb, int& cc) {
    const int K = A.K, KK = K * K;
    const double* v = O.v;
    // the box in cell coordinates: from t (the voxel's own corner) by r
    const double tx = O.ix - O.x0, ty = O.iy - O.y0, tz = O.iz - O.z0;
    const double rx = O.sx || O.ix + 1 < A.nx ? L.vx[0][2 * K] : 0.0;
    const double ry = O.sy || O.iy + 1 < A.ny ? L.vx[1][2 * K] : 0.0;
    const double rz = O.sz || O.iz + 1 < A.nz ? L.vx[2][2 * K] : 0.0;
    const double gx = O.sx ? -1.0 : 1.0, gy = O.sy ? -1.0 : 1.0, gz = O.sz ? -1.0 : 1.0;
    const double ux = tx + gx * rx, uy = ty + gy * ry, uz = tz + gz * rz;
    const double x00 = v[1] - v[0], x10 = v[3] - v[2], x01 = v[5] - v[4], x11 = v[7] - v[6];
    const double y00 = v[2] - v[0], y10 = v[3] - v[1], y01 = v[6] - v[4], y11 = v[7] - v[5];
    const double z00 = v[4] - v[0], z10 = v[5] - v[1], z01 = v[6] - v[2], z11 = v[7] - v[3];
    const bool hx = tx > 0.5, hy = ty > 0.5, hz = tz > 0.5;
    const double a0 = hx ? v[1] : v[0], a1 = hx ? v[3] : v[2], a2 = hx ? v[5] : v[4],
                 a3 = hx ? v[7] : v[6];
    const double vc = hz ? (hy ? a3 : a2) : (hy ? a1 : a0);
    const double d0 = vc - O.dr, sg = d0 > 0.0 ? 1.0 : -1.0;
    // slopes per dta, in the octant's direction, towards dr
    const double px = rx * fmax(0.0, -bilinear_min(x00, x10, x01, x11, ty, uy, tz, uz, sg * gx));
    const double py = ry * fmax(0.0, -bilinear_min(y00, y10, y01, y11, tx, ux, tz, uz, sg * gy));
    const double pz = rz * fmax(0.0, -bilinear_min(z00, z10, z01, z11, tx, ux, ty, uy, sg * gz));
    const double big = ((fabs(v[0]) + fabs(v[1])) + (fabs(v[2]) + fabs(v[3]))) +
                       ((fabs(v[4]) + fabs(v[5])) + (fabs(v[6]) + fabs(v[7])));
    const double d = fabs(d0) - 1e-12 * (big + fabs(O.dr));   // no more than 0, or NaN, beside them
    if (d > 0.0) {
        if (d * d > (O.norm2 + px * px + py * py + pz * pz) * (1.0 + 1e-9)) return false;
        const double near = d - (px + py + pz);   // the octant's closest approach to dr
        if (near > 0.0) {
            const double w = 1.0 - near * near * O.inv_n2;
            if (w < 0.0) return false;
            O.nmax = min(KK, (int)(w * KK * (1.0 + 1e-9)) + 1);
        }
    }
    // the linearised minimum, from the slopes at the voxel itself
    const double qx = rx * fmax(0.0, -sg * gx * (hz ? (hy ? x11 : x01) : (hy ? x10 : x00)));
    const double qy = ry * fmax(0.0, -sg * gy * (hz ? (hx ? y11 : y01) : (hx ? y10 : y00)));
    const double qz = rz * fmax(0.0, -sg * gz * (hy ? (hx ? z11 : z01) : (hx ? z10 : z00)));
    const double den = O.norm2 + qx * qx + qy * qy + qz * qz;
    ca = cb = cc = 0;
    if (d * d <= den) {   // then the minimum lies within dta
        const double k = K * fabs(d0) / den, ex = qx * k, ey = qy * k, ez = qz * k;
        if (ex <= K && ey <= K && ez <= K) {   // (not NaN)
            int a = (int)(ex + 0.5), b = (int)(ey + 0.5), c = (int)(ez + 0.5);
            if (a * a + b * b + c * c > KK) {
                a = (int)ex;
                b = (int)ey;
                c = (int)ez;
            }
            if (a * a + b * b + c * c <= KK) {
                ca = O.sx ? -a : a;
                cb = O.sy ? -b : b;
                cc = O.sz ? -c : c;
            }
        }
    }
    return true;
}

// The offsets (a, b, c) of one row (fixed a, b) of an octant.  Inside the
// octant's cell the trilinear value is formed factor by factor, the same
// products and sums in the same order as the definition's expression, and
// v - dr = al + be c is linear in c, so the test function sab/dta^2 + c^2
// st^2/dta^2 + (al + be c)^2/norm^2 is a convex quadratic in c: if its continuous
// minimum exceeds 1 (by 1e-9, far beyond rounding) no offset passes, and else
// the two lattice points around that minimum decide, unless both come within
// 1e-9 of 1: then the row is walked.  So are rows whose values exceed norm
// 1e5-fold, where rounding could reach 1e-9, and rows that leave the cell, these
// with the general evaluation.
__device__ __forceinline__ bool row_passes(const GammaArgs& A, const GammaLattice& L,
                                           const Octant& O, int a, int b) {
#pragma clang fp contract(off)
    const int nx = A.nx, ny = A.ny, nz = A.nz, K = A.K;
    const int left = O.nmax - a * a - b * b;
    if (left < 0) return false;
    const double fx = O.ix + L.vx[0][a + K], fy = O.iy + L.vx[1][b + K];
    if (fx < 0.0 || fx > nx - 1 || fy < 0.0 || fy > ny - 1) return false;
    int xf = (int)floor(fx), yf = (int)floor(fy);
    if (xf > nx - 2) xf = nx > 1 ? nx - 2 : 0;
    if (yf > ny - 2) yf = ny > 1 ? ny - 2 : 0;
    const bool cell = xf == O.x0 && yf == O.y0;
    const double tx = fx - O.x0, ty = fy - O.y0;
    const double c00 = O.v[0] * (1 - tx) + O.v[1] * tx, c10 = O.v[2] * (1 - tx) + O.v[3] * tx;
    const double c01 = O.v[4] * (1 - tx) + O.v[5] * tx, c11 = O.v[6] * (1 - tx) + O.v[7] * tx;
    const double c0 = c00 * (1 - ty) + c10 * ty, c1 = c01 * (1 - ty) + c11 * ty;
    const double sab = L.cm[0][a + K] * L.cm[0][a + K] + L.cm[1][b + K] * L.cm[1][b + K];
    // one offset of the row, by the definition; g: its test value
    auto test = [&](int c, double& g) {
        g = 2.0;
        const double fz = O.iz + L.vx[2][c + K];
        if (fz < 0.0 || fz > nz - 1) return false;
        int zf = (int)floor(fz);
        if (zf > nz - 2) zf = nz > 1 ? nz - 2 : 0;
        double v;
        if (cell && zf == O.z0) {
            const double tz = fz - O.z0;
            v = c0 * (1 - tz) + c1 * tz;
        } else if (!trilinear(A.ev, nx, ny, nz, fx, fy, fz, v)) {
            return false;
        }
        const double r2 = sab + L.cm[2][c + K] * L.cm[2][c + K];
        return offset_passes(A, r2, v, O.dr, O.norm2, O.inv_n2, g);
    };
    // |c| runs from lo to hi outward (the zero offset is tested apart); at
    // the grid's upper face only c = 0 stays inside
    const int lo = O.sz || (a == 0 && b == 0) ? 1 : 0;
    int hi = (int)sqrtf((float)left + 0.5f);
    if (hi > K) hi = K;
    if (!O.sz && O.iz + 1 >= nz) hi = 0;
    if (hi < lo) return false;
    const int dir = O.sz ? -1 : 1;
    const double size = fabs(c0) + fabs(c1);
    if (A.use_bound && cell && size * size * O.inv_n2 < 1e10) {
        const double t0 = (double)(O.iz - O.z0), h = L.vx[2][K + 1];
        const double al = (c0 + (c1 - c0) * t0) - O.dr, be = (c1 - c0) * h * dir;   // per |c|
        const double qa = L.cm[2][K + 1] * L.cm[2][K + 1] * A.inv_dta2;
        const double rest = (1.0 + 1e-9) - sab * A.inv_dta2;
        const double den = qa * O.norm2 + be * be, ab = al * be;
        if (ab >= 0.0) {   // rising in |c|
            if (al * al * O.inv_n2 > rest) return false;
        } else if (al * al * qa > rest * den) {
            return false;
        }
        const double cs = -ab / den;
        if (cs < 1e6) {   // (not NaN)
            const int k0 = min(max((int)fmax(cs, 0.0), lo), hi), k1 = min(k0 + 1, hi);
            double g0, g1;
            if (test(dir * k0, g0) || test(dir * k1, g1)) return true;
            if (fmin(g0, g1) > 1.0 + 1e-9) return false;
        }
    }
    for (int k = lo; k <= hi; ++k) {
        double gk;
        if (test(dir * k, gk)) return true;
    }
    return false;
}

__device__ __forceinline__ double lane_value(double x, int lane) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ int lane_value(int x, int lane) {
    return __builtin_amdgcn_readlane(x, lane);
}

// Pass 1 of the gamma index: the threshold, then the zero offset (|o|^2 /
// dta^2 = 0 / dta^2) of every reference voxel.  A voxel failing there joins the
// list of voxels to search.  Workgroups take kTile voxels at a time and append
// their finds at once: an atomic per wave and round on the one list counter
// was the kernel's time (plan map of 13.1M voxels: 410 us then, 66 us now; the
// reference's bytes alone take 21 us).
constexpr int kTile = 2048;
__global__ void __launch_bounds__(256) k_gamma_screen(GammaArgs A) {
#pragma clang fp contract(off)
    __shared__ unsigned found[kTile];
    __shared__ unsigned nfound, base;
    __shared__ unsigned long long red[8];
    const int nx = A.nx, ny = A.ny, nz = A.nz;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the maximum of the reference from k_max's partial ones
    const double* part = reinterpret_cast<const double*>(A.buf + kCountWords);
    double m = 0.0;
    for (int k = threadIdx.x; k < A.n_max; k += 256) m = fmax(m, part[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    double* redm = reinterpret_cast<double*>(red);
    if (lane == 0) redm[wave] = m;
    if (threadIdx.x == 0) nfound = 0;
    __syncthreads();
    m = fmax(fmax(redm[0], redm[1]), fmax(redm[2], redm[3]));
    if (blockIdx.x == 0 && threadIdx.x == 0) A.buf[1] = (unsigned long long)__double_as_longlong(m);
    const double thr_abs = A.thresh * m;
    unsigned ne = 0, np = 0;
    const unsigned ntile = (A.nv + kTile - 1) / kTile;
    for (unsigned tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const unsigned t0 = tile * kTile + threadIdx.x;
        double dr8[kTile / 256];
#pragma unroll
        for (int k = 0; k < kTile / 256; ++k) {
            const unsigned i = t0 + 256 * k;
            dr8[k] = i < A.nv ? A.ref[A.v0 + i] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kTile / 256; ++k) {
            const unsigned i = t0 + 256 * k;
            const double dr = dr8[k];
            bool hard = false;
            if (i < A.nv && dr >= thr_abs && dr > 0.0) {
                ne++;
                int ix, iy, iz;
                voxel_of(A, A.v0 + i, ix, iy, iz);
                const double norm = A.dd * (A.local ? dr : m);
                double de;
                bool pass = false;
                if (trilinear(A.ev, nx, ny, nz, (double)ix, (double)iy, (double)iz, de))
                    pass = 0.0 / (A.dta * A.dta) + (de - dr) * (de - dr) / (norm * norm) <= 1.0;
                if (pass) np++;
                else hard = true;
            }
            const unsigned long long mk = __ballot(hard);
            if (mk) {
                unsigned at = 0;
                if (lane == 0) at = atomicAdd(&nfound, (unsigned)__popcll(mk));
                at = __builtin_amdgcn_readfirstlane(at);
                if (hard) found[at + __popcll(mk & ((1ull << lane) - 1ull))] = i;
            }
        }
        __syncthreads();
        const unsigned n = nfound;
        __syncthreads();   // every thread has read it before the next tile adds to it
        if (n) {
            if (threadIdx.x == 0) {
                base = (unsigned)atomicAdd(&A.buf[0], (unsigned long long)n);
                nfound = 0;
            }
            __syncthreads();
            for (unsigned k = threadIdx.x; k < n; k += 256) A.list[base + k] = found[k];
            __syncthreads();
        }
    }
    const unsigned long long se = wave_sum64(ne), sp = wave_sum64(np);
    __syncthreads();
    if (lane == 0) {
        red[wave] = se;
        red[4 + wave] = sp;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long* slot = A.buf + kLine * (1 + blockIdx.x % kSlots);
        const unsigned long long e = red[0] + red[1] + red[2] + red[3];
        const unsigned long long p = red[4] + red[5] + red[6] + red[7];
        if (e) atomicAdd(slot, e);
        if (p) atomicAdd(slot + 1, p);
    }
}

// Pass 2: the listed voxels' remaining offsets.  A wave takes 8 voxels, 8
// lanes each, one octant a lane: most octants are closed by the bound of
// octant_open or decided by the one offset it names, in a few hundred
// operations with all lanes busy.  The octants left open (a band around the
// boundary; all of them where dta is above a voxel) are then searched one after
// another by the whole wave, a row of offsets per lane.  kOwn: before that, while
// their rows are no more than the whole wave would take for the open ones, each
// lane walks its own octant, outward from the voxel, until one of its voxel's
// has passed.  Bound by FP64 issue.  One thread walking all of a voxel's
// rows took 2876 us for a plan map's list (256 x 256 x 200, 82 % passing), its
// waves waiting for their longest lanes, against 407 us so; on 40 x 40 x 150,
// where one walk's latency is the time, 663 against 31 us.
template <bool kOwn>
__global__ void __launch_bounds__(256) k_gamma_search(GammaArgs A) {
    const unsigned nl = (unsigned)A.buf[0];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & 7;
    if (blockIdx.x * 32u >= nl) return;
    __shared__ GammaLattice L;
    __shared__ unsigned red[4];
    fill_lattice(A, L);
    const int nx = A.nx, ny = A.ny, nz = A.nz, K = A.K;
    unsigned np = 0;
    for (unsigned k0 = (blockIdx.x * 4u + wave) * 8u; k0 < nl; k0 += gridDim.x * 32u) {
        const unsigned k = k0 + (lane >> 3);
        Octant O;
        bool open = false, pass = false;
        O.ix = O.iy = O.iz = O.x0 = O.y0 = O.z0 = 0;
        O.dr = O.norm2 = O.inv_n2 = 0.0;
        O.nmax = K * K;
        O.sx = sub & 1;
        O.sy = (sub >> 1) & 1;
        O.sz = sub >> 2;
#pragma unroll
        for (int j = 0; j < 8; ++j) O.v[j] = 0.0;
        if (k < nl) {
            const size_t i = A.v0 + A.list[k];
            voxel_of(A, i, O.ix, O.iy, O.iz);
            O.dr = A.ref[i];
            const double norm = norm_of(A, O.dr);
            O.norm2 = norm * norm;
            O.inv_n2 = 1.0 / O.norm2;
            open = !((O.sx && O.ix == 0) || (O.sy && O.iy == 0) || (O.sz && O.iz == 0));
            if (open) {
                O.x0 = O.ix - O.sx;
                O.y0 = O.iy - O.sy;
                O.z0 = O.iz - O.sz;
                if (O.x0 > nx - 2) O.x0 = nx > 1 ? nx - 2 : 0;
                if (O.y0 > ny - 2) O.y0 = ny > 1 ? ny - 2 : 0;
                if (O.z0 > nz - 2) O.z0 = nz > 1 ? nz - 2 : 0;
                const int ox = nx > 1 ? 1 : 0;
                const size_t oy = ny > 1 ? (size_t)nx : 0, oz = nz > 1 ? (size_t)nx * ny : 0;
                const double* p = A.ev + ((size_t)O.z0 * ny + O.y0) * nx + O.x0;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    O.v[j] = p[(j & 1 ? ox : 0) + (j & 2 ? oy : 0) + (j & 4 ? oz : 0)];
                if (A.use_bound) {
                    int a, b, c;
                    open = octant_open(A, L, O, a, b, c);
                    if (open && (a | b | c))
                        pass = offset_test(A, L, O.ix, O.iy, O.iz, a, b, c, O.dr, O.norm2,
                                           O.inv_n2);
                }
            }
        }
        unsigned long long done = __ballot(pass);        // bit of any octant of a passing voxel
        unsigned long long todo = __ballot(open);
        auto drop_passed = [&]() {
            // all bits of a voxel's group when one of them passed
            unsigned long long g = done | (done >> 4);
            g |= g >> 2;
            g |= g >> 1;
            g &= 0x0101010101010101ull;
            todo &= ~(g * 0xFFull);
            return g;
        };
        drop_passed();
        // rows (|a| - sx, |b| - sy) on a square; the whole wave takes an octant's 64
        // at a time, and about two rows' time to hand it round
        if (kOwn && todo) {
            int nm = (todo >> lane) & 1 ? O.nmax : 0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) nm = max(nm, __shfl_xor(nm, o));
            const int side = min((int)sqrtf((float)nm + 0.5f), K) + 1, rows = side * side;
            for (int r = 0, q = 0, u = 0;
                 r < rows && rows - r <= __popcll(todo) * (2 + (rows + 63) / 64); ++r) {
                bool p = false;
                if (((todo >> lane) & 1) && q + O.sx <= K && u + O.sy <= K)
                    p = row_passes(A, L, O, O.sx ? -(q + 1) : q, O.sy ? -(u + 1) : u);
                const unsigned long long hit = __ballot(p);
                if (hit) {
                    done |= hit;
                    drop_passed();
                }
                if (++u == side) {
                    u = 0;
                    ++q;
                }
                if (r + 1 == rows) todo = 0;
            }
        }
        while (todo) {
            const int l = __builtin_ctzll(todo);
            todo &= todo - 1;
            Octant U;   // the lane's octant, uniform over the wave
            U.ix = lane_value(O.ix, l);
            U.iy = lane_value(O.iy, l);
            U.iz = lane_value(O.iz, l);
            U.x0 = lane_value(O.x0, l);
            U.y0 = lane_value(O.y0, l);
            U.z0 = lane_value(O.z0, l);
            U.sx = l & 1;
            U.sy = (l >> 1) & 1;
            U.sz = (l >> 2) & 1;
            U.nmax = lane_value(O.nmax, l);
            U.dr = lane_value(O.dr, l);
            U.norm2 = lane_value(O.norm2, l);
            U.inv_n2 = lane_value(O.inv_n2, l);
#pragma unroll
            for (int j = 0; j < 8; ++j) U.v[j] = lane_value(O.v[j], l);
            const int n = min((int)sqrtf((float)U.nmax + 0.5f), K) + 1;
            const float inv = 1.0f / (float)n;
            bool hit = false;
            for (int r0 = 0; r0 < n * n && !hit; r0 += 64) {
                const int r = r0 + lane, q = (int)(((float)r + 0.5f) * inv), u = r - q * n;
                const int a = U.sx ? -(q + 1) : q, b = U.sy ? -(u + 1) : u;
                bool p = false;
                if (r < n * n && q + U.sx <= K && u + U.sy <= K) p = row_passes(A, L, U, a, b);
                hit = __ballot(p) != 0ull;
            }
            if (hit) {
                done |= 1ull << l;
                drop_passed();
            }
        }
        np += (unsigned)__popcll(drop_passed());
    }
    if (lane == 0) red[wave] = np;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned s = red[0] + red[1] + red[2] + red[3];
        if (s) atomicAdd(A.buf + kLine * (1 + blockIdx.x % kSlots) + 1, (unsigned long long)s);
    }
}

// Partial maxima of a non-negative double array (NaN and negative values
// count as 0), one per workgroup, for k_gamma_screen; workgroup 0 zeroes the
// counters (a kernel, not a memset node, so the sequence can be captured).
// No atomics: with one per wave on one address 13.1M voxels took 64 us, so 18.
__global__ void __launch_bounds__(256) k_max(const double* a, size_t n, unsigned long long* buf) {
    __shared__ double red[4];
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < kCountWords; k += 256) buf[k] = 0ull;
    const size_t stride = (size_t)gridDim.x * 256;
    size_t i = blockIdx.x * (size_t)256 + threadIdx.x;
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    for (; i + 3 * stride < n; i += 4 * stride)
#pragma unroll
        for (int k = 0; k < 4; ++k) m[k] = fmax(m[k], a[i + k * stride]);
    for (; i < n; i += stride) m[0] = fmax(m[0], a[i]);
    double t = fmax(fmax(m[0], m[1]), fmax(m[2], m[3]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t = fmax(t, __shfl_xor(t, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0)
        reinterpret_cast<double*>(buf + kCountWords)[blockIdx.x] =
            fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// Zero a few counters (a kernel, not a memset node, so the sequence can be
// captured in a graph).
__global__ void k_zero_u64(unsigned long long* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

int blocks_for(size_t n, int block, int cap) {
    size_t g = (n + block - 1) / block;
    if (g > (size_t)cap) g = cap;
    if (g < 1) g = 1;
    return (int)g;
}

// Workgroups of k_max: at least 2048 values each, at most kGammaMaxParts.
int max_blocks(size_t n) { return blocks_for(n, 2048, kGammaMaxParts); }

}  // namespace

hipError_t launch_gamma(const double* ref, const double* ev, int nx, int ny, int nz, int interp,
                        double dta, double dx, double dy, double dz, double dd, double thresh,
                        double inv_dta2, int local, int use_bound, unsigned long long* buf,
                        unsigned* list, unsigned cap, hipStream_t s) {
    if (interp < 1 || interp > kMaxK || cap < 1) return hipErrorInvalidValue;
    const size_t nvox = (size_t)nx * ny * nz;
    GammaArgs A{ref, ev, nx, ny, nz, interp, dta / interp, dta, dx, dy, dz, dd, thresh, inv_dta2,
                local, use_bound, 1.0 / nx, 1.0 / ny, 0, 0, max_blocks(nvox), buf, list};
    // Above a voxel every octant is open, and mostly passes near the voxel; with
    // few offsets per octant the whole wave is mostly idle (120 x 120 x 120 voxels
    // of 1 mm, own octants first against the whole wave alone: dta 3 mm, 2 offsets
    // per dta 793 and 6658 us, 10 790 and 4268; dta 0.5 mm, 2 offsets 693 and 1765,
    // 3 946 and 1400; 4 1390 and 1260, 10 1665 and 1555)
    const bool own = !use_bound || interp <= 3;
    // a grid beyond the list's capacity goes in passes of cap voxels, so that
    // the list cannot overflow
    for (size_t v0 = 0; v0 < nvox; v0 += cap) {
        A.v0 = v0;
        A.nv = (unsigned)std::min<size_t>(cap, nvox - v0);
        hipError_t e = hipSuccess;
        if (v0 && (e = launch_zero_u64(buf, 1, s)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_gamma_screen, dim3(blocks_for(A.nv, kTile, 2048)), dim3(256), 0, s, A);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        // the list's length is on the device: at most 32 voxels a workgroup,
        // a stride over the list beyond 2048 workgroups
        const auto search = own ? k_gamma_search<true> : k_gamma_search<false>;
        hipLaunchKernelGGL(search, dim3(blocks_for(A.nv, 32, 2048)), dim3(256), 0, s, A);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_max(const double* a, size_t n, unsigned long long* buf, hipStream_t s) {
    hipLaunchKernelGGL(k_max, dim3(max_blocks(n)), dim3(256), 0, s, a, n, buf);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_u64, dim3((n + 63) / 64), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

}  // namespace sde
