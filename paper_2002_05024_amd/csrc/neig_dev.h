// neig_dev.h -- device-side building blocks shared by the libneig kernels (gfx950).
//
// The 2x2 standardisation of a real Schur block (Section 2, eq. 4), the
// negligible-subdiagonal test, the rule of nibble 0, and wavefront reductions.
// Everything is FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define NEIG_EPS 2.220446049250313e-16      // 2^-52
#define NEIG_DBL_MIN 2.2250738585072014e-308

typedef double neig_d4 __attribute__((ext_vector_type(4)));

// Column-major element access.
#define AT(M, ld, i, j) (M)[(size_t)(j) * (size_t)(ld) + (size_t)(i)]

// Smallest m * (m + 1) * 16 + 4096 byte LDS budget fits NEIG_SMALL_MAX (see the host).
#define NEIG_SMALL_MAX 96
#define NEIG_CHASE_MAX 96   // rows/cols of U in one chase window
#define NEIG_MAX_CHAINS 32

// nibble 0: the share of its window (percent) that an AED must deflate for another AED
// to follow at once, for an active block of m rows.  A sweep's cost grows with m, an
// AED's does not, so small blocks sweep more readily.  A dense matrix's form, whose
// windows deflate little, would do so at any order; a random matrix loses by it from
// some order on: by 33 percent and more above 512 rows, by 20 percent above 3000.
// (The second line is not sharp: with 20 instead of 14 the whole reduction of one random
// matrix took 3% less at orders 2500 and 2600, 2% more at 2800, 7% more at 3000, 6% more
// at 4000, and that of a dense one 1 to 7% less at every order.)  Measured on MI355X,
// ms at 14 / 20 / 33 / 45 percent:
//   order   512: dense 65.2 / 65.3 / 52.9 / 46.0, random 21.8 / 22.6 / 21.6 / 21.8
//   order   513: dense 63.9 / 59.5 / 52.9,        random 23.6 / 22.9 / 26.4
//   order  1500: dense 218 / 209 / 190 / 173,     random 64.0 / 60.8 / 69.0 / 77.6
//   order  2500: dense 412 / 401 / 372,           random 107.5 / 104.5 / 116.1
//   order  3000: dense 520 / 505 / 492,           random 113.8 / 121.9 / 149.5
//   order  4000: dense 788 / 772 / 744,           random 170.8 / 180.7 / 224.4
__host__ __device__ inline int nibble_single(int m) { return m <= 512 ? 45 : m <= 3000 ? 20 : 14; }

// The same in the batched solver, where one workgroup does both (ms at 14 / 20 / 45
// percent: 256 problems of order 32 to 300 28.0 / 27.1 / 25.4, 512 of order 32 to 1024
// 233 / 231 / 248).
__host__ __device__ inline int nibble_batched(int m) { return m <= 256 ? 45 : 20; }

// Standardisation of one 2x2 block of a real Schur form (Section 2, eq. 4).
// Result: a rotation G = [[cs -sn][sn cs]] and the block G^T B G, which is upper
// triangular when the eigenvalues are real and otherwise has equal diagonal
// entries and off-diagonal entries of opposite sign.
//
// Construction (two angles, composed):
//  1. Rotating by t changes the diagonal difference to
//     (a - d) cos 2t + (b + c) sin 2t, so tan 2t1 = (d - a) / (b + c) gives a
//     block [[m b1][c1 m]], m the mean of the diagonal.  tan t1 is taken as the
//     root of modulus <= 1 of tan 2t1 = 2 tan t1 / (1 - tan^2 t1).
//  2. The eigenvalues of that block are m +- sqrt(b1 c1).  If b1 and c1 have
//     opposite signs the pair is complex and the block is final.  Otherwise
//     rotating it by t2 leaves (2,1) entry c1 cos^2 t2 - b1 sin^2 t2, which a
//     rotation with (cos t2, sin t2) proportional to (sqrt|b1|, sqrt|c1|)
//     annihilates.
// The output block is formed from B itself by the composed rotation (one
// rounding step on the diagonal), and the entry that is zero in exact
// arithmetic is set to zero.
struct Std2 {
    double a, b, c, d, cs, sn;
};

// G^T [[a b][c d]] G for G = [[C -S][S C]]: out = (0,0), (0,1), (1,0), (1,1).
__device__ __forceinline__ void rot2_similarity(double a, double b, double c, double d, double C, double S,
                                                double (&out)[4]) {
    const double p00 = a * C + b * S, p01 = b * C - a * S;  // B G, first row
    const double p10 = c * C + d * S, p11 = d * C - c * S;  // B G, second row
    out[0] = C * p00 + S * p10;
    out[1] = C * p01 + S * p11;
    out[2] = C * p10 - S * p00;
    out[3] = C * p11 - S * p01;
}

__device__ __forceinline__ Std2 std2x2(double a, double b, double c, double d) {
    Std2 o{a, b, c, d, 1.0, 0.0};
    if (c == 0.0) return o;  // already triangular
    const double big = fmax(fmax(fabs(a), fabs(b)), fmax(fabs(c), fabs(d)));
    const double inv = 1.0 / big;
    // angle 1 (scale-free, so computed on the scaled entries)
    const double u = d * inv - a * inv, v = b * inv + c * inv;
    double t1 = 0.0;
    if (u != 0.0) {
        const double h = hypot(u, v);
        t1 = u / (v >= 0.0 ? v + h : v - h);
    }
    const double C1 = 1.0 / sqrt(1.0 + t1 * t1), S1 = t1 * C1;
    double e[4];
    rot2_similarity(a, b, c, d, C1, S1, e);
    if ((e[1] > 0.0 && e[2] < 0.0) || (e[1] < 0.0 && e[2] > 0.0)) {
        const double m = 0.5 * (e[0] + e[3]);
        o.a = m; o.b = e[1]; o.c = e[2]; o.d = m; o.cs = C1; o.sn = S1;
        return o;
    }
    // angle 2 (real pair)
    const double p = sqrt(fabs(e[1] * inv)), q = sqrt(fabs(e[2] * inv));
    const double r = hypot(p, q);
    const double C2 = (r > 0.0) ? p / r : 1.0, S2 = (r > 0.0) ? q / r : 0.0;
    const double C = C1 * C2 - S1 * S2, S = S1 * C2 + C1 * S2;
    rot2_similarity(a, b, c, d, C, S, e);
    o.a = e[0]; o.b = e[1]; o.c = 0.0; o.d = e[3]; o.cs = C; o.sn = S;
    return o;
}

// |h(k,k-1)| negligible next to its diagonal neighbours (classic criterion).
__device__ __forceinline__ bool negligible_sub(double sub, double dkm1, double dk, double hnorm, double smlnum) {
    double s = fabs(dkm1) + fabs(dk);
    if (s == 0.0) s = hnorm;
    return fabs(sub) <= fmax(smlnum, NEIG_EPS * s);
}

// One step of a wavefront reduction: the value that the given cross-lane move brings
// to a lane, or `none` where it brings nothing.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v, double none) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(none), __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(none), __double2hiint(v), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double last_lane(double v) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Sum and maximum over a wavefront, in every lane; all 64 lanes call.  Shifts
// within the rows of 16 lanes, then the rows' last lanes to the rows after them:
// register moves, about 25 cycles a step, where a shuffle goes through the LDS
// unit (about 130).
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0x111, 0xf>(v, 0.0);
    v += dpp_move<0x112, 0xf>(v, 0.0);
    v += dpp_move<0x114, 0xf>(v, 0.0);
    v += dpp_move<0x118, 0xf>(v, 0.0);
    v += dpp_move<0x142, 0xa>(v, 0.0);
    v += dpp_move<0x143, 0xc>(v, 0.0);
    return last_lane(v);
}

__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_move<0x111, 0xf>(v, v));
    v = fmax(v, dpp_move<0x112, 0xf>(v, v));
    v = fmax(v, dpp_move<0x114, 0xf>(v, v));
    v = fmax(v, dpp_move<0x118, 0xf>(v, v));
    v = fmax(v, dpp_move<0x142, 0xa>(v, v));
    v = fmax(v, dpp_move<0x143, 0xc>(v, v));
    return last_lane(v);
}

// Eigenvalues of a 2x2 block (any form): returns real parts and |imag|.
__device__ __forceinline__ void eig2x2(double a, double b, double c, double d, double *r1, double *i1, double *r2,
                                       double *i2) {
    double p = 0.5 * (a - d);
    double disc = p * p + b * c;
    double m = 0.5 * (a + d);
    if (disc >= 0.0) {
        double r = sqrt(disc);
        *r1 = m + r; *r2 = m - r; *i1 = 0.0; *i2 = 0.0;
    } else {
        double r = sqrt(-disc);
        *r1 = m; *r2 = m; *i1 = r; *i2 = -r;
    }
}
