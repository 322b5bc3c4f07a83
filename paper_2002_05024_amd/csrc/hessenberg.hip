// hessenberg.hip -- reduction of a general matrix to upper Hessenberg form,
// A = Q1 H Q1^T (Section 2, eq. 3), by the standard blocked algorithm of
// Section 3.1 (Fig. 2): panels of reflectors I - tau v v^T accumulated in the
// compact WY form I - V T V^T together with Y = A V T; then the trailing update
// A <- (I - V T V^T)^T (A - Y V^T) and the top-part update A <- A - Y V^T.
//
// Per panel column (three launches, all on the caller's stream):
//   k_hrd_a   finish the previous reflector (beta, tau, u = V^T v, its v into V, its
//             column of H and of T, the column Y(:, i-1) = tau (A v - Y u)), then
//             apply the panel's earlier reflectors to the new column from the
//             right (a -= Y V(j, :)^T) and sum w = V^T a;
//   k_hrd_b   apply them from the left (a -= V T^T w), and sum the new reflector's
//             norm and V^T (tail);
//   k_hrd_gemv  the large matrix-vector product A(:, j+2:n) v over the trailing
//             part, split over row blocks x column chunks (the memory-bound 20%
//             of the flops); the partial sums go to a workspace and are added by
//             the next k_hrd_a.
// The column kernels leave their sums over the rows (w, the tail norm, u) as
// partial sums per workgroup, which the workgroups of the next launch add for
// themselves in a fixed order, so results do not depend on scheduling.
//
// Per panel (FP64 matrix-core kernels): k_hrd_skinny forms the thin products
// A_top V, Y^T V, A_t^T V and Q V (split over the long dimension), k_hrd_reduce
// sums the partials and applies T (and a correction), and k_hrd_rank applies a
// rank-r update C -= L1 R1^T + L2 R2^T in place.
//
// Index conventions: the panel starts at column k0; its reflectors act on rows
// and columns k0+1..n-1.  "Local row" r = global row - (k0 + 1), 0 <= r < m,
// m = n - k0 - 1.  Reflector i (column j = k0 + i) has v(r) = 0 for r < i,
// v(i) = 1.  V (m x nb) is stored by local rows, Y (n x nb) by global rows.
#include "neig_dev.h"

#define HRD_NB 64        // largest panel width
#define HRD_THREADS 256
#define HRD_GR 512       // rows per workgroup in the large GEMV (two per thread)
#define HRD_GC 256       // vector entries per GEMV workgroup (512 for the largest trailing blocks)
#define HRD_GC_MAX 512

struct HrdState {
    unsigned long long amax;  // bits of max |A|
    double alpha;             // the newest column's entry on the subdiagonal
};

struct HrdArgs {
    double *A;
    double *V, *Y, *T, *Tr;  // V, Y: leading dimension ldw; T: HRD_NB x HRD_NB, Tr its transpose
    double *wpart, *upart;   // per workgroup: 64 partial entries of V^T a and of V^T (tail)
    double *spart;           // per 64 rows: scale and scaled sum of squares of the tail
    double *zpart;           // GEMV partials, chunk-major, leading dimension ldw
    HrdState *st;
    int lda, ldw;
    int n, k0, m, i, jb, nch;  // nch: chunks of the previous GEMV
    int cw;                    // vector entries per GEMV chunk
};

// The vector that the product multiplies is the column's tail times 2^-e, e from the
// tail's own largest exponent and its length, so that its norm is at most 1 and its
// largest entry at least 1 / (4 sqrt m): as safe from overflow and underflow as v
// itself, whatever the column's size beside A's.  The reflector's scaling, which is not
// known yet, follows in k_hrd_a.
// mx: the largest of the scales that k_hrd_b left, 2^em (or 0: no tail).
__device__ __forceinline__ int hrd_exponent(double mx, int m) {
    return __builtin_amdgcn_frexp_exp(mx) + (33 - __clz(m)) / 2;
}

// The tails are multiplied by 2^this before k_hrd_b's sums V^T (tail): as far up as
// the sums allow (a tail's norm is at most max |A| n < 2^17 max |A|), so that a
// subnormal tail's products with V keep their bits, on which V's orthogonality rests.
__device__ __forceinline__ int hrd_lift(const HrdState *st) {
    return max(0, 980 - ((int)(st->amax >> 52) - 1023));
}

extern "C" __global__ void k_hrd_begin(HrdState *st) {
    st->amax = 0ull;
    st->alpha = 0.0;
}

extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_amax(const double *A, int lda, int n, HrdState *st) {
    double mx = 0.0;
    for (int j = blockIdx.x; j < n; j += gridDim.x)
        for (int i = threadIdx.x; i < n; i += HRD_THREADS) mx = fmax(mx, fabs(AT(A, lda, i, j)));
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) atomicMax(&st->amax, (unsigned long long)__double_as_longlong(mx));
}

// Sum of x[e] (e < 16) over the 64 lanes of a wavefront: lane l returns the total
// of entry l % 16.  Halving over the 16 lanes of a row by register moves (mirror,
// half mirror, exchanges within quads), then across the four rows.
template <int CTRL, int S>
__device__ __forceinline__ void hrd_halve(double (&x)[16], bool up) {
#pragma unroll
    for (int k = 0; k < S; ++k) {
        const double send = up ? x[k] : x[k + S];
        const double keep = up ? x[k + S] : x[k];
        x[k] = keep + dpp_move<CTRL, 0xf>(send, 0.0);
    }
}

__device__ __forceinline__ double hrd_sum16(double (&x)[16], int lane) {
    hrd_halve<0x140, 8>(x, (lane & 8) != 0);
    hrd_halve<0x141, 4>(x, (lane & 4) != 0);
    hrd_halve<0x4E, 2>(x, (lane & 2) != 0);
    hrd_halve<0xB1, 1>(x, (lane & 1) != 0);
    double v = x[0];
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// The column kernels.  A workgroup has 64 RG rows, one per lane; wave 4 g + q takes
// the panel columns q, q + 4, ... of row group g, so a row's 64 entries of V and Y
// are 16 loads per lane, all in flight at once.  Sums over the rows leave 64
// partial entries per workgroup in memory, and every workgroup of the next launch
// adds all of them for itself: no workgroup waits for another within a launch, and
// the long product k_hrd_gemv, which needs none of these sums, starts right after
// k_hrd_b.  What bounds them is latency: a round of loads from L2, the sums, a few
// barriers.  Measured on MI355X, us per column (k_hrd_a, k_hrd_b, the product):
// order 1000: 7.5 + 5.5 + 3.5, before 15.7 + 15.1 + 14.6 (one thread per row, and
// the last workgroup to finish added the sums; 512 x 256 tiles in the product);
// order 8000, whole reduction with Q1: 831 -> 491 ms, of which the products take
// 273 ms (5 TB/s).  Four row groups per workgroup instead of two on long columns:
// 12.8 + 8.3 instead of 9.1 + 6.8.

// Column sums over nblk workgroups' partials (stride 64), in a fixed order: wave p
// adds blocks p, p + NW, ...; out[0..63] in LDS after a barrier by the caller.
template <int NW>
__device__ __forceinline__ void hrd_block_sums(const double *part, int nblk, double (*red)[HRD_NB]) {
    const int c = threadIdx.x & 63, p = threadIdx.x >> 6;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    int b = p;
    for (; b + 3 * NW < nblk; b += 4 * NW) {
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] += part[(size_t)(b + u * NW) * HRD_NB + c];
    }
    for (; b < nblk; b += NW) a[0] += part[(size_t)b * HRD_NB + c];
    red[p][c] = (a[0] + a[1]) + (a[2] + a[3]);
}

template <int NW>
__device__ __forceinline__ double hrd_add_waves(double (*red)[HRD_NB], int c) {
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < NW; ++p) s += red[p][c];
    return s;
}

// Partial entries 4 e + q of this workgroup (e = lane % 16 of wave 4 g + q) to memory.
template <int RG>
__device__ __forceinline__ void hrd_store_part(double v, double *part, double (*red)[HRD_NB], int lane, int q, int g) {
    if (RG == 1) {
        if (lane < 16) part[(size_t)blockIdx.x * HRD_NB + 4 * lane + q] = v;
    } else {
        if (lane < 16) red[g][4 * lane + q] = v;
        __syncthreads();
        if (threadIdx.x < HRD_NB) part[(size_t)blockIdx.x * HRD_NB + threadIdx.x] = hrd_add_waves<RG>(red, threadIdx.x);
    }
}

// Finish reflector i-1: beta, tau and u = V^T v from the sums of k_hrd_b; its vector
// into V, its column of H, Y(:, i-1) = tau (A v - Y u), its column of T.  Then apply
// the panel's earlier reflectors to column j = k0 + i from the right,
// a -= Y V(i-1, :)^T, and sum V^T a.
template <int RG>
__global__ void __launch_bounds__(HRD_THREADS * RG) k_hrd_a(HrdArgs p) {
    constexpr int NW = 4 * RG;
    __shared__ double red[NW][HRD_NB];
    __shared__ double comb[3][4][64 * RG];
    __shared__ double us[HRD_NB], vs[HRD_NB], coef[3];
    __shared__ int cexp[2];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), q = wave & 3, g = wave >> 2;
    const int i = p.i, ip = i - 1, j = p.k0 + i;
    const int lr = g * 64 + lane;
    const int r = blockIdx.x * 64 * RG + lr;
    const bool in = r < p.m;
    const int rr = in ? r : p.m - 1;
    const size_t gr = (size_t)p.k0 + 1 + rr;
    const bool last = i == p.jb;  // the panel's last launch only finishes reflector i-1
    const int nblk = gridDim.x;
    const int lift = hrd_lift(p.st);
    // the first wave's part of the reflector: its loads go out before all others
    double nsc[2], nsq[2], alpha = 0.0, vr = 0.0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int b = lane + 64 * e;
        nsc[e] = nsq[e] = 0.0;
        if (wave == 0 && b < nblk * RG) {
            nsc[e] = p.spart[2 * b];
            nsq[e] = p.spart[2 * b + 1];
        }
    }
    if (wave == 0) {
        alpha = p.st->alpha;
        vr = AT(p.V, p.ldw, ip, max(min(lane, ip - 1), 0));
    }
    double yv[16], vv[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        // columns from ip on: the last one again, and a zero in its place
        const int c = 4 * e + q, cc = max(min(c, ip - 1), 0);
        const double ye = AT(p.Y, p.ldw, gr, cc), ve = AT(p.V, p.ldw, rr, cc);
        yv[e] = c < ip ? ye : 0.0;
        vv[e] = c < ip ? ve : 0.0;
    }
    const double old = AT(p.A, p.lda, gr, j - 1);
    const double aj = AT(p.A, p.lda, gr, j);  // column j, not yet touched by this panel
    double tv[16 / RG];  // row `lane` of T, columns wave, wave + NW, ... (used by the first workgroup)
#pragma unroll
    for (int e = 0; e < 16 / RG; ++e) {
        const int c = wave + NW * e;
        const double te = p.T[lane + max(min(c, ip - 1), 0) * HRD_NB];
        tv[e] = c < ip ? te : 0.0;
    }
    double z = 0.0;
    {
        double zz[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int ch = q + 4 * u;
            const double ze = p.zpart[(size_t)min(ch, p.nch - 1) * p.ldw + rr];
            zz[u] = ch < p.nch ? ze : 0.0;
        }
        for (int ch = q + 32; ch < p.nch; ch += 4) zz[0] += p.zpart[(size_t)ch * p.ldw + rr];
        z = ((zz[0] + zz[1]) + (zz[2] + zz[3])) + ((zz[4] + zz[5]) + (zz[6] + zz[7]));
    }
    hrd_block_sums<NW>(p.upart, nblk, red);
    if (wave == 0) {
        // the tail's norm: scales are powers of two, so merging them is exact
        double mx = fmax(nsc[0], nsc[1]);
        for (int b = lane + 128; b < nblk * RG; b += 64) mx = fmax(mx, p.spart[2 * b]);
        mx = wave_max(mx);
        double beta = alpha, tau = 0.0, scal = 0.0;
        int ex = 0;
        if (mx > 0.0) {
            const int em = ilogb(mx);
            // by exponents, not by a reciprocal: 2^-em overflows for a subnormal tail
            const double f0 = ldexp(nsc[0], -em), f1 = ldexp(nsc[1], -em);
            double sq = nsq[0] * f0 * f0 + nsq[1] * f1 * f1;
            for (int b = lane + 128; b < nblk * RG; b += 64) {
                const double f = ldexp(p.spart[2 * b], -em);
                sq += p.spart[2 * b + 1] * f * f;
            }
            sq = wave_sum(sq);
            // the norm with alpha, and the reflector, both scaled by 2^-ex, the
            // larger exponent (1 / (alpha - beta) itself may overflow)
            const int ea = alpha != 0.0 && isfinite(alpha) ? ilogb(alpha) : em;
            ex = max(ea, em);
            const double as = ldexp(alpha, -ex);
            const double nrm = sqrt(as * as + ldexp(sq, 2 * max(em - ex, -600)));
            const double bs = alpha >= 0.0 ? -nrm : nrm;
            beta = ldexp(bs, ex);
            tau = (bs - as) / bs;
            scal = 1.0 / (as - bs);
        }
        vs[lane] = lane < ip ? vr : 0.0;
        if (lane == 0) {
            coef[0] = beta;
            coef[1] = tau;
            coef[2] = scal;
            cexp[0] = ex;
            cexp[1] = hrd_exponent(mx, p.m) - ex;
        }
    }
    __syncthreads();
    // v = 2^-ex (tail) scal
    const double beta = coef[0], tau = coef[1], scal = coef[2];
    const int ex = cexp[0], ez = cexp[1];
    if (t < HRD_NB)
        us[t] = t < ip ? fma(scal, ldexp(hrd_add_waves<NW>(red, t), -ex - lift), vs[t]) : 0.0;
    __syncthreads();
    double yu = 0.0, yw = 0.0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        yu = fma(yv[e], us[4 * e + q], yu);
        yw = fma(yv[e], vs[4 * e + q], yw);
    }
    comb[0][q][lr] = z;
    comb[1][q][lr] = yu;
    comb[2][q][lr] = yw;
    if (blockIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < 16 / RG; ++e) {
            const int c = wave + NW * e;
            if (c >= lane) s = fma(tv[e], us[c], s);  // us is zero from ip on
        }
        red[wave][lane] = s;
    }
    __syncthreads();
    if (blockIdx.x == 0 && t < HRD_NB) {
        // column i-1 of T: T(0:i-1, i-1) = -tau T(0:i-1, 0:i-1) u, T(i-1, i-1) = tau
        const double v = t < ip ? -tau * hrd_add_waves<NW>(red, t) : (t == ip ? tau : 0.0);
        p.T[t + (size_t)ip * HRD_NB] = v;
        p.Tr[ip + (size_t)t * HRD_NB] = v;
    }
    z = (comb[0][0][lr] + comb[0][1][lr]) + (comb[0][2][lr] + comb[0][3][lr]);
    yu = (comb[1][0][lr] + comb[1][1][lr]) + (comb[1][2][lr] + comb[1][3][lr]);
    yw = (comb[2][0][lr] + comb[2][1][lr]) + (comb[2][2][lr] + comb[2][3][lr]);
    const double vnew = r < ip ? 0.0 : (r == ip ? 1.0 : ldexp(old, -ex) * scal);
    const double ycol = tau * ((aj + ldexp(z * scal, ez)) - yu);
    const double a = aj - (yw + ycol);  // V(i-1, i-1) = 1
    if (q == 0 && in) {
        AT(p.V, p.ldw, r, ip) = vnew;
        AT(p.Y, p.ldw, gr, ip) = ycol;
        if (r >= ip) AT(p.A, p.lda, gr, j - 1) = (r == ip) ? beta : 0.0;
        if (!last) AT(p.A, p.lda, gr, j) = a;
    }
    if (last) return;
    double x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = in ? (4 * e + q == ip ? vnew : vv[e]) * a : 0.0;
    __syncthreads();  // red is free
    hrd_store_part<RG>(hrd_sum16(x, lane), p.wpart, red, lane, q, g);
}

// Left application a -= V T^T (V^T a) of the earlier reflectors to column j, then
// for its reflector: the scaled sum of squares of the tail and V^T (tail).
template <int RG>
__global__ void __launch_bounds__(HRD_THREADS * RG) k_hrd_b(HrdArgs p) {
    constexpr int NW = 4 * RG;
    __shared__ double red[NW][HRD_NB];
    __shared__ double comb[4][64 * RG];
    __shared__ double ws[HRD_NB], ss[HRD_NB];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), q = wave & 3, g = wave >> 2;
    const int i = p.i, j = p.k0 + i;
    const int lr = g * 64 + lane;
    const int r = blockIdx.x * 64 * RG + lr;
    const bool in = r < p.m;
    const int rr = in ? r : p.m - 1;
    const size_t gr = (size_t)p.k0 + 1 + rr;
    const int lift = hrd_lift(p.st);
    double vv[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int c = 4 * e + q;
        const double ve = AT(p.V, p.ldw, rr, max(min(c, i - 1), 0));
        vv[e] = c < i ? ve : 0.0;
    }
    double a = AT(p.A, p.lda, gr, j);
    if (i > 0) {
        double tv[16 / RG];  // column `lane` of T, rows wave, wave + NW, ...
#pragma unroll
        for (int e = 0; e < 16 / RG; ++e) {
            const int c = wave + NW * e;
            tv[e] = p.Tr[lane + min(c, i - 1) * HRD_NB];  // used for c <= lane < i
        }
        hrd_block_sums<NW>(p.wpart, gridDim.x, red);
        __syncthreads();
        if (t < HRD_NB) ws[t] = hrd_add_waves<NW>(red, t);
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < 16 / RG; ++e) {
            const int c = wave + NW * e;
            if (c <= lane && lane < i) s = fma(tv[e], ws[c], s);  // s = T^T w, T upper triangular
        }
        red[wave][lane] = s;
        __syncthreads();
        if (t < HRD_NB) ss[t] = hrd_add_waves<NW>(red, t);
        __syncthreads();
        double acc = 0.0;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc = fma(vv[e], ss[4 * e + q], acc);
        comb[q][lr] = acc;
        __syncthreads();
        a -= (comb[0][lr] + comb[1][lr]) + (comb[2][lr] + comb[3][lr]);
        if (q == 0 && in) AT(p.A, p.lda, gr, j) = a;
    }
    if (q == 0 && r == i) p.st->alpha = a;
    const double tail = (in && r > i) ? a : 0.0;
    if (q == 0) {
        const double mx = wave_max(fabs(tail));
        const double sc = (mx > 0.0 && mx < INFINITY) ? ldexp(1.0, ilogb(mx)) : (mx > 0.0 || tail != tail ? 1.0 : 0.0);
        const double scl = wave_max(sc);
        const double y = scl > 0.0 ? tail / scl : 0.0;
        const double sq = wave_sum(y * y);
        if (lane == 0) {
            p.spart[2 * (blockIdx.x * RG + g)] = scl;
            p.spart[2 * (blockIdx.x * RG + g) + 1] = sq;
        }
    }
    double x[16];
    const double lifted = ldexp(tail, lift);
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = vv[e] * lifted;
    __syncthreads();  // red is free
    hrd_store_part<RG>(hrd_sum16(x, lane), p.upart, red, lane, q, g);
}

// z(r) = sum over the chunk's entries c of A(k0+1+r, k0+1+c) * 2^-e a(c),
// a = column j's tail (local entries i+1..m-1).  Grid: row blocks x chunks.
// k_hrd_gemv_small, for trailing blocks whose large tiles would leave compute units
// idle: 64 rows per workgroup, the chunk's columns split over its four waves.
extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_gemv_small(HrdArgs p) {
    __shared__ double v[HRD_GC];
    __shared__ double red[4][64];
    const int t = threadIdx.x, lane = t & 63;
    const int q = __builtin_amdgcn_readfirstlane(t >> 6);
    const int c0 = p.i + 1 + blockIdx.y * p.cw;
    const int cn = min(p.cw, p.m - c0);
    const size_t base = (size_t)p.k0 + 1;
    const int r = blockIdx.x * 64 + lane;
    const int rr = min(r, p.m - 1);
    const int per = p.cw >> 2;  // columns per wave, a multiple of 16
    const int f = q * per, l = min(cn, f + per);
    const double *col = p.A + (base + c0) * (size_t)p.lda + base + rr;
    double x[16];
    const size_t ld = (size_t)p.lda;
    // the scales (one per lane: at most 64 groups of rows here), the vector, and the
    // first sixteen columns are on their way together
    const double sc = p.spart[2 * min(lane, (p.m + 63) / 64 - 1)];
    const double a = AT(p.A, p.lda, base + c0 + min(t, cn - 1), p.k0 + p.i);
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = col[(size_t)min(f + u, cn - 1) * ld];
    const int e = hrd_exponent(wave_max(sc), p.m);
    if (t < p.cw) v[t] = t < cn ? ldexp(a, -e) : 0.0;
    __syncthreads();
    double a0 = 0.0, a1 = 0.0;
    for (int c = f; c < l; c += 16) {
#pragma unroll
        for (int u = 0; u < 16; u += 2) {
            a0 = fma(c + u < l ? x[u] : 0.0, v[c + u], a0);
            a1 = fma(c + u + 1 < l ? x[u + 1] : 0.0, v[c + u + 1], a1);
        }
        if (c + 16 < l) {
#pragma unroll
            for (int u = 0; u < 16; ++u) x[u] = col[(size_t)min(c + 16 + u, cn - 1) * ld];
        }
    }
    red[q][lane] = a0 + a1;
    __syncthreads();
    if (t < 64 && r < p.m)
        p.zpart[(size_t)blockIdx.y * p.ldw + r] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
}

extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_gemv(HrdArgs p) {
    __shared__ double v[HRD_GC_MAX];
    const int t = threadIdx.x;
    const int c0 = p.i + 1 + blockIdx.y * p.cw;
    const int cn = min(p.cw, p.m - c0);
    const int j = p.k0 + p.i;
    const size_t base = (size_t)p.k0 + 1;
    double mx = 0.0;
    for (int b = t & 63; b < (p.m + 63) / 64; b += 64) mx = fmax(mx, p.spart[2 * b]);
    const int e = hrd_exponent(wave_max(mx), p.m);
    for (int u = t; u < cn; u += HRD_THREADS) v[u] = ldexp(AT(p.A, p.lda, base + c0 + u, j), -e);
    __syncthreads();
    const int r0 = blockIdx.x * HRD_GR + t, r1 = r0 + HRD_THREADS;
    const bool in0 = r0 < p.m, in1 = r1 < p.m;
    const double *col = p.A + (base + c0) * (size_t)p.lda + base;
    double a0 = 0.0, a1 = 0.0, b0 = 0.0, b1 = 0.0;
    int c = 0;
    if (in1) {
        // sixteen independent loads in flight per lane before their first use
        const size_t ld = (size_t)p.lda;
        for (; c + 8 <= cn; c += 8) {
            const double *c1 = col + (size_t)c * p.lda;
            double x0[8], x1[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                x0[u] = c1[u * ld + r0];
                x1[u] = c1[u * ld + r1];
            }
#pragma unroll
            for (int u = 0; u < 8; u += 2) {
                a0 = fma(x0[u], v[c + u], a0);
                a1 = fma(x1[u], v[c + u], a1);
                b0 = fma(x0[u + 1], v[c + u + 1], b0);
                b1 = fma(x1[u + 1], v[c + u + 1], b1);
            }
        }
        for (; c < cn; ++c) {
            const double *c1 = col + (size_t)c * p.lda;
            a0 = fma(c1[r0], v[c], a0);
            a1 = fma(c1[r1], v[c], a1);
        }
    } else if (in0) {
        for (; c + 2 <= cn; c += 2) {
            const double *c1 = col + (size_t)c * p.lda;
            a0 = fma(c1[r0], v[c], a0);
            b0 = fma(c1[r0 + p.lda], v[c + 1], b0);
        }
        for (; c < cn; ++c) a0 = fma(col[(size_t)c * p.lda + r0], v[c], a0);
    }
    double *z = p.zpart + (size_t)blockIdx.y * p.ldw;
    if (in0) z[r0] = a0 + b0;
    if (in1) z[r1] = a1 + b1;
}

// ---------------------------------------------------------------- panel GEMMs

#define HRD_PAD 34   // LDS row pitch (doubles) of 32-wide operand slices: conflict-free reads

struct SkArgs {
    const double *C;   // trans 0: M x K; trans 1: K x M
    const double *V;   // K x nbc
    double *P;         // partials: split s at P + s * sp, M x nbc, leading dimension M
    size_t sp;
    int ldc, ldv, M, K, nbc, kper, trans;
};

__device__ __forceinline__ neig_d4 hrd_mfma(double a, double b, neig_d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// P_s(i, c) = sum over k in split s of op(C)(i, k) V(k, c): 64 output rows per
// workgroup, K in 32-wide LDS-staged steps, four waves of 16 rows each; the
// next step's operands are loaded into registers while the matrix cores work
// on the current one.
// Operand layouts of v_mfma_f64_16x16x4_f64 (lane l): A(l%16, l/16),
// B(l/16, l%16); accumulator double r of lane l holds D(l/16 + 4r, l%16).
template <int TRANS>
__device__ __forceinline__ void hrd_skinny_body(const SkArgs &p) {
    __shared__ double Cs[64 * HRD_PAD];
    __shared__ double Vs[64 * HRD_PAD];
    const int t = threadIdx.x, lane = t & 63, q = t >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int i0 = blockIdx.x * 64;
    const int ks = blockIdx.y * p.kper;
    const int ke = min(p.K, ks + p.kper);
    neig_d4 acc[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) acc[ct] = (neig_d4){0.0, 0.0, 0.0, 0.0};
    const int nct = (p.nbc + 15) >> 4;
    double rc[8], rv[8];
    auto fetch = [&](int kb) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = t + u * HRD_THREADS;
            int ii, kk;
            if (TRANS == 0) {
                ii = idx & 63;
                kk = idx >> 6;
                rc[u] = (i0 + ii < p.M && kb + kk < ke) ? AT(p.C, p.ldc, i0 + ii, kb + kk) : 0.0;
            } else {
                kk = idx & 31;
                ii = idx >> 5;
                rc[u] = (i0 + ii < p.M && kb + kk < ke) ? AT(p.C, p.ldc, kb + kk, i0 + ii) : 0.0;
            }
            const int vk = idx & 31, vc = idx >> 5;
            rv[u] = (vc < p.nbc && kb + vk < ke) ? AT(p.V, p.ldv, kb + vk, vc) : 0.0;
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = t + u * HRD_THREADS;
            const int ii = TRANS == 0 ? (idx & 63) : (idx >> 5);
            const int kk = TRANS == 0 ? (idx >> 6) : (idx & 31);
            Cs[ii * HRD_PAD + kk] = rc[u];
            Vs[(idx >> 5) * HRD_PAD + (idx & 31)] = rv[u];
        }
    };
    if (ks < ke) fetch(ks);
    for (int kb = ks; kb < ke; kb += 32) {
        store();
        __syncthreads();
        if (kb + 32 < ke) fetch(kb + 32);
#pragma unroll
        for (int k4 = 0; k4 < 32; k4 += 4) {
            const double a = Cs[(16 * q + li) * HRD_PAD + k4 + lk];
            // all four column tiles (V is zero beyond nbc): no runtime branch
            // between the matrix-core instructions
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) acc[ct] = hrd_mfma(a, Vs[(16 * ct + li) * HRD_PAD + k4 + lk], acc[ct]);
        }
        __syncthreads();
    }
    double *P = p.P + (size_t)blockIdx.y * p.sp;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const int col = 16 * ct + li;
        if (ct < nct && col < p.nbc) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int row = i0 + 16 * q + lk + 4 * rr;
                if (row < p.M) P[row + (size_t)col * p.M] = acc[ct][rr];
            }
        }
    }
}

extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_skinny_n(SkArgs p) { hrd_skinny_body<0>(p); }
extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_skinny_t(SkArgs p) { hrd_skinny_body<1>(p); }

struct RdArgs {
    const double *P;   // ns partials of M x nbc (leading dimension M), stride sp
    size_t sp;
    int ns;
    const double *X;   // optional M x nbc (leading dimension ldx): subtract X B
    int ldx;
    const double *B;   // nbc x nbc, leading dimension HRD_NB
    const double *T;   // optional nbc x nbc upper triangular, leading dimension HRD_NB
    double *out;
    int ldo, M, nbc;
};

// out = (sum_s P_s - X B) T, 16 rows per workgroup: thread (row, g) sums the
// partials of columns 4 g.. with eight loads in flight and multiplies by B and T
// from LDS: 19 us at order 1000, 23 at 8000 (64 rows per workgroup and one load
// after another: 119 and 136).
extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_reduce(RdArgs p) {
    __shared__ double xs[16][HRD_NB + 1], xr[16][HRD_NB + 1];
    __shared__ double bt[HRD_NB * HRD_NB];
    const int t = threadIdx.x;
    const int row = t & 15, c0 = 4 * (t >> 4);
    const int i = blockIdx.x * 16 + row;
    const int ii = min(i, p.M - 1);
    double acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const double *q = p.P + ii + (size_t)min(c0 + u, p.nbc - 1) * p.M;
        double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        int k = 0;
        for (; k + 8 <= p.ns; k += 8) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += q[(size_t)(k + e) * p.sp];
        }
        for (; k < p.ns; ++k) s[0] += q[(size_t)k * p.sp];
        acc[u] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
    if (p.X) {
        for (int e = t; e < HRD_NB * HRD_NB; e += HRD_THREADS) bt[e] = p.B[e];
#pragma unroll
        for (int u = 0; u < 4; ++u) xr[row][c0 + u] = c0 + u < p.nbc ? AT(p.X, p.ldx, ii, c0 + u) : 0.0;
        __syncthreads();
        for (int k = 0; k < p.nbc; ++k) {
            const double x = xr[row][k];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = fma(-x, bt[k + (c0 + u) * HRD_NB], acc[u]);
        }
        __syncthreads();
    }
    if (p.T) {
        for (int e = t; e < HRD_NB * HRD_NB; e += HRD_THREADS) bt[e] = p.T[e];
#pragma unroll
        for (int u = 0; u < 4; ++u) xs[row][c0 + u] = acc[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = 0.0;
        for (int k = 0; k < min(c0 + 4, p.nbc); ++k) {
            const double x = xs[row][k];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k <= c0 + u) acc[u] = fma(x, bt[k + (c0 + u) * HRD_NB], acc[u]);
        }
    }
    if (i < p.M) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c0 + u < p.nbc) AT(p.out, p.ldo, i, c0 + u) = acc[u];
    }
}

struct RkArgs {
    double *C;
    const double *L1, *R1, *L2, *R2;
    int ldc, ldl1, ldr1, ldl2, ldr2;
    int M, N, r1, r2;
};

// C (M x N) -= L1 R1^T + L2 R2^T, in place: 64 x 64 tile per workgroup, the
// transposed tile accumulated on the matrix cores so that each lane group
// reads and writes 16 consecutive rows of a column; L and R staged in LDS 32
// columns at a time.  Bound by reading and writing C (n = 8000: 235 GB, 49 ms at the
// rate of a large copy).  With a branch around each staged element it took 55 ms there;
// without, and one slice ahead, the whole reduction went from 490 to 481 ms.
extern "C" __global__ void __launch_bounds__(HRD_THREADS) k_hrd_rank(RkArgs p) {
    __shared__ double Ls[64 * HRD_PAD];
    __shared__ double Rs[64 * HRD_PAD];
    const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int i0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
    // lane holds D(lk + 4 rr, li) = C^T(col, row): col = c0 + 16 q + lk + 4 rr, row = i0 + 16 it + li
    neig_d4 acc[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int row = i0 + 16 * it + li, col = c0 + 16 * q + lk + 4 * rr;
            acc[it][rr] = (row < p.M && col < p.N) ? AT(p.C, p.ldc, row, col) : 0.0;
        }
    }
    // A slice's 16 elements per thread are loaded without branches (columns past the
    // end count as zeros; rows past it are not stored), one slice ahead of the products.
    const int rt = p.r1 + p.r2;
    const int lrow = min(i0 + lane, p.M - 1), rrow = min(c0 + lane, p.N - 1);
    double lv[8], rv[8];
    auto fetch = [&](int kc) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = kc + q + 4 * e, kl = min(k, rt - 1);
            const bool second = kl >= p.r1;
            const double *l = second ? p.L2 + (size_t)(kl - p.r1) * p.ldl2 : p.L1 + (size_t)kl * p.ldl1;
            const double *r = second ? p.R2 + (size_t)(kl - p.r1) * p.ldr2 : p.R1 + (size_t)kl * p.ldr1;
            lv[e] = l[lrow];
            rv[e] = r[rrow];
            if (k >= rt) lv[e] = rv[e] = 0.0;
        }
    };
    fetch(0);
    for (int kc = 0; kc < rt; kc += 32) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            Ls[lane * HRD_PAD + q + 4 * e] = lv[e];
            Rs[lane * HRD_PAD + q + 4 * e] = -rv[e];
        }
        __syncthreads();
        if (kc + 32 < rt) fetch(kc + 32);
#pragma unroll
        for (int k4 = 0; k4 < 32; k4 += 4) {
            const double a = Rs[(16 * q + li) * HRD_PAD + k4 + lk];
#pragma unroll
            for (int it = 0; it < 4; ++it)
                acc[it] = hrd_mfma(a, Ls[(16 * it + li) * HRD_PAD + k4 + lk], acc[it]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int row = i0 + 16 * it + li, col = c0 + 16 * q + lk + 4 * rr;
            if (row < p.M && col < p.N) AT(p.C, p.ldc, row, col) = acc[it][rr];
        }
    }
}
