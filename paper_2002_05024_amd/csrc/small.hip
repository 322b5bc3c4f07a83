// small.hip -- one-workgroup kernels that keep a whole small matrix in LDS.
//
//  * k_small_qr: the double-shift QR iteration (the two-shift case of the bulge
//    chase in Section 3.2) on an m x m diagonal block, m <= NEIG_SMALL_MAX, with
//    its orthogonal factor accumulated in LDS.  Used for the final small active
//    blocks and for whole problems that fit.
//  * k_aed: aggressive early deflation (Section 3.2, "AED step") on a trailing
//    window that fits in LDS: window Schur form by the same QR, spike test of
//    every diagonal block from the bottom up, failing blocks moved to the top of
//    the window by swaps of adjacent diagonal blocks (the Bai-Demmel block swap
//    the paper cites), then a Householder Hessenberg reduction of the remaining
//    spike and undeflated part.
//
// Several waves per workgroup.  In the QR iteration wave 0 works on the window alone
// and waves 1 and 2 accumulate its reflectors into the orthogonal factor (see
// there); other phases use all waves with block barriers.
#include "neig_dev.h"
#include <climits>

#define NT 256     // threads per workgroup; the functions below take another count as NTH
// Waves 3 and up only help with what all waves share out: applying swaps and
// reflectors.  Measured on MI355X with 4 / 8 / 12 waves: 64-row deflation windows,
// spike test 755 / 672 / 629 and reduction back 284 / 238 / 263 thousand cycles, the
// random n = 20000 reduction 825 / 796 / 798 ms; reordering n = 4000 40.1 / 36.2 /
// 35.3 ms.  (The window QR alone, k_small_qr, has no use for them.)
#define AED_THREADS 512
#define REORDER_THREADS 768
#define LANES 64   // wavefront size
#define FB 15      // reflectors per batch handed to the accumulating waves

// Block-wide max / sum (all NTH threads call; result in every thread).
template <int NTH = NT>
__device__ __forceinline__ double block_reduce(double v, bool is_max) {
    __shared__ double red[NTH / LANES];
    v = is_max ? wave_max(v) : wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & (LANES - 1)) == 0) red[threadIdx.x / LANES] = v;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int w = 1; w < NTH / LANES; ++w) r = is_max ? fmax(r, red[w]) : r + red[w];
    return r;
}

// rows r, r+1 of M, columns c0..c1: (x, y) <- (cs x + sn y, -sn x + cs y)
template <int NTH = NT>
__device__ __forceinline__ void lds_rot_rows(double *M, int ld, int r, int c0, int c1, double cs, double sn) {
    for (int j = c0 + (int)threadIdx.x; j <= c1; j += NTH) {
        double x = AT(M, ld, r, j), y = AT(M, ld, r + 1, j);
        AT(M, ld, r, j) = cs * x + sn * y;
        AT(M, ld, r + 1, j) = -sn * x + cs * y;
    }
}

// columns c, c+1 of M, rows r0..r1
template <int NTH = NT>
__device__ __forceinline__ void lds_rot_cols(double *M, int ld, int c, int r0, int r1, double cs, double sn) {
    for (int i = r0 + (int)threadIdx.x; i <= r1; i += NTH) {
        double x = AT(M, ld, i, c), y = AT(M, ld, i, c + 1);
        AT(M, ld, i, c) = cs * x + sn * y;
        AT(M, ld, i, c + 1) = -sn * x + cs * y;
    }
}

// Standardise the 2x2 block at (j, j) of the m x m matrix T (rotation applied to
// whole rows and columns of T and to the columns of Q).
template <int NTH = NT>
__device__ __forceinline__ void lds_standardise(double *T, int ldt, double *Q, int ldq, int m, int j) {
    Std2 o = std2x2(AT(T, ldt, j, j), AT(T, ldt, j, j + 1), AT(T, ldt, j + 1, j), AT(T, ldt, j + 1, j + 1));
    __syncthreads();
    if (!(o.cs == 1.0 && o.sn == 0.0)) {
        lds_rot_rows<NTH>(T, ldt, j, j + 2, m - 1, o.cs, o.sn);
        lds_rot_cols<NTH>(T, ldt, j, 0, j - 1, o.cs, o.sn);
        lds_rot_cols<NTH>(Q, ldq, j, 0, m - 1, o.cs, o.sn);
    }
    if (threadIdx.x == 0) {
        AT(T, ldt, j, j) = o.a; AT(T, ldt, j, j + 1) = o.b;
        AT(T, ldt, j + 1, j) = o.c; AT(T, ldt, j + 1, j + 1) = o.d;
    }
    __syncthreads();
}

// ---------------------------------------------------------------- double-shift QR in LDS
//
// Wave 0 runs the whole iteration on T by itself, without a block barrier: the
// scan for negligible subdiagonals, the shifts, the bulge steps and the 2x2
// standardisations.  The steps of a sweep are one dependent chain, so what
// bounds them is the latency and the instruction count of one wave; T's entries
// therefore pass through registers, not through LDS, on that chain:
//
//  * the 3x3 block under the reflector (the core), the subdiagonal entry below
//    it and the generating vector are held by every lane, which all compute the
//    same values: nothing on the chain crosses lanes;
//  * lane c > k+2 holds rows k..k+2 of column c and lane r < k columns k..k+2 of
//    row r, so one instruction sequence applies the reflector from the left to
//    every column right of the core and from the right to every row above it.
//    After a step each lane stores its first entry (final for this sweep), shifts,
//    and loads the next one behind the next reflector's arithmetic; column k+3
//    enters the core through readlane, row k leaves it by a select.
//    T has at most 96 rows, so up to order 64 one vector per lane is enough and
//    two above (SETS).
//
// The orthogonal factor does not feed back into T: waves 1 and 2 apply the
// reflectors to Q's rows, in batches of FB that wave 0 publishes through a queue
// in LDS.  Measured on MI355X on random 64-row windows (36 steps a sweep): 23 550
// cycles a sweep, 45 900 when the entries passed through LDS and the other waves
// updated the far part of T; the n = 20000 random reduction 1.61 -> 1.11 s, an
// n = 40 block 1.03 -> 0.54 ms.
//
// Reflectors are kept as P = I + q u u^T, u = (x0 - beta, x1, x2),
// q = 1 / (beta (x0 - beta)): the products u^T y then run beside the reciprocal
// instead of after it.

#define QR_SLOTS 4

struct QrQueue {
    double c[QR_SLOTS][FB][4];         // q, u0, u1, u2 of each reflector; or cs, sn of a rotation
    int k0[QR_SLOTS], nb[QR_SLOTS];    // first position and count; 0: a rotation; -1: the end
    int head;                          // entries published by wave 0
    int tail[2];                       // entries applied by waves 1 and 2
    int info, iters;
    double dump[LANES];                // stores of lanes that have nothing to store
};

#define SWAP_PAIRS 32    // pairs of one round (more wait for the next one)
#define SWAP_ROWS 384    // largest window

// One round of block swaps (see there).
struct SwapState {
    double q[SWAP_PAIRS][16];        // the transforms, N x N at i + N j
    int total, cnt[4], rejected;
    int list[4][SWAP_PAIRS];         // per type: slots
    int st[SWAP_PAIRS], n[SWAP_PAIRS];  // per slot: first row (-1: rejected) and rows
    unsigned char head[SWAP_ROWS + 1];  // 1: a block starts at this row
    unsigned char mover[SWAP_ROWS];     // 1: a block that moves up starts at this row
};

// The scratch in LDS that the phases of a window kernel use in turn.
union WinScratch {
    QrQueue qr;
    SwapState sw;
};

__device__ __forceinline__ WinScratch &win_scratch() {
    __shared__ WinScratch s;
    return s;
}

struct ReflU {
    double beta, q, u0, u1, u2;
};

// The generating vector of a reflector, its squared length a, and the power of two
// that it was scaled by when a left the range (u and q then belong to the scaled
// vector; P is the same).  A zero vector becomes (1, 0, 0): a sign change, and so does
// (x0, 0, 0), as which the sweep of a block goes on when the product of its shifts has
// overflowed: thousands of exact ones leave Q orthogonal.
struct GenVec {
    double x0, x1, x2, a, sc;
};

// The range of a in which u stays as it is: (2^-664, 2^664), |u| in (2^-332, 2^333).
// The products with the matrix's entries x are then at most |u| |x| and |x| / |u|, so
// they stay finite while ||H||_F < 2^500 (similarity transforms keep the norm), and so
// does the product of two shifts; above (span 0), every vector is scaled, and u is of
// order 1 as v of I - tau v v^T is.
#define REFL_SPAN 0x53000000u
#define REFL_LOCAL 1u  // stands for the span of a window whose norm the host does not know
__host__ __device__ inline unsigned refl_span(double hnorm) { return hnorm < 0x1p500 ? REFL_SPAN : 0u; }

__device__ __forceinline__ GenVec gen_vec(double x0, double x1, double x2, unsigned span) {
    GenVec g{x0, x1, x2, fma(x0, x0, fma(x1, x1, x2 * x2)), 1.0};
    // by the exponent of a; the same in every lane
    if (__builtin_expect(__ballot((unsigned)__double2hiint(g.a) - 0x16700000u < span) == 0ull, 0)) {
        const double mx = fmax(fabs(x0), fmax(fabs(x1), fabs(x2)));
        if (x1 == 0.0 && x2 == 0.0 && mx < INFINITY) {
            g.sc = fabs(x0);
            g.x0 = copysign(1.0, x0);
        } else if (mx > 0.0 && mx < INFINITY) {
            const int e = ilogb(mx);
            g.x0 = ldexp(x0, -e); g.x1 = ldexp(x1, -e); g.x2 = ldexp(x2, -e);
            g.sc = ldexp(1.0, e);
        } else {
            g.sc = x0 + x1 + x2;  // 0, or not finite
            g.x0 = 1.0; g.x1 = 0.0; g.x2 = 0.0;
        }
        g.a = fma(g.x0, g.x0, fma(g.x1, g.x1, g.x2 * g.x2));
    }
    return g;
}

// The hardware's approximations of 1/sqrt and 1/x (about 2^-24), refined: the root by
// one coupled step (Goldschmidt) and a correction, the reciprocal, which starts from the
// unrefined root, beside it by two Newton steps.  The range scaling of the library's
// functions is left out (gen_vec sees to the range).  Over 2^20 vectors with entries
// spread over 2^+-40, in units of 2^-53: beta within 2.1 of the exact one (0.42 on
// average), 2 + q |u|^2, which is zero for an orthogonal P, within 6.0 (1.25).
__device__ __forceinline__ ReflU refl_u(const GenVec &x) {
    ReflU r;
    const double y = __builtin_amdgcn_rsq(x.a);
    double g = x.a * y, h = 0.5 * y;
    double z = __builtin_amdgcn_rcp(fma(fabs(x.x0), g, x.a));
    const double e0 = fma(-g, h, 0.5);
    g = fma(g, e0, g);
    h = fma(h, e0, h);
    g = fma(fma(-g, g, x.a), h, g);
    const double beta = -copysign(g, x.x0);
    r.u0 = x.x0 - beta;
    const double den = beta * r.u0;  // -(a + |x0| sqrt(a))
    z = -z;
    z = fma(z, fma(-den, z, 1.0), z);
    r.q = fma(z, fma(-den, z, 1.0), z);
    r.u1 = x.x1;
    r.u2 = x.x2;
    r.beta = beta * x.sc;
    return r;
}

// Orders this wave's LDS accesses across its lanes (the hardware keeps them in
// program order; this keeps the compiler to it).
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// A select of values (a conditional expression on struct members may become an
// indexed load from scratch).
__device__ __forceinline__ double pick(bool c, double a, double b) { return c ? a : b; }

__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Wave 0: the next queue slot, once the accumulating waves are done with it.
__device__ __forceinline__ int qr_slot(QrQueue &q, int entry, int nacc) {
    for (int w = 0; w < nacc; ++w)
        while (__hip_atomic_load(&q.tail[w], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) + QR_SLOTS <= entry)
            __builtin_amdgcn_s_sleep(1);
    return entry & (QR_SLOTS - 1);
}

__device__ __forceinline__ void qr_publish(QrQueue &q, int entry, int k0, int nb) {
    const int slot = entry & (QR_SLOTS - 1);
    if ((threadIdx.x & (LANES - 1)) == 0) {
        q.k0[slot] = k0;
        q.nb[slot] = nb;
        __hip_atomic_store(&q.head, entry + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Waves 1 and 2: apply the published entries to row `row` of Q (rows past m idle).
__device__ __forceinline__ void qr_accumulate(QrQueue &q, int who, double *Q, int ldq, int m, int row) {
    for (int entry = 0;; ++entry) {
        while (__hip_atomic_load(&q.head, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= entry)
            __builtin_amdgcn_s_sleep(1);
        const int slot = entry & (QR_SLOTS - 1);
        const int nb = __builtin_amdgcn_readfirstlane(q.nb[slot]);
        if (nb < 0) break;
        const int k0 = __builtin_amdgcn_readfirstlane(q.k0[slot]);
        if (row < m) {
            double *base = &AT(Q, ldq, row, k0);
            if (nb == 0) {
                const double cs = q.c[slot][0][0], sn = q.c[slot][0][1];
                const double x = base[0], y = base[ldq];
                base[0] = cs * x + sn * y;
                base[ldq] = -sn * x + cs * y;
            } else {
                // reflectors past nb are zero (wave 0 clears a short batch's rest)
                const int len = min(nb + 2, m - k0);
                double x[FB + 2];
#pragma unroll
                for (int t = 0; t < FB + 2; ++t) x[t] = (t < len) ? base[t * ldq] : 0.0;
#pragma unroll
                for (int t = 0; t < FB; ++t) {
                    const double *c = q.c[slot][t];
                    const double s = c[0] * fma(c[1], x[t], fma(c[2], x[t + 1], c[3] * x[t + 2]));
                    x[t] = fma(s, c[1], x[t]);
                    x[t + 1] = fma(s, c[2], x[t + 1]);
                    x[t + 2] = fma(s, c[3], x[t + 2]);
                }
#pragma unroll
                for (int t = 0; t < FB + 2; ++t)
                    if (t < len) base[t * ldq] = x[t];
            }
        }
        if ((threadIdx.x & (LANES - 1)) == 0)
            __hip_atomic_store(&q.tail[who], entry + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// One implicit double-shift sweep (wave 0) on the active rows l..i (i - l >= 2) of
// the m x m LDS matrix T, over all of T's rows and columns; entry counts the
// queue's entries.  ldt > m: row m of T is never read as data, and takes the
// stores of lanes that hold nothing.
template <int SETS>
__device__ __forceinline__ void qr_sweep(double *T, int ldt, int m, int l, int i, double tr, double det, unsigned span,
                                         QrQueue &q, int nacc, int &entry) {
    const int lane = threadIdx.x & (LANES - 1);
    double C[3][3], x0, x1, x2;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) C[a][b] = AT(T, ldt, l + a, l + b);
    // per lane: its 3-vector, the address of the first entry and the stride.
    // Lanes k+1 and k+2 (rows and columns of the core) go on storing as columns:
    // what they write, T(k, k+1) and T(k, k+2), is stored again by lane k as a row.
    double v[SETS][3];
    int at[SETS], st[SETS];
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const int idx = lane + LANES * s;
        at[s] = idx < l ? idx + l * ldt : (idx < m ? idx * ldt + l : m + min(idx - m, m - 1) * ldt);
        st[s] = idx < l ? ldt : (idx < m ? 1 : 0);
#pragma unroll
        for (int a = 0; a < 3; ++a) v[s][a] = T[at[s] + a * st[s]];
    }
    double h = AT(T, ldt, l + 3, l + 2);  // used only when l + 3 <= i
    {  // the bulge from the shift polynomial
        double sc = fmax(fmax(fabs(C[0][0]), fabs(C[0][1])), fmax(fmax(fabs(C[1][0]), fabs(C[1][1])), fabs(C[2][1])));
        sc = fmax(sc, fmax(fabs(tr), sqrt(fabs(det))));
        if (sc == 0.0) sc = 1.0;
        const double rs = 1.0 / sc;
        const double a = C[0][0] * rs, b = C[0][1] * rs, c = C[1][0] * rs, d = C[1][1] * rs, e = C[2][1] * rs;
        const double t = tr * rs, dt = det * rs * rs;
        x0 = a * a + b * c - t * a + dt;
        x1 = c * (a + d - t);
        x2 = c * e;
    }
    int k0 = l;
    int slot = qr_slot(q, entry, nacc);
    // lanes 0..3 store a reflector's q, u0, u1, u2 into the queue, lane 4 its beta
    double *qc = lane < 4 ? &q.c[slot][0][lane] : (lane == 4 ? T + (l + 1) + l * ldt : &q.dump[lane]);
    const int qinc = lane < 4 ? 4 : (lane == 4 ? ldt + 1 : 0);
    auto publish = [&](int nb) {
        if (lane >= nb && lane < FB)
            for (int a = 0; a < 4; ++a) q.c[slot][lane][a] = 0.0;
        qr_publish(q, entry, k0, nb);
        ++entry;
        k0 += nb;
        slot = qr_slot(q, entry, nacc);
        if (lane < 4) qc = &q.c[slot][0][lane];
    };
    auto record = [&](const ReflU &r, bool first) __attribute__((always_inline)) {
        const double w = pick(lane == 0, r.q, pick(lane == 1, r.u0, pick(lane == 2, r.u1,
                                                                    pick(lane == 3, r.u2, r.beta))));
        if (first) {  // no column left of the active block
            *(lane == 4 ? &q.dump[lane] : qc) = w;
            qc += lane < 4 ? 4 : 0;
        } else {
            *qc = w;
            qc += qinc;
        }
    };
    // The lanes' part of step k (reflector r, J the row k of the core): behind the
    // chain of the next step, in the same block of instructions.  more: column
    // k + 3 enters the core next.
    auto lanes_step = [&](const ReflU &r, const double (&J)[3], int k, bool more) __attribute__((always_inline)) {
        // row k joins the lanes
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const bool mine = lane + LANES * s == k;
#pragma unroll
            for (int b = 0; b < 3; ++b) v[s][b] = mine ? J[b] : v[s][b];
            at[s] = mine ? k + k * ldt : at[s];
            st[s] = mine ? ldt : st[s];
        }
        // left on the columns, right on the rows
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const double t = r.q * fma(r.u0, v[s][0], fma(r.u1, v[s][1], r.u2 * v[s][2]));
            T[at[s]] = fma(t, r.u0, v[s][0]);
            v[s][0] = fma(t, r.u1, v[s][1]);
            v[s][1] = fma(t, r.u2, v[s][2]);
        }
        wave_fence();
        if (more) {
            const int c = k + 3;
            double p1 = lane_value(v[0][0], c & (LANES - 1)), p2 = lane_value(v[0][1], c & (LANES - 1));
            if (SETS == 2) {
                const double p3 = lane_value(v[SETS - 1][0], c & (LANES - 1));
                const double p4 = lane_value(v[SETS - 1][1], c & (LANES - 1));
                p1 = c >= LANES ? p3 : p1;
                p2 = c >= LANES ? p4 : p2;
            }
            C[0][2] = p1;
            C[1][2] = p2;
#pragma unroll
            for (int s = 0; s < SETS; ++s) v[s][2] = T[at[s] + 3 * st[s]];
        }
#pragma unroll
        for (int s = 0; s < SETS; ++s) at[s] += st[s];
    };
    // The core's part of step k; more: row and column k + 3 belong to the active block.
    ReflU r;
    double J[3];
    auto core_step = [&](const GenVec &x, int k, bool first, bool more) __attribute__((always_inline)) {
        r = refl_u(x);
#pragma unroll
        for (int b = 0; b < 3; ++b) {  // left
            const double t = r.q * fma(r.u0, C[0][b], fma(r.u1, C[1][b], r.u2 * C[2][b]));
            J[b] = fma(t, r.u0, C[0][b]);
            C[1][b] = fma(t, r.u1, C[1][b]);
            C[2][b] = fma(t, r.u2, C[2][b]);
        }
#pragma unroll
        for (int a = 1; a < 3; ++a) {  // right, on rows k+1, k+2: they move up
            const double t = r.q * fma(r.u0, C[a][0], fma(r.u1, C[a][1], r.u2 * C[a][2]));
            (a == 1 ? x0 : x1) = fma(t, r.u0, C[a][0]);
            C[a - 1][0] = fma(t, r.u1, C[a][1]);
            C[a - 1][1] = fma(t, r.u2, C[a][2]);
        }
        if (more) {  // right, on row k+3
            const double t = r.q * (r.u2 * h);
            x2 = t * r.u0;
            C[2][0] = t * r.u1;
            C[2][1] = fma(t, r.u2, h);
            const int c = k + 3;
            C[2][2] = AT(T, ldt, c, c);
            h = AT(T, ldt, c + 1, c);  // row m, unused, when c = m - 1
        }
        record(r, first);
    };
    int k = l;
    core_step(gen_vec(x0, x1, x2, span), k, true, k < i - 2);
    ++k;
    // One step: the range check of its reflector, then the lanes' part of the step
    // before it between the dependent operations of this one's reflector.  The
    // scheduling barriers keep that order (left alone, the compiler issues the
    // reflector's chain in one piece, with a wait at every operation).
    auto step = [&](bool more) __attribute__((always_inline)) {
        const GenVec x = gen_vec(x0, x1, x2, span);
        const double q = r.q, u0 = r.u0, u1 = r.u1, u2 = r.u2;  // step k - 1
        double vv[SETS][3], t[SETS];
        const double y = __builtin_amdgcn_rsq(x.a);
#pragma unroll
        for (int s = 0; s < SETS; ++s) {  // row k - 1 joins the lanes
            const bool mine = lane + LANES * s == k - 1;
#pragma unroll
            for (int b = 0; b < 3; ++b) vv[s][b] = pick(mine, J[b], v[s][b]);
            at[s] = mine ? (k - 1) + (k - 1) * ldt : at[s];
            st[s] = mine ? ldt : st[s];
        }
        __builtin_amdgcn_sched_barrier(0);
        double g = x.a * y, h2 = 0.5 * y;
#pragma unroll
        for (int s = 0; s < SETS; ++s) t[s] = u2 * vv[s][2];
        __builtin_amdgcn_sched_barrier(0);
        double z = -__builtin_amdgcn_rcp(fma(fabs(x.x0), g, x.a));
        const double e0 = fma(-g, h2, 0.5);
#pragma unroll
        for (int s = 0; s < SETS; ++s) t[s] = fma(u1, vv[s][1], t[s]);
        __builtin_amdgcn_sched_barrier(0);
        g = fma(g, e0, g);
        h2 = fma(h2, e0, h2);
#pragma unroll
        for (int s = 0; s < SETS; ++s) t[s] = fma(u0, vv[s][0], t[s]);
        __builtin_amdgcn_sched_barrier(0);
        const double d = fma(-g, g, x.a);
#pragma unroll
        for (int s = 0; s < SETS; ++s) t[s] *= q;
        __builtin_amdgcn_sched_barrier(0);
        g = fma(d, h2, g);
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            T[at[s]] = fma(t[s], u0, vv[s][0]);
            v[s][0] = fma(t[s], u1, vv[s][1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        const double beta = -copysign(g, x.x0);
        const double w0 = x.x0 - beta, w1 = x.x1, w2 = x.x2;
#pragma unroll
        for (int s = 0; s < SETS; ++s) v[s][1] = fma(t[s], u2, vv[s][2]);
        __builtin_amdgcn_sched_barrier(0);
        const double den = beta * w0;
        {  // column k + 2 enters the core
            const int c = (k + 2) & (LANES - 1);
            double p1 = lane_value(v[0][0], c), p2 = lane_value(v[0][1], c);
            if (SETS == 2) {
                const double p3 = lane_value(v[SETS - 1][0], c), p4 = lane_value(v[SETS - 1][1], c);
                p1 = k + 2 >= LANES ? p3 : p1;
                p2 = k + 2 >= LANES ? p4 : p2;
            }
            C[0][2] = p1;
            C[1][2] = p2;
        }
        __builtin_amdgcn_sched_barrier(0);
        const double e1 = fma(-den, z, 1.0);
        double dot[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) dot[b] = w2 * C[2][b];
        __builtin_amdgcn_sched_barrier(0);
        z = fma(z, e1, z);
#pragma unroll
        for (int b = 0; b < 3; ++b) dot[b] = fma(w1, C[1][b], dot[b]);
        __builtin_amdgcn_sched_barrier(0);
        const double e2 = fma(-den, z, 1.0);
#pragma unroll
        for (int b = 0; b < 3; ++b) dot[b] = fma(w0, C[0][b], dot[b]);
        const double w2h = w2 * h;
        __builtin_amdgcn_sched_barrier(0);
        const double p = fma(z, e2, z);
        wave_fence();
        if (SETS == 1) v[0][2] = T[at[0] + 3 * st[0]];
        else
#pragma unroll
            for (int s = 0; s < SETS; ++s) v[s][2] = T[at[s] + 3 * st[s]];
#pragma unroll
        for (int s = 0; s < SETS; ++s) at[s] += st[s];
        double C22 = 0.0, hn = 0.0;
        if (more) {
            C22 = AT(T, ldt, k + 3, k + 3);
            hn = AT(T, ldt, k + 4, k + 3);  // row m, unused, when k + 3 = m - 1
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < 3; ++b) dot[b] *= p;
        const double th = p * w2h;
        double R1[3], R2[3];
#pragma unroll
        for (int b = 2; b >= 0; --b) {  // left, on the core
            R1[b] = fma(dot[b], w1, C[1][b]);
            R2[b] = fma(dot[b], w2, C[2][b]);
        }
        // right, on its rows 1 and 2
        double s1 = w2 * R1[2], s2 = w2 * R2[2];
        s1 = fma(w1, R1[1], s1);
        s2 = fma(w1, R2[1], s2);
        s1 = p * fma(w0, R1[0], s1);
        s2 = p * fma(w0, R2[0], s2);
        x0 = fma(s1, w0, R1[0]);
        x1 = fma(s2, w0, R2[0]);
        if (more) x2 = th * w0;
#pragma unroll
        for (int b = 0; b < 3; ++b) J[b] = fma(dot[b], w0, C[0][b]);
        C[0][0] = fma(s1, w1, R1[1]);
        C[0][1] = fma(s1, w2, R1[2]);
        C[1][0] = fma(s2, w1, R2[1]);
        C[1][1] = fma(s2, w2, R2[2]);
        if (more) {  // row k + 3
            C[2][0] = th * w1;
            C[2][1] = fma(th, w2, h);
            C[2][2] = C22;
            h = hn;
        }
        r.q = p; r.u0 = w0; r.u1 = w1; r.u2 = w2; r.beta = beta * x.sc;
        record(r, false);
        ++k;
    };
    while (k < i - 2) {
        const int ke = min(i - 2, k0 + FB);
        // by three, so that the shifts cost no moves; the loop starts on a multiple of 8
        // bytes (64-row windows: 23 550 cycles a sweep, 1% more where the code before it
        // ended half way, as most of its instructions then straddle two such units)
        asm volatile(".p2align 6");
        while (k + 3 <= ke) {
            step(true);
            step(true);
            step(true);
        }
        while (k < ke) step(true);
        if (k - k0 == FB) publish(FB);
    }
    if (k == i - 2) step(false);
    if (k - k0 == FB) publish(FB);
    lanes_step(r, J, k - 1, false);
    // the last, two-row reflector at k = i - 1, on core rows 0, 1 and columns 0, 1
    {
        const ReflU e = refl_u(gen_vec(x0, x1, 0.0, span));
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const double t = e.q * fma(e.u0, C[0][b], e.u1 * C[1][b]);
            C[0][b] = fma(t, e.u0, C[0][b]);
            C[1][b] = fma(t, e.u1, C[1][b]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const double t = e.q * fma(e.u0, C[a][0], e.u1 * C[a][1]);
            C[a][0] = fma(t, e.u0, C[a][0]);
            C[a][1] = fma(t, e.u1, C[a][1]);
        }
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const int idx = lane + LANES * s;
            const double t = e.q * fma(e.u0, v[s][0], e.u1 * v[s][1]);
            if ((unsigned)(idx - k) > 1u && idx < m) {
                T[at[s]] = fma(t, e.u0, v[s][0]);
                T[at[s] + st[s]] = fma(t, e.u1, v[s][1]);
            }
        }
        record(e, false);
        if (lane == 0) {
            AT(T, ldt, k, k) = C[0][0]; AT(T, ldt, k, k + 1) = C[0][1];
            AT(T, ldt, k + 1, k) = C[1][0]; AT(T, ldt, k + 1, k + 1) = C[1][1];
        }
    }
    publish(k - k0 + 1);
    wave_fence();
}

// Wave 0: standard form of the 2x2 block at (j, j) of T.
__device__ __forceinline__ void qr_standardise(double *T, int ldt, int m, int j, QrQueue &q, int nacc, int &entry) {
    const int lane = threadIdx.x & (LANES - 1);
    const Std2 o = std2x2(AT(T, ldt, j, j), AT(T, ldt, j, j + 1), AT(T, ldt, j + 1, j), AT(T, ldt, j + 1, j + 1));
    if (!(o.cs == 1.0 && o.sn == 0.0)) {
        for (int idx = lane; idx < m; idx += LANES) {
            if (idx == j || idx == j + 1) continue;
            double *p = (idx < j) ? &AT(T, ldt, idx, j) : &AT(T, ldt, j, idx);
            const int s = (idx < j) ? ldt : 1;
            const double x = p[0], y = p[s];
            p[0] = o.cs * x + o.sn * y;
            p[s] = -o.sn * x + o.cs * y;
        }
        const int slot = qr_slot(q, entry, nacc);
        if (lane == 0) {
            q.c[slot][0][0] = o.cs;
            q.c[slot][0][1] = o.sn;
        }
        qr_publish(q, entry, j, 0);
        ++entry;
    }
    if (lane == 0) {
        AT(T, ldt, j, j) = o.a; AT(T, ldt, j, j + 1) = o.b;
        AT(T, ldt, j + 1, j) = o.c; AT(T, ldt, j + 1, j + 1) = o.d;
    }
    wave_fence();
}

// Wave 0: the whole iteration.  Returns 0, or i+1 when rows/cols 0..i did not
// converge within maxit iterations.
template <int SETS>
__device__ __forceinline__ int qr_iterate(double *T, int ldt, int m, double hnorm, double smlnum, int maxit, QrQueue &q,
                                          int nacc, int &entry, int *iters) {
    const int lane = threadIdx.x & (LANES - 1);
    const unsigned span = __builtin_amdgcn_readfirstlane(refl_span(hnorm));
    int i = m - 1, its = 0, total = 0, info = 0;
    while (i >= 0) {
        int l = 0;
        for (int base = i; base >= 1; base -= LANES) {
            const int k = base - lane;
            bool neg = false;
            if (k >= 1)
                neg = negligible_sub(AT(T, ldt, k, k - 1), AT(T, ldt, k - 1, k - 1), AT(T, ldt, k, k), hnorm, smlnum);
            const unsigned long long mask = __ballot(neg);
            if (mask) {
                l = base - (__ffsll(mask) - 1);
                break;
            }
        }
        wave_fence();
        if (l > 0 && lane == 0) AT(T, ldt, l, l - 1) = 0.0;
        wave_fence();
        if (l == i) {
            --i;
            its = 0;
            continue;
        }
        if (l == i - 1) {
            qr_standardise(T, ldt, m, i - 1, q, nacc, entry);
            i -= 2;
            its = 0;
            continue;
        }
        if (total >= maxit) {
            info = i + 1;
            break;
        }
        ++total;
        ++its;
        double tr, det;
        if (its == 10 || its == 20) {
            const double s = fabs(AT(T, ldt, i, i - 1)) + fabs(AT(T, ldt, i - 1, i - 2));
            const double x = AT(T, ldt, i, i);
            tr = 2.0 * x + 1.5 * s;
            det = x * x + 1.5 * s * x + s * s;
        } else {
            const double a = AT(T, ldt, i - 1, i - 1), b = AT(T, ldt, i - 1, i);
            const double c = AT(T, ldt, i, i - 1), d = AT(T, ldt, i, i);
            tr = a + d;
            det = a * d - b * c;
        }
        qr_sweep<SETS>(T, ldt, m, l, i, tr, det, span, q, nacc, entry);
    }
    *iters = total;
    return info;
}

// Double-shift QR iteration on the m x m LDS matrix T (upper Hessenberg, m <= 96)
// with Q accumulated; all threads (three waves or more) call, after a barrier.  Returns
// 0, or i+1 when rows/cols 0..i did not converge within maxit iterations.  *iters
// receives the iteration count.
__device__ __forceinline__ int lds_small_qr(double *T, int ldt, double *Q, int ldq, int m, double hnorm, double smlnum,
                                            int maxit, int *iters) {
    static_assert(NEIG_SMALL_MAX <= 2 * LANES, "two vectors per lane");
    QrQueue &q = win_scratch().qr;
    const int lane = threadIdx.x & (LANES - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
    if (threadIdx.x == 0) {
        q.head = 0;
        q.tail[0] = q.tail[1] = 0;
    }
    __syncthreads();
    const int nacc = (m + LANES - 1) / LANES;  // accumulating waves
    if (wave == 0) {
        int entry = 0, its = 0;
        const int info = (m <= LANES) ? qr_iterate<1>(T, ldt, m, hnorm, smlnum, maxit, q, nacc, entry, &its)
                                      : qr_iterate<2>(T, ldt, m, hnorm, smlnum, maxit, q, nacc, entry, &its);
        qr_slot(q, entry, nacc);
        qr_publish(q, entry, 0, -1);
        if (lane == 0) {
            q.info = info;
            q.iters = its;
        }
    } else if (wave <= nacc) {
        qr_accumulate(q, wave - 1, Q, ldq, m, lane + LANES * (wave - 1));
    }
    __syncthreads();
    *iters = q.iters;
    const int info = q.info;
    __syncthreads();
    return info;
}

// Load the m x m diagonal block of H at (off, off) into T (zeros below the
// subdiagonal) and set Q = I.
template <int NTH = NT>
__device__ __forceinline__ void lds_load_block(const double *H, int ldh, int off, int m, double *T, int ldt, double *Q, int ldq) {
    for (int idx = threadIdx.x; idx < m * m; idx += NTH) {
        const int i = idx % m, j = idx / m;
        AT(T, ldt, i, j) = (i <= j + 1) ? AT(H, ldh, off + i, off + j) : 0.0;
        AT(Q, ldq, i, j) = (i == j) ? 1.0 : 0.0;
    }
    __syncthreads();
}

// Write T back to H's diagonal block and Q^T to Ut (column-major, ld ldut).
template <int NTH = NT>
__device__ __forceinline__ void lds_store(double *H, int ldh, int off, int m, const double *T, int ldt, const double *Q, int ldq,
                          double *Ut, int ldut) {
    for (int idx = threadIdx.x; idx < m * m; idx += NTH) {
        const int i = idx % m, j = idx / m;
        AT(H, ldh, off + i, off + j) = (i <= j + 1) ? AT(T, ldt, i, j) : 0.0;
        AT(Ut, ldut, i, j) = AT(Q, ldq, j, i);
    }
}

extern "C" __global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_small_qr(double *H, int ldh, int off, int m, double hnorm, double smlnum, int maxit, double *Ut, int ldut,
           int *status) {
    extern __shared__ double lds[];
    const int ld = m + 1;
    double *T = lds;
    double *Q = lds + (size_t)m * ld;
    lds_load_block(H, ldh, off, m, T, ld, Q, ld);
    int iters = 0;
    const int info = lds_small_qr(T, ld, Q, ld, m, hnorm, smlnum, maxit, &iters);
    __syncthreads();
    lds_store(H, ldh, off, m, T, ld, Q, ld, Ut, ldut);
    if (threadIdx.x == 0) {
        status[0] = info;
        status[1] = iters;
    }
}

// ---------------------------------------------------------------- block swap
//
// Swapping adjacent diagonal blocks A (p x p, on top) and C (q x q) of a
// quasi-triangular matrix [[A B][0 C]]: solve A X - X C = B; the columns of
// [[-X][I]] span C's invariant subspace, so the orthogonal factor Q of their QR
// factorisation gives Q^T [[A B][0 C]] Q = [[C' *][0 A']].  The swap is
// rejected when the computed lower-left block or the reconstruction error is
// not at roundoff level.  Sizes are template parameters so that every array
// below has constant indices and lives in registers.

// Solve the K x K system M x = r by Gaussian elimination with complete
// pivoting; row and column exchanges are done with selects.  Tiny pivots are
// raised to smin.
template <int K>
__device__ __forceinline__ bool solve_cp(double (&M)[K][K], double (&r)[K], double (&x)[K]) {
    int perm[K];
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        perm[i] = i;
#pragma unroll
        for (int j = 0; j < K; ++j) mx = fmax(mx, fabs(M[i][j]));
    }
    const double smin = fmax(NEIG_EPS * mx, NEIG_DBL_MIN);
    double rinv[K];
#pragma unroll
    for (int s = 0; s < K; ++s) {
        int pr = s, pc = s;
        double best = -1.0;
#pragma unroll
        for (int i = s; i < K; ++i)
#pragma unroll
            for (int j = s; j < K; ++j) {
                const double v = fabs(M[i][j]);
                if (v > best) { best = v; pr = i; pc = j; }
            }
#pragma unroll
        for (int i = s + 1; i < K; ++i) {
            const bool sw = (i == pr);
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const double a = M[s][j], b = M[i][j];
                M[s][j] = sw ? b : a;
                M[i][j] = sw ? a : b;
            }
            const double a = r[s], b = r[i];
            r[s] = sw ? b : a;
            r[i] = sw ? a : b;
        }
#pragma unroll
        for (int j = s + 1; j < K; ++j) {
            const bool sw = (j == pc);
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const double a = M[i][s], b = M[i][j];
                M[i][s] = sw ? b : a;
                M[i][j] = sw ? a : b;
            }
            const int pa = perm[s], pb = perm[j];
            perm[s] = sw ? pb : pa;
            perm[j] = sw ? pa : pb;
        }
        if (fabs(M[s][s]) < smin) M[s][s] = smin;
        const double inv = 1.0 / M[s][s];
        rinv[s] = inv;
#pragma unroll
        for (int i = s + 1; i < K; ++i) {
            const double f = M[i][s] * inv;
#pragma unroll
            for (int j = s; j < K; ++j) M[i][j] -= f * M[s][j];
            r[i] -= f * r[s];
        }
    }
    double y[K];
#pragma unroll
    for (int s = K - 1; s >= 0; --s) {
        double t = r[s];
#pragma unroll
        for (int j = s + 1; j < K; ++j) t -= M[s][j] * y[j];
        y[s] = t * rinv[s];
    }
    bool ok = true;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        double v = 0.0;
#pragma unroll
        for (int s = 0; s < K; ++s) v = (perm[s] == i) ? y[s] : v;
        x[i] = v;
        ok = ok && isfinite(v);
    }
    return ok;
}

// The swap transform from a solution X of the Sylvester equation A X - X C = B12
// (A the leading P x P block of B, C the trailing Q x Q block, X(i, j) at index
// i + P j): the columns of [[-X][I]] span C's invariant subspace, Qm is the
// orthogonal factor of their QR factorisation and Bn = Qm^T B Qm.  Returns false
// when Bn's lower-left block or the reconstruction error B - Qm Bn Qm^T is not at
// roundoff level (then the swap is rejected).
template <int P, int Q>
__device__ __forceinline__ bool swap_from_x(const double (&B)[P + Q][P + Q], const double (&X)[P * Q], double bnorm,
                                            double (&Qm)[P + Q][P + Q], double (&Bn)[P + Q][P + Q]) {
    constexpr int N = P + Q;
    constexpr int K = P * Q;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) Qm[i][j] = (i == j) ? 1.0 : 0.0;
    double xm = 0.0;
#pragma unroll
    for (int t = 0; t < K; ++t) xm = fmax(xm, fabs(X[t]));
    const double g = 1.0 / fmax(1.0, xm);
    double Y[N][Q];
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int i = 0; i < N; ++i) Y[i][j] = (i < P) ? -g * X[i + P * j] : ((i - P == j) ? g : 0.0);
    // Householder QR of Y, reflectors accumulated into Qm
#pragma unroll
    for (int c = 0; c < Q; ++c) {
        double v[N];
#pragma unroll
        for (int t = 0; t < N; ++t) v[t] = (t >= c) ? Y[t][c] : 0.0;
        double mx = 0.0;
#pragma unroll
        for (int t = c + 1; t < N; ++t) mx = fmax(mx, fabs(v[t]));
        if (mx == 0.0) continue;
        const double sc = fmax(mx, fabs(v[c]));
        const double rsc = 1.0 / sc;
        double ss = 0.0;
#pragma unroll
        for (int t = c; t < N; ++t) ss += (v[t] * rsc) * (v[t] * rsc);
        const double nrm = sc * sqrt(ss);
        const double alpha = v[c];
        const double beta = alpha >= 0.0 ? -nrm : nrm;
        const double dd = alpha - beta;
        const double qq = 1.0 / (beta * dd);  // one division for 1/beta and 1/(alpha - beta)
        const double tau = -dd * dd * qq;     // (beta - alpha) / beta
        const double inv = beta * qq;         // 1 / (alpha - beta)
#pragma unroll
        for (int t = c + 1; t < N; ++t) v[t] *= inv;
        v[c] = 1.0;
#pragma unroll
        for (int j = c; j < Q; ++j) {
            double d = 0.0;
#pragma unroll
            for (int t = c; t < N; ++t) d += v[t] * Y[t][j];
            d *= tau;
#pragma unroll
            for (int t = c; t < N; ++t) Y[t][j] -= d * v[t];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double d = 0.0;
#pragma unroll
            for (int t = c; t < N; ++t) d += Qm[i][t] * v[t];
            d *= tau;
#pragma unroll
            for (int t = c; t < N; ++t) Qm[i][t] -= d * v[t];
        }
    }
    // Bn = Qm^T (B Qm); B is block upper triangular (rows P.. are zero in
    // columns ..P-1)
    double W[N][N];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double d = 0.0;
#pragma unroll
            for (int k = (i < P ? 0 : P); k < N; ++k) d += B[i][k] * Qm[k][j];
            W[i][j] = d;
        }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double d = 0.0;
#pragma unroll
            for (int k = 0; k < N; ++k) d += Qm[k][i] * W[k][j];
            Bn[i][j] = d;
        }
    const double thresh = fmax(20.0 * NEIG_EPS * bnorm, NEIG_DBL_MIN);
    double low = 0.0;
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int i = Q; i < N; ++i) {
            low = fmax(low, fabs(Bn[i][j]));
            Bn[i][j] = 0.0;
        }
    if (!(low <= thresh)) return false;
    // reconstruction: B ~ Qm Bn Qm^T (Bn now block upper triangular: rows Q..
    // are zero in columns ..Q-1)
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double d = 0.0;
#pragma unroll
            for (int k = (i < Q ? 0 : Q); k < N; ++k) d += Bn[i][k] * Qm[j][k];
            W[i][j] = d;
        }
    double err = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double d = 0.0;
#pragma unroll
            for (int k = 0; k < N; ++k) d += Qm[i][k] * W[k][j];
            err = fmax(err, fabs(d - B[i][j]));
        }
    return err <= thresh;
}

// Closed-form solve of the 2 x 2 Sylvester equation A X - X C = R.  With
// p(z) = z^2 - tr(C) z + det(C) the characteristic polynomial of C,
// Cayley-Hamilton (C^2 = tr(C) C - det(C) I) turns the equation into
// p(A) X = A R + R (C - tr(C) I), a 2 x 2 linear system solved by its adjugate;
// one step of residual correction follows.  Returns false when p(A) is singular
// or the result is not finite (the caller then solves the 4 x 4 system).
__device__ __forceinline__ bool sylv22_closed(const double (&B)[4][4], double (&X)[4]) {
    const double a00 = B[0][0], a01 = B[0][1], a10 = B[1][0], a11 = B[1][1];
    const double c00 = B[2][2], c01 = B[2][3], c10 = B[3][2], c11 = B[3][3];
    const double trc = c00 + c11, detc = c00 * c11 - c01 * c10;
    const double d = a00 + a11 - trc;
    const double p00 = a00 * a00 + a01 * a10 - trc * a00 + detc;
    const double p01 = a01 * d, p10 = a10 * d;
    const double p11 = a10 * a01 + a11 * a11 - trc * a11 + detc;
    const double detp = p00 * p11 - p01 * p10;
    if (!(fabs(detp) > 0.0)) return false;
    const double rd = 1.0 / detp;
    const double q00 = p11 * rd, q01 = -p01 * rd, q10 = -p10 * rd, q11 = p00 * rd;  // p(A)^-1
    // C - tr(C) I = [[-c11, c01], [c10, -c00]]
    double r00 = B[0][2], r01 = B[0][3], r10 = B[1][2], r11 = B[1][3];
    double x00 = 0.0, x01 = 0.0, x10 = 0.0, x11 = 0.0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const double s00 = a00 * r00 + a01 * r10 - r00 * c11 + r01 * c10;
        const double s01 = a00 * r01 + a01 * r11 + r00 * c01 - r01 * c00;
        const double s10 = a10 * r00 + a11 * r10 - r10 * c11 + r11 * c10;
        const double s11 = a10 * r01 + a11 * r11 + r10 * c01 - r11 * c00;
        x00 += q00 * s00 + q01 * s10;
        x01 += q00 * s01 + q01 * s11;
        x10 += q10 * s00 + q11 * s10;
        x11 += q10 * s01 + q11 * s11;
        if (pass == 0) {  // residual R - (A X - X C)
            r00 = B[0][2] - (a00 * x00 + a01 * x10 - x00 * c00 - x01 * c10);
            r01 = B[0][3] - (a00 * x01 + a01 * x11 - x00 * c01 - x01 * c11);
            r10 = B[1][2] - (a10 * x00 + a11 * x10 - x10 * c00 - x11 * c10);
            r11 = B[1][3] - (a10 * x01 + a11 * x11 - x10 * c01 - x11 * c11);
        }
    }
    X[0] = x00; X[1] = x10; X[2] = x01; X[3] = x11;
    return isfinite(x00) && isfinite(x01) && isfinite(x10) && isfinite(x11);
}

// Closed-form solve of the Sylvester equation when one block is 1x1: for
// (P, Q) = (1, 2) it reads X (a I - C) = R (X a row), for (2, 1) it reads
// (A - c I) X = R (X a column); either is one 2 x 2 system, solved by its
// adjugate, with one step of residual correction.  Returns false when the
// system is singular or the result is not finite (the caller then solves by
// complete pivoting).
template <int P, int Q>
__device__ __forceinline__ bool sylv12_closed(const double (&B)[P + Q][P + Q], double (&X)[2]) {
    static_assert(P * Q == 2, "one 1x1 and one 2x2 block");
    double m00, m01, m10, m11, r0, r1;
    if constexpr (P == 1) {  // [x0 x1] M = [r0 r1], M = a I - C
        m00 = B[0][0] - B[1][1]; m01 = -B[1][2]; m10 = -B[2][1]; m11 = B[0][0] - B[2][2];
        r0 = B[0][1]; r1 = B[0][2];
    } else {  // M [x0; x1] = [r0; r1], M = A - c I
        m00 = B[0][0] - B[2][2]; m01 = B[0][1]; m10 = B[1][0]; m11 = B[1][1] - B[2][2];
        r0 = B[0][2]; r1 = B[1][2];
    }
    const double det = m00 * m11 - m01 * m10;
    if (!(fabs(det) > 0.0)) return false;
    const double rd = 1.0 / det;
    double x0 = 0.0, x1 = 0.0, e0 = r0, e1 = r1;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        if constexpr (P == 1) {  // row vector: e M^-1
            x0 += (e0 * m11 - e1 * m10) * rd;
            x1 += (e1 * m00 - e0 * m01) * rd;
            if (pass == 0) { e0 = r0 - (x0 * m00 + x1 * m10); e1 = r1 - (x0 * m01 + x1 * m11); }
        } else {  // column vector: M^-1 e
            x0 += (m11 * e0 - m01 * e1) * rd;
            x1 += (m00 * e1 - m10 * e0) * rd;
            if (pass == 0) { e0 = r0 - (m00 * x0 + m01 * x1); e1 = r1 - (m10 * x0 + m11 * x1); }
        }
    }
    X[0] = x0; X[1] = x1;
    return isfinite(x0) && isfinite(x1);
}

// Orthogonal Qm (N x N) and the swapped block Bn = Qm^T B Qm for block sizes (P, Q).
template <int P, int Q>
__device__ __forceinline__ bool swap_transform(const double (&B)[P + Q][P + Q], double (&Qm)[P + Q][P + Q],
                                               double (&Bn)[P + Q][P + Q]) {
    constexpr int N = P + Q;
    double bnorm = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) bnorm = fmax(bnorm, fabs(B[i][j]));
    bnorm *= N;  // >= Frobenius norm
    if constexpr (P == 1 && Q == 1) {
        const double a = B[0][0], b = B[0][1], c = B[1][1];
        const double x0 = b, x1 = c - a;
        Qm[0][0] = 1.0; Qm[0][1] = 0.0; Qm[1][0] = 0.0; Qm[1][1] = 1.0;
        if (x0 == 0.0 && x1 == 0.0) {
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int j = 0; j < N; ++j) Bn[i][j] = B[i][j];
            return true;
        }
        const double rr = hypot(x0, x1);
        const double cs = x0 / rr, sn = x1 / rr;
        Qm[0][0] = cs; Qm[1][0] = sn; Qm[0][1] = -sn; Qm[1][1] = cs;
        Bn[0][0] = c; Bn[0][1] = b; Bn[1][0] = 0.0; Bn[1][1] = a;
        return true;
    } else {
        if constexpr (P == 2 && Q == 2) {
            double Xc[4];
            if (sylv22_closed(B, Xc) && swap_from_x<2, 2>(B, Xc, bnorm, Qm, Bn)) return true;
        } else {
            double Xc[2];
            if (sylv12_closed<P, Q>(B, Xc) && swap_from_x<P, Q>(B, Xc, bnorm, Qm, Bn)) return true;
        }
        constexpr int K = P * Q;
        double M[K][K], rhs[K], X[K];
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int j = 0; j < K; ++j) M[i][j] = 0.0;
        // unknown X(i, j) at index i + P j; equation (i, j): sum_k A(i,k) X(k,j) - sum_k X(i,k) C(k,j) = B(i, P+j)
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int row = i + P * j;
                rhs[row] = B[i][P + j];
#pragma unroll
                for (int k = 0; k < P; ++k) M[row][k + P * j] += B[i][k];
#pragma unroll
                for (int k = 0; k < Q; ++k) M[row][i + P * k] -= B[P + k][P + j];
            }
        if (!solve_cp<K>(M, rhs, X)) return false;
        return swap_from_x<P, Q>(B, X, bnorm, Qm, Bn);
    }
}

// ---------------------------------------------------------------- rounds of swaps
//
// Blocks that move up ("movers") are swapped past the blocks above them in
// rounds: in one round every mover whose upper neighbour is not a mover swaps
// with it.  The pairs of a round are disjoint, so their transforms act on
// disjoint rows and columns and commute; the order of the swaps along each path
// is that of moving the blocks one after another.  A round computes all
// transforms first, one per lane, wave (p - 1) * 2 + (q - 1) those of a p x p
// block above a q x q one (a transform is 700 dependent instructions for two 2x2
// blocks: it costs a round once, not once per swap), then applies them from the
// left to the rows right of each pair, then from the right to the columns above
// it and to V.  What bounds a round is the 2x2-2x2 transform and the four
// barriers (about 7000 cycles).  Measured on MI355X: random 64-row deflation
// windows (555 swaps each) 1.80 -> 0.73 million cycles, the random n = 20000
// reduction 1.11 -> 0.83 s; 96-row reordering windows 1183 -> 418 us.

// Block starts of the quasi-triangular window T, no movers.  All NTH threads
// call, after a barrier; ends with one.
template <int NTH = NT>
__device__ __forceinline__ void swap_begin(SwapState &w, const double *T, int ld, int nw) {
    for (int r = threadIdx.x; r <= nw; r += NTH) {
        w.head[r] = r == 0 || r == nw || AT(T, ld, r, r - 1) == 0.0;
        if (r < nw) w.mover[r] = 0;
    }
    if (threadIdx.x == 0) {
        w.total = 0;
        w.rejected = 0;
        for (int t = 0; t < 4; ++t) w.cnt[t] = 0;
    }
    __syncthreads();
}

// Whether the block at row r is a mover that goes up this round, and then its pair:
// p rows above it, q of its own.
__device__ __forceinline__ bool swap_pair(const SwapState &w, int r, int top, int &p, int &q) {
    if (!w.mover[r]) return false;
    p = w.head[r - 1] ? 1 : 2;
    q = w.head[r + 1] ? 1 : 2;
    return r - p >= top && !w.mover[r - p];
}

// The pairs of a round that has more than SWAP_PAIRS: the first ones from the top.
// Which ones go first decides in which order their transforms meet in a row and a
// column, so it must not be left to the order in which the waves come in: results are
// the same bit for bit.  Waves 0..3 each go through the rows, wave t lists type t.
__device__ __forceinline__ void swap_first_pairs(SwapState &w, int wave, int top, int kend) {
    if (wave >= 4) return;
    const int lane = threadIdx.x & (LANES - 1);
    const unsigned long long below = (1ull << lane) - 1ull;
    int total = 0, mine = 0;
    for (int r0 = top + 1; r0 < kend && total < SWAP_PAIRS; r0 += LANES) {
        const int r = r0 + lane;
        int p = 1, q = 1;
        const bool up = r < kend && swap_pair(w, r, top, p, q);
        const unsigned long long all = __ballot(up);
        const int slot = total + __popcll(all & below);
        const bool take = up && (p - 1) * 2 + (q - 1) == wave && slot < SWAP_PAIRS;
        const unsigned long long taken = __ballot(take);
        if (take) {
            w.st[slot] = r - p;
            w.n[slot] = p + q;
            w.list[wave][mine + __popcll(taken & below)] = slot;
        }
        total += __popcll(all);
        mine += __popcll(taken);
    }
    if (lane == 0) w.cnt[wave] = mine;
}

// The transforms of one type's pairs, one per lane.
template <int P, int Q>
__device__ __forceinline__ void swap_transforms(SwapState &w, int type, double *T, int ld) {
    constexpr int N = P + Q;
    const int lane = threadIdx.x & (LANES - 1);
    if (lane >= w.cnt[type]) return;
    const int slot = w.list[type][lane];
    const int st = w.st[slot];
    double B[N][N], Qm[N][N], Bn[N][N];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) B[i][j] = AT(T, ld, st + i, st + j);
    if (!swap_transform<P, Q>(B, Qm, Bn)) {
        w.st[slot] = -1;
        w.rejected = 1;
        return;
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            w.q[slot][i + N * j] = Qm[i][j];
            AT(T, ld, st + i, st + j) = Bn[i][j];
        }
    w.mover[st + P] = 0;
    w.head[st + P] = P == Q;
    w.head[st + Q] = 1;
    w.mover[st] = 1;
}

// Apply a pair's transform: rows st.. right of the pair (left), or columns st..
// of the rows above it and of V (right); one wave.
template <int N>
__device__ __forceinline__ void swap_apply(double *T, double *V, int ld, int nw, int st, const double *q, bool left) {
    const int lane = threadIdx.x & (LANES - 1);
    double Qm[N][N];
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int i = 0; i < N; ++i) Qm[i][j] = q[i + N * j];
    if (left) {
        for (int c = st + N + lane; c < nw; c += LANES) {
            double o[N];
#pragma unroll
            for (int i = 0; i < N; ++i) o[i] = AT(T, ld, st + i, c);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                double d = 0.0;
#pragma unroll
                for (int k = 0; k < N; ++k) d += Qm[k][i] * o[k];
                AT(T, ld, st + i, c) = d;
            }
        }
    } else {
        for (int it = lane; it < st + nw; it += LANES) {
            double *p = (it < st) ? &AT(T, ld, it, st) : &AT(V, ld, it - st, st);
            double o[N];
#pragma unroll
            for (int k = 0; k < N; ++k) o[k] = p[(size_t)k * ld];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                double d = 0.0;
#pragma unroll
                for (int k = 0; k < N; ++k) d += o[k] * Qm[k][j];
                p[(size_t)j * ld] = d;
            }
        }
    }
}

template <int NTH = NT>
__device__ __forceinline__ void swap_apply_all(SwapState &w, double *T, double *V, int ld, int nw, int pairs,
                                               bool left) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
    for (int s = wave; s < pairs; s += NTH / LANES) {
        const int st = __builtin_amdgcn_readfirstlane(w.st[s]), n = __builtin_amdgcn_readfirstlane(w.n[s]);
        if (st < 0) continue;
        if (n == 2) swap_apply<2>(T, V, ld, nw, st, w.q[s], left);
        else if (n == 3) swap_apply<3>(T, V, ld, nw, st, w.q[s], left);
        else swap_apply<4>(T, V, ld, nw, st, w.q[s], left);
    }
}

// One round on rows top..kend-1: every mover swaps with the block above it if
// that is not a mover.  Returns the number of pairs (0: nothing can move); all
// NTH threads call, after a barrier; ends with one.
template <int NTH = NT>
__device__ __forceinline__ int swap_round(SwapState &w, double *T, double *V, int ld, int nw, int top, int kend) {
    static_assert(NTH >= 4 * LANES, "a wave per type of pair");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / LANES);
    for (int r = top + 1 + (int)threadIdx.x; r < kend; r += NTH) {
        int p, q;
        if (!swap_pair(w, r, top, p, q)) continue;
        const int slot = atomicAdd(&w.total, 1);
        if (slot >= SWAP_PAIRS) continue;
        const int type = (p - 1) * 2 + (q - 1);
        w.st[slot] = r - p;
        w.n[slot] = p + q;
        w.list[type][atomicAdd(&w.cnt[type], 1)] = slot;
    }
    __syncthreads();
    const int found = w.total, pairs = min(found, SWAP_PAIRS);
    if (pairs == 0) return 0;
    if (found > SWAP_PAIRS) {
        swap_first_pairs(w, wave, top, kend);
        __syncthreads();
    }
    if (wave == 0) swap_transforms<1, 1>(w, 0, T, ld);
    else if (wave == 1) swap_transforms<1, 2>(w, 1, T, ld);
    else if (wave == 2) swap_transforms<2, 1>(w, 2, T, ld);
    else if (wave == 3) swap_transforms<2, 2>(w, 3, T, ld);
    __syncthreads();
    swap_apply_all<NTH>(w, T, V, ld, nw, pairs, true);
    if (threadIdx.x == 0) {
        w.total = 0;
        for (int t = 0; t < 4; ++t) w.cnt[t] = 0;
    }
    __syncthreads();
    swap_apply_all<NTH>(w, T, V, ld, nw, pairs, false);
    __syncthreads();
    // the 2x2 blocks of a swapped pair are similar to the old ones but not in
    // standard form; the caller standardises them once, after all swaps
    return pairs;
}

// ---------------------------------------------------------------- Householder helpers

// Sum over the four lanes of a quad; the same in all four.
__device__ __forceinline__ double quad_sum(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xf, 0xf, true);
    v += __hiloint2double(hi, lo);
    const int lo2 = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x4E, 0xf, 0xf, true);
    const int hi2 = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x4E, 0xf, 0xf, true);
    return v + __hiloint2double(hi2, lo2);
}

// The Householder vector of g(0..len-1), computed by every wave on its own (no
// barrier) and written to x with x[0] = 1 by the first; tau = 0 when the tail is
// zero.  sc scales the vector into range.
template <class G>
__device__ __forceinline__ void win_house(G g, double *x, int len, double *tau, double *beta) {
    const int lane = threadIdx.x & (LANES - 1);
    const double alpha = g(0);
    double mx = 0.0;
    for (int t = 1 + lane; t < len; t += LANES) mx = fmax(mx, fabs(g(t)));
    mx = wave_max(mx);
    if (mx == 0.0) {
        *tau = 0.0;
        *beta = alpha;
        return;
    }
    const double sc = fmax(mx, fabs(alpha)), rs = 1.0 / sc;
    double ss = 0.0;
    for (int t = 1 + lane; t < len; t += LANES) ss += (g(t) * rs) * (g(t) * rs);
    ss = wave_sum(ss) + (alpha * rs) * (alpha * rs);
    const double nrm = sc * sqrt(ss);
    const double b = alpha >= 0.0 ? -nrm : nrm;
    *tau = (b - alpha) / b;
    *beta = b;
    const double inv = 1.0 / (alpha - b);
    if (threadIdx.x < LANES)
        for (int t = lane; t < len; t += LANES) x[t] = (t == 0) ? 1.0 : g(t) * inv;
}

// Householder vectors are applied by quads: the four lanes of a quad share a
// column (left) or a row (right) and take every fourth element of the vector, so
// a window's 64 columns or rows go through in one pass of quarter length
// (64-row windows, 39 columns reduced: 0.56 -> 0.28 million cycles; one thread per
// column or row and block-wide reductions before).

// rows r0..r0+len-1 of M, columns c0..c1, from the left by I - tau v v^T
template <int NTH = NT>
__device__ __forceinline__ void win_refl_left(double *M, int ld, int r0, int len, int c0, int c1, double tau,
                                              const double *v) {
    const int part = threadIdx.x & 3;
    for (int j0 = c0; j0 <= c1; j0 += NTH / 4) {
        const int j = j0 + (int)threadIdx.x / 4;
        const bool on = j <= c1;
        double *p = &AT(M, ld, r0, on ? j : c1);
        double d = 0.0;
        for (int t = part; t < len; t += 4) d += v[t] * p[t];
        d = tau * quad_sum(d);
        if (on)
            for (int t = part; t < len; t += 4) p[t] -= d * v[t];
    }
}

// columns c0..c0+len-1 of M (rows 0..r1) and of M2 (rows 0..r2-1), from the right
template <int NTH = NT>
__device__ __forceinline__ void win_refl_right2(double *M, int ld, int r1, double *M2, int r2, int c0, int len,
                                                double tau, const double *v) {
    const int part = threadIdx.x & 3;
    const int total = r1 + 1 + r2;
    for (int i0 = 0; i0 < total; i0 += NTH / 4) {
        const int it = i0 + (int)threadIdx.x / 4;
        const bool on = it < total;
        const int i = on ? it : total - 1;
        double *p = (i <= r1) ? &AT(M, ld, i, c0) : &AT(M2, ld, i - r1 - 1, c0);
        double d = 0.0;
        for (int t = part; t < len; t += 4) d += p[(size_t)t * ld] * v[t];
        d = tau * quad_sum(d);
        if (on)
            for (int t = part; t < len; t += 4) p[(size_t)t * ld] -= d * v[t];
    }
}

// ---------------------------------------------------------------- AED

// Result of the AED core (returned in every thread).
struct AedOut {
    int nd;       // deflated count
    int nritz;    // Ritz values written
    int infqr;    // rows not converged by the window QR
    int swapfail; // a swap was rejected
    int iters;    // window QR iterations
    int nswap;    // block swaps
    int late;     // deflations found above a failed block
    double spike0;  // new coupling entry h(kwtop, kwtop-1) when nd > 0
    long long cyc_qr, cyc_defl, cyc_hess;
};

// AED on the nw x nw window already in LDS (T upper Hessenberg, V = I), coupled
// to the rest by the spike s (Section 3.2, "AED step"): Schur form of T by the
// window QR, spike test bottom-up with failing blocks moved to the top by block
// swaps, undeflated Ritz values written to sr/si (thread 0), and, if anything
// deflated, the spike and the undeflated part reduced back to Hessenberg form.
// On return T and V hold the transformed window and its orthogonal factor.
// Spike test of the diagonal block at j (size bs) of the AED window: the
// window criterion |s v| <= max(smlnum, eps |lambda|) (criterion 0) or the
// norm-stable |s v| <= max(smlnum, eps ||H||_F) (criterion 1), v the block's
// entries in the first row of V.
__device__ __forceinline__ bool aed_block_deflates(const double *T, const double *V, int ld, double s, int j, int bs,
                                                   double hnorm, double smlnum, int criterion) {
    double sp = fabs(s * AT(V, ld, 0, j));
    if (bs == 2) sp = fmax(sp, fabs(s * AT(V, ld, 0, j + 1)));
    double tol;
    if (criterion == 1) {
        tol = NEIG_EPS * hnorm;
    } else {
        double lam = (bs == 1) ? fabs(AT(T, ld, j, j))
                               : sqrt(fabs(AT(T, ld, j, j) * AT(T, ld, j + 1, j + 1) -
                                           AT(T, ld, j, j + 1) * AT(T, ld, j + 1, j)));
        if (lam == 0.0) lam = fabs(s);
        tol = NEIG_EPS * lam;
    }
    tol = fmax(tol, smlnum);
    return sp <= tol;
}

// Second half of the AED step on a window already in real Schur form (rows
// 0..o.infqr-1 unconverged and never tested): the spike test bottom-up with
// block swaps, standardisation of the deflated 2x2 blocks, the undeflated Ritz
// values, and the reduction of the spike and the undeflated part back to
// Hessenberg form.  T, V and the vector scratch x (nw doubles) may be in LDS or
// in global memory (generic pointers); all NTH threads call.
template <int NTH = NT>
__device__ __forceinline__ void aed_deflate(double *T, double *V, int ld, double *x, int nw, double s, double hnorm,
                                            double smlnum, int criterion, double *sr, double *si, AedOut &o) {
    const int tid = threadIdx.x;
    const long long c1 = clock64();
    o.nswap = 0;
    o.late = 0;
    o.swapfail = 0;
    SwapState &w = win_scratch().sw;
    swap_begin<NTH>(w, T, ld, nw);
    const int top = o.infqr;
    int kend = nw;
    bool moving = false;
    while (kend > top) {
        // test the bottom block unless it is on its way up; what lies below a
        // block that failed has already passed it
        const int j = w.head[kend - 1] ? kend - 1 : kend - 2;
        if (!w.mover[j]) {
            const int bs = kend - j;
            if (aed_block_deflates(T, V, ld, s, j, bs, hnorm, smlnum, criterion)) {
                if (moving) o.late += bs;
                kend = j;
                continue;
            }
            moving = true;
            __syncthreads();  // every thread has read the marks
            if (tid == 0) w.mover[j] = 1;
            __syncthreads();
        }
        const int pairs = swap_round<NTH>(w, T, V, ld, nw, top, kend);
        if (pairs == 0) break;  // all movers have arrived
        if (w.rejected) {
            // the rest counts as undeflatable
            o.swapfail = 1;
            break;
        }
        o.nswap += pairs;
    }
    o.nd = nw - kend;
    // standard form for the deflated 2x2 blocks (swaps leave them in any form);
    // a block whose eigenvalues came out real is split into two 1x1 blocks
    for (int j = kend; j + 1 < nw;) {
        if (AT(T, ld, j + 1, j) != 0.0) {
            const double a = AT(T, ld, j, j), b = AT(T, ld, j, j + 1), c = AT(T, ld, j + 1, j), d = AT(T, ld, j + 1, j + 1);
            if (!(a == d && b * c < 0.0)) lds_standardise<NTH>(T, ld, V, ld, nw, j);
            j += 2;
        } else {
            ++j;
        }
    }
    const long long c2 = clock64();

    // undeflated Ritz values (shift candidates), top to bottom
    int c = 0;
    for (int j = o.infqr; j < kend;) {
        if (j + 1 < kend && AT(T, ld, j + 1, j) != 0.0) {
            if (tid == 0) {
                double re1, im1, re2, im2;
                eig2x2(AT(T, ld, j, j), AT(T, ld, j, j + 1), AT(T, ld, j + 1, j), AT(T, ld, j + 1, j + 1), &re1,
                       &im1, &re2, &im2);
                sr[c] = re1; si[c] = im1; sr[c + 1] = re2; si[c + 1] = im2;
            }
            c += 2;
            j += 2;
        } else {
            if (tid == 0) {
                sr[c] = AT(T, ld, j, j);
                si[c] = 0.0;
            }
            ++c;
            ++j;
        }
    }
    o.nritz = c;
    o.spike0 = 0.0;
    o.cyc_defl = c2 - c1;
    o.cyc_hess = 0;
    if (o.nd == 0) return;

    if (kend > 0 && s != 0.0) {
        __syncthreads();
        if (kend > 1) {
            double tau, beta;
            win_house([&](int t) { return s * AT(V, ld, 0, t); }, x, kend, &tau, &beta);
            o.spike0 = beta;
            __syncthreads();
            if (tau != 0.0) {
                win_refl_left<NTH>(T, ld, 0, kend, 0, nw - 1, tau, x);
                __syncthreads();
                win_refl_right2<NTH>(T, ld, kend - 1, V, nw, 0, kend, tau, x);
                __syncthreads();
            }
            // Householder Hessenberg reduction of the undeflated leading block
            for (int cc = 0; cc + 2 < kend; ++cc) {
                const int len = kend - cc - 1;
                double *col = &AT(T, ld, cc + 1, cc);
                double tau2, beta2;
                win_house([&](int t) { return col[t]; }, x, len, &tau2, &beta2);
                __syncthreads();
                if (tau2 == 0.0) continue;
                for (int t = tid; t < len; t += NTH) col[t] = (t == 0) ? beta2 : 0.0;
                win_refl_left<NTH>(T, ld, cc + 1, len, cc + 1, nw - 1, tau2, x);
                __syncthreads();
                win_refl_right2<NTH>(T, ld, kend - 1, V, nw, cc + 1, len, tau2, x);
                __syncthreads();
            }
        } else {
            o.spike0 = s * AT(V, ld, 0, 0);
        }
    }
    __syncthreads();
    o.cyc_hess = clock64() - c2;
}

template <int NTH = NT>
__device__ __forceinline__ AedOut aed_core(double *T, double *V, int ld, double *x, int nw, double s, double hnorm,
                                           double smlnum, int criterion, int maxit, double *sr, double *si) {
    AedOut o;
    const long long c0 = clock64();
    o.iters = 0;
    o.infqr = lds_small_qr(T, ld, V, ld, nw, hnorm, smlnum, maxit, &o.iters);
    __syncthreads();
    o.cyc_qr = clock64() - c0;
    aed_deflate<NTH>(T, V, ld, x, nw, s, hnorm, smlnum, criterion, sr, si, o);
    return o;
}

// One AED window of a k_aed launch.  flip = 0: the trailing window of the
// active block [ktop, kbot] (rows/cols kbot-nw+1..kbot, coupled to the rest by
// H(kwtop, kwtop-1)).  flip = 1: the leading window (rows/cols ktop..ktop+nw-1,
// coupled by H(ktop+nw, ktop+nw-1)), handled as the trailing window of the
// flipped block J B^T J (B the active block, J the reversal), which is upper
// Hessenberg again: the window is loaded as J W^T J, the same AED runs on it,
// and the result is mapped back (T -> J T^T J, V -> J V J), so its deflated
// eigenvalues end at the top of the window.
struct AedJob {
    int ktop, kbot, nw, flip;
    double *Vt;   // V^T out (ld ldvt)
    int *status;  // 12 ints (layout below)
    double *sr, *si;
};

struct AedJobs {
    AedJob j[2];
};

// status: [0] nd (deflated count), [1] number of Ritz values written to sr/si,
// [2] 1 if H and the window transform V were updated (the host then applies V^T
// to the rest of H and Z), [3] rows not converged by the window QR, [4] 1 if a
// swap was rejected, [5] window QR iterations, [6] block swaps, [7..9] shader
// clock cycles spent in the window QR, the spike test with its swaps, and the
// re-Hessenberg reduction with the write-back, [10] deflations found above a
// block that failed the test.
extern "C" __global__ void __launch_bounds__(AED_THREADS)
k_aed(double *H, int ldh, AedJobs jobs, double hnorm, double smlnum, int criterion, int maxit, int ldvt) {
    extern __shared__ double lds[];
    const AedJob J = jobs.j[blockIdx.x];
    const int nw = J.nw;
    const int ld = nw + 1;
    double *T = lds;
    double *V = lds + (size_t)nw * ld;
    double *x = V + (size_t)nw * ld;  // nw doubles of vector scratch
    int off;
    double s;
    if (!J.flip) {
        off = J.kbot - nw + 1;
        s = (off > J.ktop) ? AT(H, ldh, off, off - 1) : 0.0;
        lds_load_block<AED_THREADS>(H, ldh, off, nw, T, ld, V, ld);
    } else {
        off = J.ktop;
        s = (off + nw <= J.kbot) ? AT(H, ldh, off + nw, off + nw - 1) : 0.0;
        for (int idx = threadIdx.x; idx < nw * nw; idx += AED_THREADS) {
            const int i = idx % nw, j = idx / nw;
            AT(T, ld, i, j) = (i <= j + 1) ? AT(H, ldh, off + nw - 1 - j, off + nw - 1 - i) : 0.0;
            AT(V, ld, i, j) = (i == j) ? 1.0 : 0.0;
        }
        __syncthreads();
    }
    const AedOut o = aed_core<AED_THREADS>(T, V, ld, x, nw, s, hnorm, smlnum, criterion, maxit, J.sr, J.si);
    if (threadIdx.x == 0) {
        int *status = J.status;
        status[0] = o.nd;
        status[1] = o.nritz;
        status[2] = (o.nd > 0) ? 1 : 0;
        status[3] = o.infqr;
        status[4] = o.swapfail;
        status[5] = o.iters;
        status[6] = o.nswap;
        status[7] = (int)min(o.cyc_qr, (long long)INT_MAX);
        status[8] = (int)min(o.cyc_defl, (long long)INT_MAX);
        status[9] = (int)min(o.cyc_hess, (long long)INT_MAX);
        status[10] = o.late;
    }
    if (o.nd == 0) return;  // H untouched; only the shifts are used
    if (!J.flip) {
        lds_store<AED_THREADS>(H, ldh, off, nw, T, ld, V, ld, J.Vt, ldvt);
        if (off > J.ktop && threadIdx.x == 0) AT(H, ldh, off, off - 1) = o.spike0;
    } else {
        for (int idx = threadIdx.x; idx < nw * nw; idx += AED_THREADS) {
            const int r = idx % nw, c = idx / nw;
            AT(H, ldh, off + r, off + c) = (r <= c + 1) ? AT(T, ld, nw - 1 - c, nw - 1 - r) : 0.0;
            AT(J.Vt, ldvt, r, c) = AT(V, ld, nw - 1 - c, nw - 1 - r);
        }
        if (off + nw <= J.kbot && threadIdx.x == 0) AT(H, ldh, off + nw, off + nw - 1) = o.spike0;
    }
}

// ---------------------------------------------------------------- reordering window

#define REORDER_WMAX 96

struct ReorderWin {
    int off, w;             // the window: rows/cols off .. off+w-1 of S
    int sel[REORDER_WMAX];  // 1 at the positions of selected eigenvalues of the window
};

// Reorder non-overlapping w x w diagonal windows of the quasi-triangular S, one
// workgroup per window (window b = wins[blockIdx.x]; its factor goes to
// Vt + b * ldvt * ldvt, its status to status + 2 b).  In each window at (off, off): the
// selected blocks move to the top of the window in their order, by swaps of
// adjacent diagonal blocks (the block exchange the paper's reordering phase
// uses), with the window's orthogonal factor accumulated in LDS.  The window
// must not split a 2x2 block.  Afterwards every 2x2 block of the window is put
// in standard form.  Outputs: the window back in S, its factor transposed in
// Vt, status[0] = selected eigenvalues now at the top, status[1] = 1 if a swap
// was rejected (the window is then partly reordered, still a valid Schur form).
// The caller applies Vt to the rest of S and to Z.
extern "C" __global__ void __launch_bounds__(REORDER_THREADS)
k_reorder_window(double *S, int lds_, const ReorderWin *wins, double *Vt_all, int ldvt, int *status_all) {
    extern __shared__ double lds[];
    const ReorderWin &f = wins[blockIdx.x];
    const int off = f.off, w = f.w;
    double *Vt = Vt_all + (size_t)blockIdx.x * ldvt * ldvt;
    int *status = status_all + 2 * blockIdx.x;
    const int ld = w + 1;
    double *T = lds, *V = lds + (size_t)w * ld;
    lds_load_block<REORDER_THREADS>(S, lds_, off, w, T, ld, V, ld);
    // every selected block moves up past the unselected ones above it
    SwapState &sw = win_scratch().sw;
    swap_begin<REORDER_THREADS>(sw, T, ld, w);
    for (int j = threadIdx.x; j < w; j += REORDER_THREADS) sw.mover[j] = sw.head[j] && f.sel[j];
    __syncthreads();
    while (swap_round<REORDER_THREADS>(sw, T, V, ld, w, 0, w) > 0 && !sw.rejected) {
    }
    const int fail = sw.rejected;
    int placed = 0;  // selected blocks at the top
    while (placed < w && sw.mover[placed]) placed += sw.head[placed + 1] ? 1 : 2;
    // standard form for every 2x2 block of the window (swaps leave them in any form)
    for (int k = 0; k + 1 < w;) {
        if (AT(T, ld, k + 1, k) != 0.0) {
            const double a = AT(T, ld, k, k), b = AT(T, ld, k, k + 1), c = AT(T, ld, k + 1, k), d = AT(T, ld, k + 1, k + 1);
            if (!(a == d && b * c < 0.0)) lds_standardise<REORDER_THREADS>(T, ld, V, ld, w, k);
            k += 2;
        } else {
            ++k;
        }
    }
    lds_store<REORDER_THREADS>(S, lds_, off, w, T, ld, V, ld, Vt, ldvt);
    if (threadIdx.x == 0) {
        status[0] = placed;
        status[1] = fail;
    }
}
