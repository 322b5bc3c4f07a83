// chase.hip -- the window task of the multishift sweep (Section 3.2).
//
// One workgroup per diagonal window.  A chain of up to 8 bulges, spaced three
// rows apart, is chased through the window; at each step every active bulge's
// 3-element reflector is applied from the left to the window's rows, from the
// right to the window's columns, and accumulated into the window's orthogonal
// factor U.  The window (and U) live in LDS with odd leading dimensions (no bank
// conflicts on strided columns); the kernel writes back the window and U^T, which
// the update kernels apply to the rest of H and to Z (the left/right update
// tasks).
//
// A step is a chain of dependent latencies, and with 12 waves on 4 SIMDs it is
// also bound by how many instructions the waves issue, so the work is split by
// who waits for it:
//
//  * near: wave b owns bulge b.  It applies its reflector to all
//    columns from the left (one column per lane), then, after a barrier, from the
//    right to the rows of the zone only: the rows between the trailing bulge and
//    the leading one (one row per lane, at most 30).  The lanes of rows
//    pos+1..pos+3 then hold the column that generates the bulge's next reflector;
//    every lane of the wave gets it through readlane and computes the reflector,
//    so it never passes through LDS.  Two barriers per step.  (Two bulges per wave
//    took 4300 cycles a step against 2000: more shifts run as more chains.)
//  * far: the rows above the zone and the rows of U see right reflections only, and
//    nothing in the window waits for them.  Four other waves apply them one batch
//    of 6 steps late: a lane loads its row's span of columns into registers, applies
//    the batch's reflectors (bulge by bulge: a bulge's columns lie
//    right of those of the bulges behind it at every earlier step, so this order
//    gives the same result), and stores it, with the steps' barriers in between.
//
// Measured on MI355X, 8 bulges in 64-row windows: 2030 cycles a step (1780 without
// the far waves), 3600 when all waves shared all rows and one wave built all
// reflectors; a launch 69 -> 45 us, the n = 4000 reduction of a dense matrix's form
// 856 -> 729 ms.  Giving the rows of U and H to one wave (half the reflector reads
// from LDS) was slower, 3000 cycles: its chain then exceeds the half steps.
#include "neig_dev.h"

#define CHASE_NEAR 8      // waves that own bulges
#define CHASE_FAR 4       // waves for the far rows
#define CHASE_THREADS (64 * (CHASE_NEAR + CHASE_FAR))
#define CHASE_MAX_BULGES CHASE_NEAR
#define CHASE_BATCH 6     // steps per far batch
#define CHASE_SPAN (3 * (CHASE_NEAR - 1) + CHASE_BATCH + 2)  // columns of eight bulges' batch

struct ChaseWin {
    int r0, r1;  // reflectors act on rows/cols r0..r1 (U is (r1-r0+1)^2)
    int t0, t1;  // chain steps [t0, t1)
    int chain;   // chain index; its bulges use polynomials chain*nbc + b
    int nb;      // bulges in this chain
};

struct ChaseArgs {
    ChaseWin win[NEIG_MAX_CHAINS];
    int nwin;
    int ktop, kbot;
    int nbc;   // bulges per full chain
    int ldut;  // leading dimension (and slot stride ldut*ldut) of the U^T outputs
    unsigned span;  // refl_span of ||H||_F, or REFL_LOCAL: of each window by itself
};

// Reflector of the bulge introduced at ktop (shifts of its polynomial
// z^2 - tr z + det, scaled), from the leading 3 x 2 corner of the active block
// (local index p of row ktop).
__device__ __forceinline__ ReflU chase_intro(const double *Hs, int ldhs, int p, int m3, double tr, double det,
                                             unsigned span) {
    const double h00 = AT(Hs, ldhs, p, p), h01 = AT(Hs, ldhs, p, p + 1);
    const double h10 = AT(Hs, ldhs, p + 1, p), h11 = AT(Hs, ldhs, p + 1, p + 1);
    const double h21 = (m3 == 3) ? AT(Hs, ldhs, p + 2, p + 1) : 0.0;
    double sc = fmax(fmax(fabs(h00), fabs(h01)), fmax(fmax(fabs(h10), fabs(h11)), fabs(h21)));
    sc = fmax(sc, fmax(fabs(tr), sqrt(fabs(det))));
    if (sc == 0.0) sc = 1.0;
    const double rs = 1.0 / sc;
    const double aa = h00 * rs, bb = h01 * rs, cc = h10 * rs, dd = h11 * rs, ee = h21 * rs;
    const double tt = tr * rs, dt = det * rs * rs;
    return refl_u(gen_vec(aa * aa + bb * cc - tt * aa + dt, cc * (aa + dd - tt), cc * ee, span));
}

// One batch of reflectors c[step][bulge] on one far row (on: this lane has one) of M
// (ncol columns); cfirst is the column of bulge 0 at the batch's first step.  full:
// a full batch of steps runs meanwhile, and its 48 reflectors are spread over its
// 12 half steps; else no barrier is met here.
template <bool full>
__device__ __forceinline__ void chase_far(double *M, int ldm, int ncol, int row, bool on, int cfirst,
                                          const double (*c)[CHASE_MAX_BULGES][4]) {
    const int c0 = cfirst - 3 * (CHASE_NEAR - 1);
    const bool inside = c0 >= 0 && c0 + CHASE_SPAN <= ncol;
    double x[CHASE_SPAN];
    double *p = M + row + (ptrdiff_t)c0 * ldm;
    double f[4][4];  // the next four reflectors
    auto fetch = [&](int u) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                f[e][v] = c[(u + e) % CHASE_BATCH][(u + e) / CHASE_BATCH][v];
    };
    fetch(0);
    if (inside) {
        if (on) {
#pragma unroll
            for (int k = 0; k < CHASE_SPAN; ++k) x[k] = p[(ptrdiff_t)k * ldm];
        }
    } else {
#pragma unroll
        for (int k = 0; k < CHASE_SPAN; ++k) {
            x[k] = 0.0;
            if ((unsigned)(c0 + k) < (unsigned)ncol && on) x[k] = p[(ptrdiff_t)k * ldm];
        }
    }
#pragma unroll
    for (int u = 0; u < CHASE_NEAR * CHASE_BATCH; u += 4) {
        double h[4][4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < 4; ++v) h[e][v] = f[e][v];
        // four reflectors are read ahead, and no more (left alone, the compiler
        // reads all of them first and runs out of registers)
        if (u + 4 < CHASE_NEAR * CHASE_BATCH) fetch(u + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 3 * (CHASE_NEAR - 1 - (u + e) / CHASE_BATCH) + (u + e) % CHASE_BATCH;
            const double t = h[e][0] * fma(h[e][1], x[k], fma(h[e][2], x[k + 1], h[e][3] * x[k + 2]));
            x[k] = fma(t, h[e][1], x[k]);
            x[k + 1] = fma(t, h[e][2], x[k + 1]);
            x[k + 2] = fma(t, h[e][3], x[k + 2]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the last barrier comes after the stores
        if (full && u + 4 < CHASE_NEAR * CHASE_BATCH) __builtin_amdgcn_s_barrier();
    }
    // the values exist from here on (else the compiler moves their arithmetic into
    // the branches of the stores)
#pragma unroll
    for (int k = 0; k < CHASE_SPAN; ++k) asm volatile("" : "+v"(x[k]));
    if (inside) {
        if (on) {
#pragma unroll
            for (int k = 0; k < CHASE_SPAN; ++k) p[(ptrdiff_t)k * ldm] = x[k];
        }
    } else {
#pragma unroll
        for (int k = 0; k < CHASE_SPAN; ++k)
            if ((unsigned)(c0 + k) < (unsigned)ncol && on) p[(ptrdiff_t)k * ldm] = x[k];
    }
    if (full) __syncthreads();
}

// A three-row reflector from the left on one column (if on), e its first entry.
__device__ __forceinline__ void chase_left3(double *e, bool on, const ReflU &r) {
    if (on) {
        const double x0 = e[0], x1 = e[1], x2 = e[2];
        const double s = r.q * fma(r.u0, x0, fma(r.u1, x1, r.u2 * x2));
        e[0] = fma(s, r.u0, x0);
        e[1] = fma(s, r.u1, x1);
        e[2] = fma(s, r.u2, x2);
    }
}

// A three-row reflector from the right on the zone's rows up to pos+3 (lane lx holds
// row pos+1, e its entry in column pos), and the bulge's next reflector from what
// column pos then holds in rows pos+1..pos+3.
__device__ __forceinline__ void chase_right3(double *e, int ld, int lane, int lx, unsigned span, ReflU &r) {
    const bool on = lane <= lx + 2;
    double x0 = 0.0, x1 = 0.0, x2 = 0.0;
    if (on) {
        x0 = e[0];
        x1 = e[ld];
        x2 = e[2 * ld];
    }
    const double s = r.q * fma(r.u0, x0, fma(r.u1, x1, r.u2 * x2));
    x0 = fma(s, r.u0, x0);
    x1 = fma(s, r.u1, x1);
    x2 = fma(s, r.u2, x2);
    const GenVec g = gen_vec(lane_value(x0, lx), lane_value(x0, lx + 1), lane_value(x0, lx + 2), span);
    if (on) {
        e[ld] = x1;
        e[2 * ld] = x2;
    }
    r = refl_u(g);
    x0 = pick(lane == lx, r.beta, pick(lane > lx, 0.0, x0));
    if (on) e[0] = x0;
}

// The near waves' part of one window: wave b chases bulge b.
__device__ __forceinline__ void chase_near(double *Hs, int ldhs, int mb, int b0, const ChaseWin &W, int ktop, int kbot,
                                           const double *poly, unsigned span,
                                           double (*cq)[CHASE_BATCH][CHASE_MAX_BULGES][4], int b) {
    const int lane = threadIdx.x & 63;
    const bool wide = W.r1 - W.r0 >= 64;
    int pos = ktop + W.t0 - 3 * b;
    bool act = b < W.nb && pos >= ktop && pos <= kbot - 1;
    ReflU r{0.0, 0.0, 0.0, 0.0, 0.0};
    if (act) {  // the reflector of the window's first step
        const int p = pos - b0, m3 = (pos <= kbot - 2) ? 3 : 2;
        if (pos == ktop) {
            r = chase_intro(Hs, ldhs, p, m3, poly[2 * b], poly[2 * b + 1], span);
        } else {
            double *c = &AT(Hs, ldhs, p, p - 1);
            r = refl_u(gen_vec(c[0], c[1], m3 == 3 ? c[2] : 0.0, span));
            if (lane < m3) c[lane] = lane == 0 ? r.beta : 0.0;
        }
    }
    __syncthreads();
    const int c0 = W.r0 - b0 + lane;  // this lane's (first) column
    int tb = W.t0, buf = 0, steps = 0;
    for (;; tb += CHASE_BATCH, buf ^= 1) {
        steps = min(CHASE_BATCH, W.t1 - tb);
        const int z0 = max(W.r0, ktop + tb - 3 * (W.nb - 1)) - b0;  // the zone's first row
        if (act && tb + CHASE_BATCH < W.t1 && pos + CHASE_BATCH + 2 <= kbot) {
            // the bulge goes through all steps of the batch and one more inside the
            // active block: no case distinctions in the steps
            int p = pos - b0;
            double *el = Hs + p + c0 * ldhs, *er = Hs + z0 + lane + p * ldhs, *c = cq[buf][0][b];
            // the loop starts 16 bytes into a unit of 32 (n = 4000 dense form: the chase
            // launches take 220.4 ms, 224.3 to 224.8 from its beginning or off by 4)
            asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
#pragma unroll 1
            for (int s = 0; s < CHASE_BATCH; ++s) {
                chase_left3(el, c0 >= p && c0 < mb, r);
                if (wide) chase_left3(el + 64 * ldhs, c0 + 64 >= p && c0 + 64 < mb, r);
                if (lane == 0) {
                    c[0] = r.q; c[1] = r.u0; c[2] = r.u1; c[3] = r.u2;
                }
                __syncthreads();
                chase_right3(er, ldhs, lane, p + 1 - z0, span, r);
                __syncthreads();
                ++p;
                ++el;
                er += ldhs;
                c += 4 * CHASE_MAX_BULGES;
            }
            pos += CHASE_BATCH;
            continue;
        }
        for (int t = tb; t < tb + steps; ++t) {
            const bool more = t + 1 < W.t1;
            const int p = pos - b0, lx = p + 1 - z0;
            const bool three = pos <= kbot - 2;
            // left: rows pos..pos+2 of columns pos..r1, one column per lane
            if (act) {
                double *e = Hs + p + c0 * ldhs;
                if (three) {
                    chase_left3(e, c0 >= p && c0 < mb, r);
                    if (wide) chase_left3(e + 64 * ldhs, c0 + 64 >= p && c0 + 64 < mb, r);
                } else {
                    for (int c = c0; c < mb; c += 64, e += 64 * ldhs)
                        if (c >= p) {
                            const double s = r.q * fma(r.u0, e[0], r.u1 * e[1]);
                            e[0] = fma(s, r.u0, e[0]);
                            e[1] = fma(s, r.u1, e[1]);
                        }
                }
            }
            if (lane == 0) {
                double *c = cq[buf][t - tb][b];
                c[0] = r.q; c[1] = r.u0; c[2] = r.u1; c[3] = r.u2;
            }
            __syncthreads();
            // right: the zone's rows up to pos+3 of columns pos..pos+2; the next reflector
            double *e = Hs + z0 + lane + p * ldhs;
            if (act && more && pos + 3 <= kbot) {
                chase_right3(e, ldhs, lane, lx, span, r);
            } else if (act) {
                const bool on = z0 + lane <= min(pos + 3, kbot) - b0;
                const bool build = more && pos + 1 <= kbot - 1;
                double x0 = 0.0, x1 = 0.0, x2 = 0.0;
                if (on) {
                    x0 = e[0];
                    x1 = e[ldhs];
                    if (three) x2 = e[2 * ldhs];
                }
                const double s = r.q * fma(r.u0, x0, fma(r.u1, x1, r.u2 * x2));
                x0 = fma(s, r.u0, x0);
                x1 = fma(s, r.u1, x1);
                x2 = fma(s, r.u2, x2);
                if (on) {
                    if (!(build && lane >= lx)) e[0] = x0;
                    e[ldhs] = x1;
                    if (three) e[2 * ldhs] = x2;
                }
                if (build) {  // pos + 3 > kbot: rows pos+1, pos+2 of column pos
                    r = refl_u(gen_vec(lane_value(x0, lx), lane_value(x0, lx + 1), 0.0, span));
                    if (on && lane >= lx) e[0] = lane == lx ? r.beta : 0.0;
                }
            }
            ++pos;
            act = more && b < W.nb && pos >= ktop && pos <= kbot - 1;
            if (!act) r.q = r.u0 = r.u1 = r.u2 = 0.0;
            __syncthreads();
            if (act && pos == ktop)  // enters with the next step
                r = chase_intro(Hs, ldhs, ktop - b0, (ktop <= kbot - 2) ? 3 : 2, poly[2 * b], poly[2 * b + 1], span);
        }
        if (tb + CHASE_BATCH >= W.t1) break;
    }
    // the rest of the last batch
    for (int s = steps; s < CHASE_BATCH; ++s)
        if (lane < 4) cq[buf][s][b][lane] = 0.0;
}

// The far waves' part: while batch j runs, batch j - 1 is applied.
__device__ __forceinline__ void chase_far_rows(double *Hs, int ldhs, int mb, double *Us, int ldus, int b0,
                                               const ChaseWin &W, int ktop,
                                               double (*cq)[CHASE_BATCH][CHASE_MAX_BULGES][4], int f) {
    const int lane = threadIdx.x & 63;
    const int w = W.r1 - W.r0 + 1;
    const bool isU = (f & 1) == 0;
    const int row = lane + 64 * (f >> 1);
    __syncthreads();
    int rows = 0, cfirst = 0;  // of the batch that is still to be applied
    for (int tb = W.t0;; tb += CHASE_BATCH) {
        const int steps = max(0, min(CHASE_BATCH, W.t1 - tb));
        const double(*c)[CHASE_MAX_BULGES][4] = cq[(((tb - W.t0) / CHASE_BATCH) & 1) ^ 1];
        double *M = isU ? Us : Hs;
        const int ldm = isU ? ldus : ldhs, ncol = isU ? w : mb;
        const bool any = rows > 64 * (f >> 1);
        if (any && steps == CHASE_BATCH) {
            chase_far<true>(M, ldm, ncol, row, row < rows, cfirst, c);
        } else {
            // one barrier when no step follows: the last batch's reflectors are complete
            for (int h = 0; h < max(1, 2 * steps); ++h) __syncthreads();
            if (any) chase_far<false>(M, ldm, ncol, row, row < rows, cfirst, c);
        }
        if (steps == 0) break;
        const int z0 = max(W.r0, ktop + tb - 3 * (W.nb - 1)) - b0;
        rows = isU ? w : z0;
        cfirst = ktop + tb - (isU ? W.r0 : b0);
    }
}

// One window by CHASE_THREADS threads: load, chase, write the window back to H.
// Hs and Us take mb and w columns of odd length; U stays in Us (leading dimension
// w | 1); ends with a barrier.
__device__ __forceinline__ void chase_window(double *H, int ldh, const ChaseWin &W, int ktop, int kbot,
                                             const double *poly, unsigned span, double *Hs, double *Us) {
    __shared__ double cq[2][CHASE_BATCH][CHASE_MAX_BULGES][4];  // two batches' reflectors (q, u0, u1, u2)
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = W.r0, r1 = W.r1;
    const int b0 = (r0 > 0) ? r0 - 1 : 0;
    const int mb = r1 - b0 + 1;  // LDS block order
    const int w = r1 - r0 + 1;   // U order
    const int ldhs = mb | 1, ldus = w | 1;

    // a wave takes every twelfth column, its rows over the lanes; all of a thread's
    // loads are in flight together (n = 4000 dense form 606 -> 601 ms, 512 batched
    // problems 230 -> 227 ms against a loop over single entries)
    const int lane = tid & 63;
    constexpr int WAVES = CHASE_THREADS / 64, PER = (NEIG_CHASE_MAX + 1 + WAVES - 1) / WAVES;
    const bool tall = mb > 64;
    const int i0 = min(lane, mb - 1), i1 = min(lane + 64, mb - 1);
    {
        double x[PER][2];
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const double *p = &AT(H, ldh, b0, b0 + min(wave + WAVES * c, mb - 1));
            x[c][0] = p[i0];
            if (tall) x[c][1] = p[i1];
        }
        for (int j = wave; j < w; j += WAVES) {
            if (lane < w) AT(Us, ldus, lane, j) = (lane == j) ? 1.0 : 0.0;
            if (lane + 64 < w) AT(Us, ldus, lane + 64, j) = (lane + 64 == j) ? 1.0 : 0.0;
        }
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int j = wave + WAVES * c;
            if (j < mb && lane < mb) AT(Hs, ldhs, lane, j) = x[c][0];
            if (j < mb && lane + 64 < mb) AT(Hs, ldhs, lane + 64, j) = x[c][1];
        }
        if (span == REFL_LOCAL) {
            double mx = 0.0;
#pragma unroll
            for (int c = 0; c < PER; ++c) mx = fmax(mx, fmax(fabs(x[c][0]), tall ? fabs(x[c][1]) : 0.0));
            span = refl_span((NEIG_CHASE_MAX + 1) * block_reduce<CHASE_THREADS>(mx, true));
        }
    }
    __syncthreads();
    // both kinds of waves meet the same barriers: one before the first step, two
    // per step, one after the last
    if (wave < CHASE_NEAR) {
        chase_near(Hs, ldhs, mb, b0, W, ktop, kbot, poly, span, cq, wave);
        __syncthreads();
    } else {
        chase_far_rows(Hs, ldhs, mb, Us, ldus, b0, W, ktop, cq, wave - CHASE_NEAR);
    }
    __syncthreads();

    // write back what the window changed: columns r0..r1 (rows b0..r1) and the three
    // entries of column b0 below r0
    const int off = r0 - b0;
    for (int j = off + wave; j < mb; j += WAVES) {
        if (lane < mb) AT(H, ldh, b0 + lane, b0 + j) = AT(Hs, ldhs, lane, j);
        if (lane + 64 < mb) AT(H, ldh, b0 + lane + 64, b0 + j) = AT(Hs, ldhs, lane + 64, j);
    }
    if (off == 1 && r0 > ktop && tid < 3 && tid + 1 < mb) AT(H, ldh, r0 + tid, b0) = AT(Hs, ldhs, 1 + tid, 0);
    __syncthreads();
}

extern "C" __global__ void __launch_bounds__(CHASE_THREADS)
k_chase(double *H, int ldh, const double *poly, double *Ut, ChaseArgs a) {
    extern __shared__ double lds[];
    const ChaseWin W = a.win[blockIdx.x];
    const int mb = W.r1 - ((W.r0 > 0) ? W.r0 - 1 : 0) + 1, w = W.r1 - W.r0 + 1;
    double *Us = lds + (size_t)mb * (mb | 1);
    chase_window(H, ldh, W, a.ktop, a.kbot, poly + 2 * (size_t)W.chain * a.nbc, a.span, lds, Us);
    double *Uo = Ut + (size_t)blockIdx.x * a.ldut * a.ldut;
    const int lane = threadIdx.x & 63;
    for (int c = threadIdx.x >> 6; c < w; c += CHASE_THREADS / 64) {
        if (lane < w) AT(Uo, a.ldut, lane, c) = AT(Us, w | 1, c, lane);
        if (lane + 64 < w) AT(Uo, a.ldut, lane + 64, c) = AT(Us, w | 1, c, lane + 64);
    }
}
