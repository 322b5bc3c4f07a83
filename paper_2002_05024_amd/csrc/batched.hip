// batched.hip -- many independent Schur reductions in one persistent launch.
//
// Each workgroup (12 waves) takes problems from a device work queue (largest
// first) and runs the whole method of Section 3.2 on its problem: splitting at
// negligible subdiagonals, the in-LDS double-shift QR for small blocks,
// aggressive early deflation on the trailing window, and single-chain
// multishift sweeps whose windows are chased in LDS.  The orthogonal factors
// never leave LDS: the workgroup applies them to its problem's off-diagonal
// strips of H and Z in HBM with FP64 matrix-core instructions.  All control
// decisions are taken on the device, so one launch covers the whole batch and
// can be captured in a graph.  Parallelism comes from the batch: one problem per
// CU at a time (a window and its factor take the CU's whole LDS).
//
// A batch ends with its largest problem, so what bounds it is the time of one
// problem on one CU.  Measured on MI355X, 512 problems of order 32 to 1024: 515 ms
// with 4 waves (window chasing in three phases, 14200 cycles a step of 16 bulges;
// updates through a staged tile, 1.06 million cycles a window), 227 ms now:
//  * the windows are chased by the sweep kernel's code (chase.hip: 2550 cycles a step
//    of 8 bulges), so the workgroup has its 12 waves;
//  * a factor is applied by each wave on its own, sixteen rows or columns at a time,
//    straight from memory into the matrix cores' layout and back (260 thousand cycles
//    a window; 435 thousand before the phases were functions of their own).
// What is left is the window QR and the spike test (half the time, one wave's
// chain of dependent steps) and, while all CUs work, the passes over H and Z.
#include "neig_dev.h"

#define BT CHASE_THREADS  // threads per workgroup
#define B_MAX_BULGES 16   // per sweep
#define B_NBUCKET 6

struct BProb {
    double *H, *Z, *wr, *wi;
    int n, ldh, ldz, pad;
};

struct BTune {
    int nw;      // AED window
    int ns;      // shifts per sweep (<= 2 * B_MAX_BULGES)
    int nmin;    // blocks of at most nmin rows go to the in-LDS QR
    int wchase;  // chase window
};

// The method's own operation count of one problem (the same formulas as the
// single-matrix path's neig_stats.alg_flops: 10 m^3 per window or small block solved in
// LDS, 2 m^2 per row or column its factor is applied to, 20 n per bulge position of a
// sweep), and what small blocks have of it.
struct BCount {
    double all, small;  // flops; small: the blocks' own 10 m^3
    int solves;         // small blocks
    int info;           // written for a problem alone
};

struct BArgs {
    const BProb *probs;
    const int *order;   // processing order (largest problems first)
    int nprob;
    int *next;          // work counter, zero before the launch; next + 2 (8-byte
                        // aligned) holds the launch's algorithmic flop count
                        // (a double), also zeroed by k_batched_pack
    int *info;          // per problem, in the caller's order
    BProb one;          // probs null: this problem alone (tune[0]); its counts go to *count
    struct BCount *count;
    int bucket_hi[B_NBUCKET];  // problems with n <= bucket_hi[b] use tune[b]
    BTune tune[B_NBUCKET];
    int criterion, nibble, exc, maxit_factor;
};

// What a problem's steps hand on to each other: the Ritz values of the last AED
// window, and the polynomials (trace, determinant) of the sweep's shift pairs.
struct BShifts {
    double rr[NEIG_SMALL_MAX], ri[NEIG_SMALL_MAX];
    double poly[2 * B_MAX_BULGES];
    int nritz, nsh;
};

__device__ __forceinline__ BShifts &batch_shifts() {
    __shared__ BShifts s;
    return s;
}

// ---------------------------------------------------------------- workgroup helpers

// ||H||_F over the Hessenberg part, zeros below the subdiagonal; false on NaN/Inf.
__device__ __forceinline__ bool wg_prep(double *H, int ldh, int n, double *hnorm) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double mx = 0.0;
    int bad = 0;
    for (int j = wave; j < n; j += BT / 64) {
        double *c = &AT(H, ldh, 0, j);
        for (int i = lane; i < n; i += 64) {
            if (i > j + 1) {
                c[i] = 0.0;
            } else {
                const double v = c[i];
                if (!isfinite(v)) bad = 1;
                else mx = fmax(mx, fabs(v));
            }
        }
    }
    mx = block_reduce<BT>(mx, true);
    const double anybad = block_reduce<BT>((double)bad, true);
    if (anybad != 0.0) return false;
    double ssq = 0.0;
    if (mx > 0.0) {
        for (int j = wave; j < n; j += BT / 64) {
            const double *c = &AT(H, ldh, 0, j);
            const int last = min(j + 1, n - 1);
            for (int i = lane; i <= last; i += 64) {
                const double v = c[i] / mx;
                ssq += v * v;
            }
        }
    }
    ssq = block_reduce<BT>(ssq, false);
    *hnorm = mx * sqrt(ssq);
    return true;
}

// Largest k in [1, kbot] whose subdiagonal is negligible (zeroed), else 0.
__device__ __forceinline__ int wg_scan(double *H, int ldh, int kbot, double hnorm, double smlnum) {
    double best = 0.0;
    for (int k = 1 + (int)threadIdx.x; k <= kbot; k += BT) {
        const double sub = AT(H, ldh, k, k - 1);
        if (sub == 0.0 || negligible_sub(sub, AT(H, ldh, k - 1, k - 1), AT(H, ldh, k, k), hnorm, smlnum)) {
            if (sub != 0.0) AT(H, ldh, k, k - 1) = 0.0;
            best = fmax(best, (double)k);
        }
    }
    return (int)block_reduce<BT>(best, true);
}

// Sixteen vectors of length w (NTL = ceil(w / 16)) times U, in place, by one wave:
// x_i <- U^T x_i, entry k of vector i at C[i * si + k * sk].  Columns of H (si = ldh,
// sk = 1) or rows of H and Z (si = 1, sk = ld: then lanes read and write runs of 16
// entries); vectors from len on are left alone.  U in LDS.
template <int NTL>
__device__ __forceinline__ void wave_update(double *C, size_t sk, size_t si, int len, int w, const double *U, int ldu) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const bool on = li < len;
    typedef __attribute__((address_space(1))) double global_double;  // also after the asm below
    global_double *const p = (global_double *)(C + (on ? li : 0) * si + lk * sk), *q = p;
    double b[4 * NTL];
#pragma unroll
    for (int s = 0; s < 4 * NTL; ++s, q += 4 * sk) {
        // entries past the end (in the last tile) count as zeros
        if (s < 4 * (NTL - 1)) {
            b[s] = *q;
        } else {
            b[s] = 0.0;
            if (4 * s + lk < w) b[s] = *q;
        }
    }
    neig_d4 acc[NTL];
    int col[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
        acc[t] = (neig_d4){0.0, 0.0, 0.0, 0.0};
        const int c = 16 * t + li;
        col[t] = ((t < NTL - 1) ? c : min(c, w - 1)) * ldu;
    }
    double a[NTL];
    auto fetch = [&](int s) __attribute__((always_inline)) {
        int k = 4 * s + lk;
        if (s >= 4 * (NTL - 1)) {
            k = min(k, w - 1);
            asm volatile("" : "+v"(k));  // computed here, not kept for the next tile
        }
#pragma unroll
        for (int t = 0; t < NTL; ++t) a[t] = U[k + col[t]];
    };
    fetch(0);
#pragma unroll
    for (int s = 0; s < 4 * NTL; ++s) {
        double f[NTL];
#pragma unroll
        for (int t = 0; t < NTL; ++t) f[t] = a[t];
        // one column of U is read ahead and no more: reads of all of them first would
        // not fit the registers
        if (s + 1 < 4 * NTL) fetch(s + 1);
#pragma unroll
        for (int t = 0; t < NTL; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[t], b[s], acc[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    q = p;
    asm volatile("" : "+v"(q));  // the loads' addresses are not kept for the stores
    if (on) {
#pragma unroll
        for (int s = 0; s < 4 * NTL; ++s, q += 4 * sk)
            if (s < 4 * (NTL - 1) || 4 * s + lk < w) *q = acc[s / 4][s % 4];
    }
}

// The rest of H and Z after rows and columns lo..lo+w-1 were transformed by U (w x w,
// in LDS): columns right..n-1 and rows 0..above-1 of H, all rows of Z.  The vectors
// are shared out to the waves sixteen at a time, without a barrier (they are
// disjoint); ends with one.
template <int NTL>
__device__ __forceinline__ void wg_update_tiles(double *H, int ldh, double *Z, int ldz, int n, int lo, int w, int above,
                                                int right, const double *U, int ldu) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tl = (n - right + 15) >> 4, ta = (above + 15) >> 4, tz = (n + 15) >> 4;
#pragma unroll 1
    for (int t = wave; t < tl + ta + tz; t += BT / 64) {
        double *C;
        size_t sk, si;
        int len;
        if (t < tl) {
            const int c = right + 16 * t;
            C = H + lo + (size_t)c * ldh;
            sk = 1;
            si = ldh;
            len = n - c;
        } else {
            const bool inH = t < tl + ta;
            const int r = 16 * (t - tl - (inH ? 0 : ta));
            C = (inH ? H : Z) + r + (size_t)lo * (inH ? ldh : ldz);
            sk = inH ? ldh : ldz;
            si = 1;
            len = (inH ? above : n) - r;
        }
        wave_update<NTL>(C, sk, si, len, w, U, ldu);
    }
}

// ---------------------------------------------------------------- phases
//
// The phases are functions of their own (not inlined): each then has the 168
// registers of a lane to itself, where in one body the compiler kept values of all
// phases alive and spilled in the innermost loops (the window QR 14% slower).  Their
// arguments arrive in vector registers; uni() makes them uniform again.  All
// BT threads call, after a barrier; all end with one.

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni(double v) {
    return __hiloint2double(uni(__double2hiint(v)), uni(__double2loint(v)));
}
__device__ __forceinline__ double *uni(double *p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned long long u = ((unsigned long long)(unsigned)uni((int)(v >> 32)) << 32) | (unsigned)uni((int)v);
    return (double *)(__attribute__((address_space(1))) double *)u;  // global memory, not LDS
}

// The rest of H and Z after rows and columns lo..lo+w-1 were transformed by the
// w x w matrix at lds + uoff.
__device__ __attribute__((noinline)) void b_update(double *H, int ldh, double *Z, int ldz, int n, int lo, int w, int above,
                                                   int right, int uoff, int ldu) {
    extern __shared__ double lds[];
    static_assert(NEIG_CHASE_MAX <= 96 && NEIG_SMALL_MAX <= 96, "six row tiles");
    H = uni(H); ldh = uni(ldh); Z = uni(Z); ldz = uni(ldz); n = uni(n); lo = uni(lo); w = uni(w);
    above = uni(above); right = uni(right); ldu = uni(ldu);
    const double *U = lds + uni(uoff);
    switch ((w + 15) >> 4) {
    case 1: wg_update_tiles<1>(H, ldh, Z, ldz, n, lo, w, above, right, U, ldu); break;
    case 2: wg_update_tiles<2>(H, ldh, Z, ldz, n, lo, w, above, right, U, ldu); break;
    case 3: wg_update_tiles<3>(H, ldh, Z, ldz, n, lo, w, above, right, U, ldu); break;
    case 4: wg_update_tiles<4>(H, ldh, Z, ldz, n, lo, w, above, right, U, ldu); break;
    case 5: wg_update_tiles<5>(H, ldh, Z, ldz, n, lo, w, above, right, U, ldu); break;
    default: wg_update_tiles<6>(H, ldh, Z, ldz, n, lo, w, above, right, U, ldu); break;
    }
    __syncthreads();
}

// The m x m diagonal block of H at off into LDS and its Schur form there, its factor
// behind it (leading dimensions m + 1); what lds_small_qr returns.
__device__ __attribute__((noinline)) int b_qr(const double *H, int ldh, int off, int m, double hnorm, double smlnum) {
    extern __shared__ double lds[];
    H = uni((double *)H); ldh = uni(ldh); off = uni(off); m = uni(m); hnorm = uni(hnorm); smlnum = uni(smlnum);
    const int ld = m + 1;
    double *Q = lds + (size_t)m * ld;
    lds_load_block<BT>(H, ldh, off, m, lds, ld, Q, ld);
    int iters = 0;
    return lds_small_qr(lds, ld, Q, ld, m, hnorm, smlnum, 30 * (m > 10 ? m : 10), &iters);
}

// Write the m x m block in LDS back to H's diagonal block at off.
__device__ __forceinline__ void b_store(double *H, int ldh, int off, int m) {
    extern __shared__ double lds[];
    for (int idx = threadIdx.x; idx < m * m; idx += BT) {
        const int i = idx % m, j = idx / m;
        AT(H, ldh, off + i, off + j) = (i <= j + 1) ? AT(lds, m + 1, i, j) : 0.0;
    }
}

// The deflation half of the AED step on the window in LDS (infqr: b_qr's result); the
// window back to H if anything deflated, the Ritz values to sr, si and their number to
// *nritz (all in LDS).  Returns the number of deflated rows.
__device__ __attribute__((noinline)) int b_deflate(double *H, int ldh, int ktop, int kwtop, int nw, int infqr, double s,
                                                   double hnorm, double smlnum, int criterion) {
    extern __shared__ double lds[];
    H = uni(H); ldh = uni(ldh); ktop = uni(ktop); kwtop = uni(kwtop); nw = uni(nw); infqr = uni(infqr);
    s = uni(s); hnorm = uni(hnorm); smlnum = uni(smlnum); criterion = uni(criterion);
    BShifts &b = batch_shifts();
    const int ld = nw + 1;
    double *V = lds + (size_t)nw * ld;
    AedOut o;
    o.infqr = infqr;
    aed_deflate<BT>(lds, V, ld, V + (size_t)nw * ld, nw, s, hnorm, smlnum, criterion, b.rr, b.ri, o);
    if (o.nd > 0) {
        b_store(H, ldh, kwtop, nw);
        if (kwtop > ktop && threadIdx.x == 0) AT(H, ldh, kwtop, kwtop - 1) = o.spike0;
    }
    if (threadIdx.x == 0) b.nritz = o.nritz;
    __syncthreads();
    return o.nd;
}

// One window of a sweep; its factor stays in LDS behind the window.
__device__ __attribute__((noinline)) void b_chase(double *H, int ldh, int ktop, int kbot, int r0, int r1, int t0, int t1,
                                                  int nb, int bulge0, unsigned span) {
    extern __shared__ double lds[];
    H = uni(H); ldh = uni(ldh); ktop = uni(ktop); kbot = uni(kbot);
    ChaseWin W;
    W.r0 = uni(r0); W.r1 = uni(r1); W.t0 = uni(t0); W.t1 = uni(t1); W.nb = uni(nb);
    W.chain = 0;
    const int mb = W.r1 - ((W.r0 > 0) ? W.r0 - 1 : 0) + 1;
    chase_window(H, ldh, W, ktop, kbot, batch_shifts().poly + 2 * uni(bulge0), (unsigned)uni((int)span), lds,
                 lds + (size_t)mb * (mb | 1));
}

// ---------------------------------------------------------------- shifts (thread 0)

// Up to ns shifts from the Ritz values (complex pairs kept together, real values
// paired), smallest magnitude first; returns the count written to (xr, xi).
__device__ __forceinline__ int pick_shifts_dev(const double *rr, const double *ri, int nr, int ns, double *xr, double *xi) {
    // items: complex pair (j, j+1) or a pair of reals
    double mag[64];
    int ia[64], ib[64];
    int nit = 0;
    int realidx[96];
    int nreal = 0;
    for (int t = 0; t < nr && nit < 64;) {
        if (ri[t] != 0.0 && t + 1 < nr) {
            mag[nit] = hypot(rr[t], ri[t]);
            ia[nit] = t;
            ib[nit] = t + 1;
            ++nit;
            t += 2;
        } else {
            if (nreal < 96) realidx[nreal++] = t;
            ++t;
        }
    }
    for (int a = 1; a < nreal; ++a) {  // reals by magnitude
        const int v = realidx[a];
        int b = a - 1;
        while (b >= 0 && fabs(rr[realidx[b]]) > fabs(rr[v])) {
            realidx[b + 1] = realidx[b];
            --b;
        }
        realidx[b + 1] = v;
    }
    for (int a = 0; a + 1 < nreal && nit < 64; a += 2) {
        mag[nit] = fmax(fabs(rr[realidx[a]]), fabs(rr[realidx[a + 1]]));
        ia[nit] = realidx[a];
        ib[nit] = realidx[a + 1];
        ++nit;
    }
    for (int a = 1; a < nit; ++a) {  // stable insertion sort by magnitude
        const double m = mag[a];
        const int x = ia[a], y = ib[a];
        int b = a - 1;
        while (b >= 0 && mag[b] > m) {
            mag[b + 1] = mag[b]; ia[b + 1] = ia[b]; ib[b + 1] = ib[b];
            --b;
        }
        mag[b + 1] = m; ia[b + 1] = x; ib[b + 1] = y;
    }
    int out = 0;
    for (int a = 0; a < nit && out + 2 <= ns; ++a) {
        xr[out] = rr[ia[a]]; xi[out] = ri[ia[a]];
        xr[out + 1] = rr[ib[a]]; xi[out + 1] = ri[ib[a]];
        out += 2;
    }
    return out;
}

// ---------------------------------------------------------------- one problem

// *cnt receives the operation count; every thread holds the same values.
__device__ __forceinline__ int solve_one(const BProb &P, const BTune &tu, const BArgs &A, BCount *cnt) {
    BShifts &sh = batch_shifts();
    const int tid = threadIdx.x;
    const int n = P.n;
    double *H = P.H, *Z = P.Z;
    const int ldh = P.ldh, ldz = P.ldz;
    *cnt = {0.0, 0.0, 0, 0};
    if (n <= 0) return 0;
    double hnorm = 0.0;
    if (!wg_prep(H, ldh, n, &hnorm)) return -2;
    const double smlnum = NEIG_DBL_MIN * ((double)n / NEIG_EPS);
    const int nmin = tu.nmin;
    const int maxit = A.maxit_factor * (n > 10 ? n : 10);
    int info = 0;
    int kbot = n - 1, total = 0, ndefl = 0;
    double fl = 0.0;
    while (kbot >= 0) {
        const int ktop = wg_scan(H, ldh, kbot, hnorm, smlnum);
        const int m = kbot - ktop + 1;
        if (m <= nmin) {
            if (m > 1) {  // whole block in LDS, then its factor to the rest
                const int bad = uni(b_qr(H, ldh, ktop, m, hnorm, smlnum));
                b_store(H, ldh, ktop, m);
                b_update(H, ldh, Z, ldz, n, ktop, m, ktop, kbot + 1, m * (m + 1), m + 1);
                fl += 10.0 * m * (double)m * m + 2.0 * m * (double)m * (ktop + (n - kbot - 1) + n);
                cnt->small += 10.0 * m * (double)m * m;
                cnt->solves++;
                if (bad > 0) {
                    info = ktop + bad;
                    break;
                }
            }
            kbot = ktop - 1;
            ndefl = 0;
            continue;
        }
        if (++total > maxit) {
            info = kbot + 1;
            break;
        }
        // AED on the trailing window
        int nw = tu.nw < m ? tu.nw : m;
        const int kwtop = kbot - nw + 1;
        const double spike = (kwtop > ktop) ? AT(H, ldh, kwtop, kwtop - 1) : 0.0;
        const int infqr = uni(b_qr(H, ldh, kwtop, nw, hnorm, smlnum));
        const int nd = uni(b_deflate(H, ldh, ktop, kwtop, nw, infqr, spike, hnorm, smlnum, A.criterion));
        fl += 10.0 * nw * (double)nw * nw;
        if (nd > 0) {
            fl += 2.0 * nw * (double)nw * (kwtop + (n - kbot - 1) + n);
            b_update(H, ldh, Z, ldz, n, kwtop, nw, kwtop, kbot + 1, nw * (nw + 1), nw + 1);
        }
        kbot -= nd;
        ndefl = (nd > 0) ? 0 : ndefl + 1;
        const int m2 = kbot - ktop + 1;
        if (m2 <= nmin) continue;
        const int nibble = A.nibble > 0 ? A.nibble : nibble_batched(m2);
        if (nd > 0 && 100 * nd > nibble * nw) continue;
        // shifts
        int ns = tu.ns;
        if (ns > 2 * B_MAX_BULGES) ns = 2 * B_MAX_BULGES;
        if (ns > m2 / 3) ns = m2 / 3;
        ns -= ns % 2;
        if (ns < 2) ns = 2;
        __syncthreads();
        if (tid == 0) {
            double xr[2 * B_MAX_BULGES], xi[2 * B_MAX_BULGES];
            int got = 0;
            if (ndefl > 0 && ndefl % A.exc == 0) {
                for (int i = kbot; i >= ktop + 2 && got + 2 <= ns; i -= 2) {
                    const double sx = fabs(AT(H, ldh, i, i - 1)) + fabs(AT(H, ldh, i - 1, i - 2));
                    const double c = AT(H, ldh, i, i);
                    xr[got] = c + 0.75 * sx; xi[got] = sqrt(0.4375) * sx;
                    xr[got + 1] = c + 0.75 * sx; xi[got + 1] = -sqrt(0.4375) * sx;
                    got += 2;
                }
            } else {
                got = pick_shifts_dev(sh.rr, sh.ri, sh.nritz, ns, xr, xi);
            }
            if (got < 2) {
                const double a = AT(H, ldh, kbot - 1, kbot - 1), b = AT(H, ldh, kbot - 1, kbot);
                const double c = AT(H, ldh, kbot, kbot - 1), d = AT(H, ldh, kbot, kbot);
                double r1, i1, r2, i2;
                eig2x2(a, b, c, d, &r1, &i1, &r2, &i2);
                if (i1 == 0.0) {
                    const double pick = (fabs(r1 - d) < fabs(r2 - d)) ? r1 : r2;
                    r1 = r2 = pick;
                }
                xr[0] = r1; xi[0] = i1; xr[1] = r2; xi[1] = i2;
                got = 2;
            }
            for (int g = 0; g < got / 2; ++g) {
                sh.poly[2 * g] = xr[2 * g] + xr[2 * g + 1];
                sh.poly[2 * g + 1] = xr[2 * g] * xr[2 * g + 1] - xi[2 * g] * xi[2 * g + 1];
            }
            sh.nsh = got;
        }
        __syncthreads();
        // sweep: chains of at most CHASE_MAX_BULGES bulges, one after another
        const int nbulge = uni(sh.nsh) / 2;
        const int wmax = tu.wchase;
        fl += 20.0 * n * (double)nbulge * (kbot - ktop);
        for (int c0 = 0; c0 < nbulge; c0 += CHASE_MAX_BULGES) {
            const int nb = (nbulge - c0 < CHASE_MAX_BULGES) ? nbulge - c0 : CHASE_MAX_BULGES;
            const int tend = kbot - 1 - ktop + 3 * (nb - 1);
            int t = 0;
            while (t <= tend) {
                const int r0 = (ktop + t - 3 * (nb - 1) > ktop) ? ktop + t - 3 * (nb - 1) : ktop;
                const int r1 = (r0 + wmax - 1 < kbot) ? r0 + wmax - 1 : kbot;
                const int t1 = (r1 < kbot) ? r1 - 3 - ktop + 1 : tend + 1;
                const int b0 = (r0 > 0) ? r0 - 1 : 0;
                const int mb = r1 - b0 + 1, w = r1 - r0 + 1;
                b_chase(H, ldh, ktop, kbot, r0, r1, t, t1, nb, c0, refl_span(hnorm));
                b_update(H, ldh, Z, ldz, n, r0, w, b0, r1 + 1, mb * (mb | 1), w | 1);
                t = t1;
            }
        }
    }
    // standardise any decoupled 2x2 block not yet in standard form, then (wr, wi)
    __syncthreads();
    double nflag = 0.0;
    for (int j = tid; j + 1 < n; j += BT) {
        const double c = AT(H, ldh, j + 1, j);
        if (c == 0.0) continue;
        if (j > 0 && AT(H, ldh, j, j - 1) != 0.0) continue;
        if (j + 2 < n && AT(H, ldh, j + 2, j + 1) != 0.0) continue;
        if (!(AT(H, ldh, j, j) == AT(H, ldh, j + 1, j + 1) && AT(H, ldh, j, j + 1) * c < 0.0)) nflag += 1.0;
    }
    nflag = block_reduce<BT>(nflag, false);
    for (int j = 0; nflag > 0.0 && j + 1 < n; ++j) {
        const double c = AT(H, ldh, j + 1, j);
        if (c == 0.0) continue;
        if (j > 0 && AT(H, ldh, j, j - 1) != 0.0) continue;
        if (j + 2 < n && AT(H, ldh, j + 2, j + 1) != 0.0) continue;
        const double a = AT(H, ldh, j, j), b = AT(H, ldh, j, j + 1), d = AT(H, ldh, j + 1, j + 1);
        if (a == d && b * c < 0.0) continue;
        const Std2 o = std2x2(a, b, c, d);
        __syncthreads();
        for (int idx = tid; idx < n; idx += BT) {
            if (idx >= j + 2) {
                const double xx = AT(H, ldh, j, idx), yy = AT(H, ldh, j + 1, idx);
                AT(H, ldh, j, idx) = o.cs * xx + o.sn * yy;
                AT(H, ldh, j + 1, idx) = -o.sn * xx + o.cs * yy;
            }
            if (idx < j) {
                const double xx = AT(H, ldh, idx, j), yy = AT(H, ldh, idx, j + 1);
                AT(H, ldh, idx, j) = o.cs * xx + o.sn * yy;
                AT(H, ldh, idx, j + 1) = -o.sn * xx + o.cs * yy;
            }
            const double xx = AT(Z, ldz, idx, j), yy = AT(Z, ldz, idx, j + 1);
            AT(Z, ldz, idx, j) = o.cs * xx + o.sn * yy;
            AT(Z, ldz, idx, j + 1) = -o.sn * xx + o.cs * yy;
        }
        if (tid == 0) {
            AT(H, ldh, j, j) = o.a; AT(H, ldh, j, j + 1) = o.b;
            AT(H, ldh, j + 1, j) = o.c; AT(H, ldh, j + 1, j + 1) = o.d;
        }
        __syncthreads();
    }
    for (int j = tid; j < n; j += BT) {
        const bool starts = (j + 1 < n) && AT(H, ldh, j + 1, j) != 0.0;
        const bool ends = (j > 0) && AT(H, ldh, j, j - 1) != 0.0;
        if (starts && !ends) {
            P.wr[j] = AT(H, ldh, j, j);
            P.wi[j] = sqrt(fabs(AT(H, ldh, j, j + 1))) * sqrt(fabs(AT(H, ldh, j + 1, j)));
        } else if (ends && !(j >= 2 && AT(H, ldh, j - 1, j - 2) != 0.0)) {
            P.wr[j] = AT(H, ldh, j, j);
            P.wi[j] = -(sqrt(fabs(AT(H, ldh, j - 1, j))) * sqrt(fabs(AT(H, ldh, j, j - 1))));
        } else {
            P.wr[j] = AT(H, ldh, j, j);
            P.wi[j] = 0.0;
        }
    }
    __syncthreads();
    cnt->all = fl;
    return info;
}

extern "C" __global__ void __launch_bounds__(BT) k_batched(BArgs A) {
    __shared__ int s_idx;
    for (;;) {
        int p = 0, b = 0;
        BProb P = A.one;
        if (A.probs) {
            if (threadIdx.x == 0) s_idx = atomicAdd(A.next, 1);
            __syncthreads();
            const int k = s_idx;
            __syncthreads();
            if (k >= A.nprob) break;
            p = A.order[k];
            P = A.probs[p];
            if (P.pad) continue;  // rejected by k_batched_pack (uniform across the workgroup)
            while (b + 1 < B_NBUCKET && P.n > A.bucket_hi[b]) ++b;
        }
        BCount cnt;
        const int info = solve_one(P, A.tune[b], A, &cnt);
        if (!A.probs) {
            cnt.info = info;
            if (threadIdx.x == 0) *A.count = cnt;
            break;
        }
        if (threadIdx.x == 0) {
            A.info[p] = info;
            atomicAdd((double *)(A.next + 2), cnt.all);
        }
        __syncthreads();
    }
}

// Problem descriptors from the caller's device arrays, per-problem argument
// checks (a rejected problem gets its negative code in info and is skipped), the
// largest-first processing order (rank of each problem by descending order, ties
// by index), and the reset of the work counter.  Everything the persistent kernel
// reads is rebuilt here on the device, so a captured launch pair replays
// correctly with whatever the caller's arrays hold at replay time.
extern "C" __global__ void __launch_bounds__(256) k_batched_pack(BProb *out, int *order, int *next, int *info,
                                                                  const int *n, const int *ldh, const int *ldz,
                                                                  double *const *H, double *const *Z,
                                                                  double *const *wr, double *const *wi, int batch) {
    __shared__ int sk[256];
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    const bool mine = b < batch;
    if (b == 0) {
        *next = 0;
        *(double *)(next + 2) = 0.0;  // the launch's flop count
    }
    int key = -1;
    if (mine) {
        BProb p;
        p.H = H[b]; p.Z = Z[b]; p.wr = wr[b]; p.wi = wi[b];
        p.n = n[b]; p.ldh = ldh[b]; p.ldz = ldz[b];
        int code = 0;
        if (p.n < 0) code = -2;
        else if (p.n > 0 && !p.H) code = -3;
        else if (p.ldh < max(1, p.n)) code = -4;
        else if (p.n > 0 && !p.Z) code = -5;
        else if (p.ldz < max(1, p.n)) code = -6;
        else if (p.n > 0 && !p.wr) code = -7;
        else if (p.n > 0 && !p.wi) code = -8;
        p.pad = code;
        out[b] = p;
        if (code) info[b] = code;
        key = max(p.n, -1);  // the key every thread computes for this problem
    }
    // rank = number of problems that come before this one: larger order, or the
    // same order and a smaller index; the sizes pass through LDS 256 at a time
    int rank = 0;
    for (int c0 = 0; c0 < batch; c0 += 256) {
        const int c = c0 + (int)threadIdx.x;
        sk[threadIdx.x] = (c < batch) ? max(n[c], -1) : -2;
        __syncthreads();
        const int lim = min(256, batch - c0);
        for (int u = 0; u < lim; ++u) {
            const int kc = sk[u];
            rank += (kc > key) || (kc == key && c0 + u < b);
        }
        __syncthreads();
    }
    if (mine) order[rank] = b;
}
