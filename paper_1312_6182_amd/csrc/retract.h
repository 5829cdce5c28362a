// Retraction device code shared by the stop kernels and the persistent solve
// kernel: the Jacobi eigensolver, the inverse square root of a Gram matrix and
// the coefficients X_{k+1} = G Omega + X_k Psi of the block forms.
//
// Each function runs on a group of threads: the whole workgroup, or (WAVE) one
// wave of it, whose barriers only order its own LDS operations.  One wave is
// enough up to m = 16: a Jacobi step then has at most 36 blocks of A and 128
// rows of V (kItems = 3 per thread), a product at most 64 register blocks.
#pragma once

#include <hip/hip_runtime.h>

#include "gpspca_internal.h"

namespace gpspca {

constexpr int LDM = kMaxM + 1;  // padded leading dimension of m x m LDS matrices

template <bool WAVE>
__device__ __forceinline__ int group_thread() {
    return WAVE ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
}
template <bool WAVE>
__device__ __forceinline__ int group_size() {
    return WAVE ? 64 : (int)blockDim.x;
}
template <bool WAVE>
__device__ __forceinline__ void group_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}
template <bool WAVE>
__device__ __forceinline__ int group_any(int v) {
    if constexpr (WAVE) {
        group_sync<true>();
        return __any(v);
    } else {
        return __syncthreads_or(v);
    }
}

// ---------------------------------------------------------------------------
// Symmetric eigen-decomposition by the cyclic Jacobi method with a parallel
// (round-robin) ordering: each step applies msz/2 disjoint plane rotations.
// a (msz x msz, leading dim LDM, LDS) is diagonalized in place; v receives the
// eigenvectors (columns).  With `warm`, v already holds an orthogonal V0 and a
// holds V0^T M V0: the rotations continue from there (V <- V0 J ...).
//
// Layout: during a sweep the matrix is kept in slot coordinates.  With mm =
// msz rounded up to even (an odd size gets a zero padding row and column that
// never rotates), step r of the round-robin schedule pairs slot k with slot
// mm - 1 - k, and slot s holds index 0 (s = 0) or 1 + (s - 1 + r) mod (mm - 1).
// Moving to step r + 1 then shifts the contents of every slot s >= 2 to s - 1
// and slot 1 to mm - 1, the same permutation at every step, so each step reads
// its pairs at fixed addresses and writes the rotated entries straight to
// their places for the next step: every thread's LDS offsets are computed once
// for the whole eigensolve.  A sweep is mm - 1 steps, after which the slots
// are back in index order.  Only one entry of each symmetric pair is kept
// during the sweeps (the one whose row slot belongs to the pair of lower
// number, or the upper one within a pair); the other is filled in at the end.
//
// A step: threads k < mm/2 compute the rotation of pair k while every thread
// loads its items (2 x 2 blocks of A over a pair of pairs, upper half only,
// and rows of V over one pair); then each item applies its rotations
// (A <- R A R^T, V <- V R^T) and stores the results at the next step's slots.
//
// A pair is rotated while |a_pq| > 2^-16 sqrt(|a_pp a_qq|) (the relative test,
// which keeps the small eigenvalues of a graded matrix accurate); the inverse
// square root is then built with the first-order correction of the remaining
// off-diagonal (inv_sqrt_from_eig), which leaves an error of second order,
// far below the FP32 of the retracted X.  The rotated pair's off-diagonal entry is
// set to zero exactly, as the rotation makes it: computed, it would keep a
// rounding residue of about 2^-52 max(a_pp, a_qq), which the relative test
// would chase without end when a_pp / a_qq is large.
// a and v need mm rows.  Executed by the whole workgroup.

// Items per thread of a Jacobi step; the kernels that call jacobi_eig launch
// at least jacobi_threads(m) threads.
constexpr int kItems = 3;

// Threads for an m x m Jacobi step: m > 32: 1024 (at most 32 x 33 / 2 blocks
// of A + 64 x 32 rows of V = 2576 items); m > 16: 512 (at most 648); m > 8: 256
// (at most 164); else one wave (at most 42 items and 16 entries of a product,
// and a barrier of a single wave costs almost nothing).
inline int jacobi_threads(int m) { return m > 32 ? 1024 : m > 16 ? 512 : m > 8 ? 256 : 64; }

__device__ __forceinline__ int jac_pidx(int s, int mm) { return s < mm / 2 ? s : mm - 1 - s; }

// slot that receives slot s's contents at the next step
__device__ __forceinline__ int jac_next(int s, int mm) {
    return s == 0 ? 0 : (s == 1 ? mm - 1 : s - 1);
}

// offset of the kept entry of the symmetric pair (u, w)
__device__ __forceinline__ int jac_kept(int u, int w, int mm) {
    const int pu = jac_pidx(u, mm), pw = jac_pidx(w, mm);
    const bool swap = pu > pw || (pu == pw && u > w);
    return swap ? w * LDM + u : u * LDM + w;
}

template <bool WAVE = false>
__device__ void jacobi_eig(double* a, double* v, int msz, double* rot, bool warm = false) {
    const int t = group_thread<WAVE>(), nt = group_size<WAVE>();
    // |a_pq| > 2^-16 sqrt(|a_pp a_qq|), tested squared (no square root)
    constexpr double kTol2 = 2.3283064365386963e-10;  // 2^-32
    if (!warm) {
        for (int e = t; e < msz * msz; e += nt) {
            const int i = e / msz, j = e % msz;
            v[i * LDM + j] = (i == j) ? 1.0 : 0.0;
        }
    }
    if (msz < 2) {
        group_sync<WAVE>();
        return;
    }
    const int mm = msz + (msz & 1), half = mm / 2;
    if (msz & 1) {
        for (int e = t; e < mm; e += nt) {
            a[msz * LDM + e] = 0.0;
            a[e * LDM + msz] = 0.0;
        }
        for (int e = t; e < msz; e += nt) v[e * LDM + msz] = 0.0;
    }
    // items: upper blocks (k1 <= k2) of A, then rows of V; thread t owns
    // items t, t + nt, ... (at most kItems: blockDim.x is chosen for that)
    const int nA = half * (half + 1) / 2, nitem = nA + msz * half;
    int kind[kItems];     // 0 none, 1 block of A, 2 diagonal block of A, 3 row of V
    int rk1[kItems], rk2[kItems];
    int ld[kItems][4], sto[kItems][4];
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
        const int e = t + u * nt;
        kind[u] = 0;
        rk1[u] = rk2[u] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) ld[u][q] = sto[u][q] = 0;
        if (e >= nitem) continue;
        if (e < nA) {
            int k1 = 0, rem = e;
            while (rem >= half - k1) {
                rem -= half - k1;
                ++k1;
            }
            const int k2 = k1 + rem;
            const int P1 = k1, Q1 = mm - 1 - k1, P2 = k2, Q2 = mm - 1 - k2;
            const int nP1 = jac_next(P1, mm), nQ1 = jac_next(Q1, mm);
            const int nP2 = jac_next(P2, mm), nQ2 = jac_next(Q2, mm);
            rk1[u] = k1;
            rk2[u] = k2;
            if (k1 < k2) {
                kind[u] = 1;
                ld[u][0] = P1 * LDM + P2;
                ld[u][1] = P1 * LDM + Q2;
                ld[u][2] = Q1 * LDM + P2;
                ld[u][3] = Q1 * LDM + Q2;
                sto[u][0] = jac_kept(nP1, nP2, mm);
                sto[u][1] = jac_kept(nP1, nQ2, mm);
                sto[u][2] = jac_kept(nQ1, nP2, mm);
                sto[u][3] = jac_kept(nQ1, nQ2, mm);
            } else {
                kind[u] = 2;
                ld[u][0] = P1 * LDM + P1;
                ld[u][1] = P1 * LDM + Q1;
                ld[u][3] = Q1 * LDM + Q1;
                sto[u][0] = jac_kept(nP1, nP1, mm);
                sto[u][1] = jac_kept(nP1, nQ1, mm);
                sto[u][3] = jac_kept(nQ1, nQ1, mm);
            }
        } else {
            const int f = e - nA, row = f % msz, k = f / msz;
            const int P = k, Q = mm - 1 - k;
            kind[u] = 3;
            rk1[u] = k;
            ld[u][0] = row * LDM + P;
            ld[u][1] = row * LDM + Q;
            sto[u][0] = row * LDM + jac_next(P, mm);
            sto[u][1] = row * LDM + jac_next(Q, mm);
        }
    }
    group_sync<WAVE>();
    for (int sweep = 0; sweep < 40; ++sweep) {
        // a sweep that would apply no rotation ends the iteration.  Every pair
        // is tested at once before the sweep (the slots are in index order
        // here): if none qualifies, no step of the sweep would rotate.
        int need = 0;
        for (int e = t; e < msz * msz; e += nt) {
            const int i = e / msz, j = e % msz;
            if (i != j && jac_kept(i, j, mm) == i * LDM + j) {
                const double apq = a[i * LDM + j];
                need |= (apq * apq > kTol2 * fabs(a[i * LDM + i] * a[j * LDM + j]) &&
                         fabs(apq) > 1e-300) ? 1 : 0;
            }
        }
        if (!group_any<WAVE>(need)) break;
        for (int r = 0; r < mm - 1; ++r) {
            // phase 1: the rotations of this step, and every item's loads
            if (t < half) {
                const int P = t, Q = mm - 1 - t;
                const double apq = a[P * LDM + Q];
                const double app = a[P * LDM + P], aqq = a[Q * LDM + Q];
                double c = 1.0, sn = 0.0;
                if (apq * apq > kTol2 * fabs(app * aqq) && fabs(apq) > 1e-300) {
                    const double tau = (aqq - app) / (2.0 * apq);
                    const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                    c = rsqrt(1.0 + tt * tt);
                    sn = tt * c;
                }
                rot[2 * t] = c;
                rot[2 * t + 1] = sn;
            }
            double x[kItems][4];
#pragma unroll
            for (int u = 0; u < kItems; ++u) {
                x[u][0] = x[u][1] = x[u][2] = x[u][3] = 0.0;
                if (kind[u] == 1) {
                    x[u][0] = a[ld[u][0]];
                    x[u][1] = a[ld[u][1]];
                    x[u][2] = a[ld[u][2]];
                    x[u][3] = a[ld[u][3]];
                } else if (kind[u] == 2) {
                    x[u][0] = a[ld[u][0]];
                    x[u][1] = a[ld[u][1]];
                    x[u][3] = a[ld[u][3]];
                } else if (kind[u] == 3) {
                    x[u][0] = v[ld[u][0]];
                    x[u][1] = v[ld[u][1]];
                }
            }
            group_sync<WAVE>();
            // phase 2: rotate and store at the next step's slots
#pragma unroll
            for (int u = 0; u < kItems; ++u) {
                if (kind[u] == 0) continue;
                const double c1 = rot[2 * rk1[u]], s1 = rot[2 * rk1[u] + 1];
                if (kind[u] == 3) {
                    const double vp = x[u][0], vq = x[u][1];
                    v[sto[u][0]] = c1 * vp - s1 * vq;
                    v[sto[u][1]] = s1 * vp + c1 * vq;
                    continue;
                }
                const double c2 = rot[2 * rk2[u]], s2 = rot[2 * rk2[u] + 1];
                const double x00 = x[u][0], x01 = x[u][1], x11 = x[u][3];
                const double x10 = (kind[u] == 2) ? x01 : x[u][2];
                // rows
                const double r00 = c1 * x00 - s1 * x10, r01 = c1 * x01 - s1 * x11;
                const double r10 = s1 * x00 + c1 * x10, r11 = s1 * x01 + c1 * x11;
                // columns
                a[sto[u][0]] = c2 * r00 - s2 * r01;
                if (kind[u] == 1) {
                    a[sto[u][1]] = s2 * r00 + c2 * r01;
                    a[sto[u][2]] = c2 * r10 - s2 * r11;
                } else {
                    // the rotated pair's off-diagonal is zero by construction
                    a[sto[u][1]] = (s1 != 0.0) ? 0.0 : x01;
                }
                a[sto[u][3]] = s2 * r10 + c2 * r11;
            }
            group_sync<WAVE>();
        }
    }
    // fill in the other entry of every symmetric pair
    for (int e = t; e < msz * msz; e += nt) {
        const int i = e / msz, j = e % msz;
        const int kp = jac_kept(i, j, mm);
        if (kp != i * LDM + j) a[i * LDM + j] = a[kp];
    }
    group_sync<WAVE>();
}

// C = op(A) op(B) for n x n matrices in LDS (leading dim LDM), op(X) = X or
// X^T.  With h = ceil(n/2), thread t = ii h + jj computes the four entries
// (ii | ii + h) x (jj | jj + h) of C in registers, summing over k in order
// (h^2 <= blockDim.x: jacobi_threads): the lanes of a wave then read
// consecutive entries of B (and share those of A), free of LDS bank
// conflicts.  C is written after a barrier, so it may be A or B.  Executed by
// the whole workgroup.
template <bool TA, bool TB, bool WAVE = false>
__device__ void lds_gemm(int n, const double* A, const double* B, double* C) {
    const int t = group_thread<WAVE>(), h = (n + 1) / 2;
    const bool mine = t < h * h;
    const int ii = mine ? t / h : 0, jj = mine ? t % h : 0;
    const int i1 = ii + h < n ? ii + h : ii, j1 = jj + h < n ? jj + h : jj;
    double c00 = 0.0, c01 = 0.0, c10 = 0.0, c11 = 0.0;
    if (mine) {
        for (int k = 0; k < n; ++k) {
            const double a0 = TA ? A[k * LDM + ii] : A[ii * LDM + k];
            const double a1 = TA ? A[k * LDM + i1] : A[i1 * LDM + k];
            const double b0 = TB ? B[jj * LDM + k] : B[k * LDM + jj];
            const double b1 = TB ? B[j1 * LDM + k] : B[k * LDM + j1];
            c00 += a0 * b0;
            c01 += a0 * b1;
            c10 += a1 * b0;
            c11 += a1 * b1;
        }
    }
    group_sync<WAVE>();
    if (mine) {
        C[ii * LDM + jj] = c00;
        if (jj + h < n) C[ii * LDM + jj + h] = c01;
        if (ii + h < n) C[(ii + h) * LDM + jj] = c10;
        if (ii + h < n && jj + h < n) C[(ii + h) * LDM + jj + h] = c11;
    }
    group_sync<WAVE>();
}

// out = V Y V^T ~ (V a V^T)^{-1/2} from the Jacobi result: a = V^T M V is
// diagonal up to off-diagonal entries below the stopping tolerance.  Y is the
// inverse square root of a to first order in its off-diagonal (the
// Daleckii-Krein formula): Y_ii = a_ii^{-1/2}, and for i != j
//   Y_ij = f[a_ii, a_jj] a_ij,  f[x, y] = (x^{-1/2} - y^{-1/2}) / (x - y)
//        = -1 / (sqrt(x) sqrt(y) (sqrt(x) + sqrt(y))),
// a divided difference that stays finite for equal diagonal entries.  The
// error left is second order in the relative off-diagonal e (measured below
// 250 e^2 on the retracted X: 6e-8 at e = 2^-16, the FP32 rounding of X), so
// the sweeps stop there.
// Eigenvalues below (msz * eps)^2 * lam_max count as zero (their row and
// column of Y are dropped) and set *rankdef.  a is overwritten.
template <bool WAVE = false>
__device__ void inv_sqrt_from_eig(double* a, const double* v, double* out, int msz,
                                  double* lam, int* rankdef) {
    const int t = group_thread<WAVE>(), nt = group_size<WAVE>();
    const int ne = msz * msz;
    // every thread finds the largest eigenvalue; thread i inverts the root of
    // eigenvalue i
    double lmax = 0.0;
    for (int i = 0; i < msz; ++i) lmax = fmax(lmax, a[i * LDM + i]);
    const double thr = lmax * ((double)msz * 2.220446049250313e-16) * ((double)msz * 2.220446049250313e-16);
    int rd = !(lmax > 0.0);
    for (int i = t; i < msz; i += nt) {
        const double l = a[i * LDM + i];
        if (l > thr && l > 0.0) lam[i] = 1.0 / sqrt(l);
        else { lam[i] = 0.0; rd = 1; }
    }
    rd = group_any<WAVE>(rd);
    if (t == 0) *rankdef = rd;
    // Y in place of a: with l_i = a_ii^{-1/2}, f[a_ii, a_jj] = -(l_i l_j)^2 / (l_i + l_j)
    for (int e = t; e < ne; e += nt) {
        const int i = e / msz, j = e % msz;
        const double li = lam[i], lj = lam[j];
        double y;
        if (i == j) y = li;
        else if (li == 0.0 || lj == 0.0) y = 0.0;
        else y = -a[i * LDM + j] * (li * lj) * (li * lj) / (li + lj);
        a[i * LDM + j] = y;
    }
    group_sync<WAVE>();
    // T = V Y over Y, then out = T V^T
    lds_gemm<false, false, WAVE>(msz, v, a, a);
    lds_gemm<false, true, WAVE>(msz, a, v, out);
}

// Sum over the 64 lanes of a wave by a fixed butterfly (every lane gets it).
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sums over the 64 lanes of a wave by row shifts and broadcasts in the vector
// ALU (a cross-lane read through LDS has ten times the latency, and the small
// phases of a pass are chains of them); every lane gets lane 63's total.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xF, true);
    return v + __longlong_as_double(((uint64_t)hi << 32) | lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, true);
}
template <typename T>
__device__ __forceinline__ T dpp_scan63(T v) {
    v = dpp_add<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8: lane 15 of each row
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ double wave_sum_s(double v) {
    const uint64_t u = __double_as_longlong(dpp_scan63(v));
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, 63);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(u >> 32), 63);
    return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int wave_sum_s(int v) {
    return __builtin_amdgcn_readlane(dpp_scan63(v), 63);
}

// W = M^{-1/2} of the m x m (m <= 8) symmetric positive definite M (LDS, leading
// dim m) by one wave, lane (i, j) holding entry (i, j): the coupled
// Newton-Schulz iteration Y <- Y T, Z <- T Z, T = (3 I - Z Y) / 2, from Y = M / c,
// Z = I with c = ||M||_F / 2 (so the eigenvalues of Y lie in (0, 2]).  Z -> c^{1/2}
// M^{-1/2} quadratically once Z Y is near I, with an error of about
// cond(M) eps.  A well-conditioned M, which is what the polar factor of a pass
// has, takes 6 to 10 iterations of two LDS round trips each, where the Jacobi
// sweeps are chains of FP64 divisions and roots: 3 against 13 us per pass at
// m = 5 in k_small.  False when 20 iterations are not enough (cond(M) beyond
// about 10^5, or not positive definite): the caller then runs the Jacobi
// eigensolve.
__device__ inline bool newton_inv_sqrt(int m, const double* M, double* W, double* buf) {
    const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
    double* const Yb = buf;            // 8 x 8 each, leading dim 10
    double* const Zb = buf + 80;
    double* const Tb = buf + 160;
    const bool in = i < m && j < m;
    const double mij = in ? M[i * m + j] : 0.0;
    const double f2 = wave_sum_s(mij * mij);
    const double c = 0.5 * sqrt(f2);
    if (!(c > 0.0) || !isfinite(c)) return false;
    const double id = i == j ? 1.0 : 0.0;
    double y = in ? mij / c : id, z = id;
    auto row_dot = [&](const double* A, const double* B) {   // both symmetric
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int k = 0; k < 8; k += 2) {
            s0 = __builtin_fma(A[i * 10 + k], B[j * 10 + k], s0);
            s1 = __builtin_fma(A[i * 10 + k + 1], B[j * 10 + k + 1], s1);
        }
        return s0 + s1;
    };
    bool last = false;
    for (int it = 0; it < 20; ++it) {
        Yb[i * 10 + j] = y;
        Zb[i * 10 + j] = z;
        group_sync<true>();
        const double r = row_dot(Zb, Yb);
        const double e = fabs(id - r);
        if (__any(!(e < 1e100))) return false;
        last = !__any(e > 1e-8);       // the update below squares it
        Tb[i * 10 + j] = 1.5 * id - 0.5 * r;
        group_sync<true>();
        const double yn = row_dot(Yb, Tb);
        z = row_dot(Tb, Zb);
        y = yn;
        group_sync<true>();
        if (last) break;
    }
    if (!last) return false;
    Zb[i * 10 + j] = z;
    group_sync<true>();
    if (in) W[i * m + j] = 0.5 * (z + Zb[j * 10 + i]) / sqrt(c);
    group_sync<true>();
    return true;
}

// The same for 9 <= m <= 64 by the whole workgroup (at least one wave per 16 x 16
// tile: 64 ceil(m / 16)^2 threads): a wave keeps its tile of Y, Z and T in the
// accumulator layout of v_mfma_f64_16x16x4_f64 (lane l, entry v: row 4 v + l / 16,
// column l % 16), and the products read rows of both operands from LDS (they are
// symmetric; leading dim 66 keeps the reads free of bank conflicts).  buf: three
// matrices of 16 ceil(m / 16) rows.  The Jacobi sweeps at m = 64 are 63 dependent
// steps each: with this iteration the stop kernel of a BL1 pass at m = 64 takes 68
// instead of 175 us and the projection of a start 60 instead of 577 (m = 16: 12 and
// 10 instead of 17 and 60; m = 8, by the one-wave form: 8.5 and 5 instead of 19
// and 24).
constexpr int kNewtonLd = 66;
constexpr int kNewtonIter = 24;   // cond(M) up to about 10^7
__device__ inline bool newton_inv_sqrt_mfma(int m, const double* M, double* W, double* buf,
                                            double* red) {
    typedef double d4 __attribute__((ext_vector_type(4)));
    constexpr int LD = kNewtonLd;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nt = (m + 15) / 16, mp = 16 * nt;
    double* const Yb = buf;
    double* const Zb = buf + mp * LD;
    double* const Tb = buf + 2 * mp * LD;
    const bool mine = wv < nt * nt;
    const int ti = mine ? wv / nt : 0, tj = mine ? wv % nt : 0;
    const int i0 = 16 * ti + (lane >> 4), j = 16 * tj + (lane & 15);   // rows i0 + 4 v
    double y[4], z[4], id[4];
    double f2 = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = i0 + 4 * v;
        const bool in = mine && i < m && j < m;
        y[v] = in ? M[i * m + j] : 0.0;
        id[v] = i == j ? 1.0 : 0.0;
        z[v] = id[v];
        f2 += y[v] * y[v];
    }
    f2 = wave_sum_s(f2);
    if (lane == 0) red[wv] = mine ? f2 : 0.0;
    __syncthreads();
    double tot = 0.0;
    for (int w = 0; w < nt * nt; ++w) tot += red[w];
    const double c = 0.5 * sqrt(tot);
    if (!(c > 0.0) || !isfinite(c)) return false;   // the same in every thread
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = i0 + 4 * v;
        y[v] = i < m && j < m ? y[v] / c : id[v];
    }
    auto store = [&](double* B, const double (&x)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) B[(i0 + 4 * v) * LD + j] = x[v];
    };
    // tile (ti, tj) of A B for symmetric A and B
    auto prod = [&](const double* A, const double* B) {
        d4 s = d4{0.0, 0.0, 0.0, 0.0};
        const double* ar = A + (16 * ti + (lane & 15)) * LD + (lane >> 4);
        const double* br = B + (16 * tj + (lane & 15)) * LD + (lane >> 4);
        for (int k = 0; k < mp; k += 4)
            s = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[k], br[k], s, 0, 0, 0);
        return s;
    };
    bool last = false;
    for (int it = 0; it < kNewtonIter; ++it) {
        if (mine) {
            store(Yb, y);
            store(Zb, z);
        }
        __syncthreads();
        int bad = 0, more = 0;
        if (mine) {
            const d4 r = prod(Zb, Yb);
            double tv[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double e = fabs(id[v] - r[v]);
                bad |= !(e < 1e100);
                more |= e > 1e-8;      // the update below squares it
                tv[v] = 1.5 * id[v] - 0.5 * r[v];
            }
            store(Tb, tv);
        }
        if (__syncthreads_or(bad)) return false;
        last = !__syncthreads_or(more);
        if (mine) {
            const d4 yn = prod(Yb, Tb), zn = prod(Tb, Zb);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                y[v] = yn[v];
                z[v] = zn[v];
            }
        }
        __syncthreads();
        if (last) break;
    }
    if (!last) return false;
    if (mine) store(Zb, z);
    __syncthreads();
    if (mine) {
        const double sc = 0.5 / sqrt(c);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + 4 * v;
            if (i < m && j < m) W[i * m + j] = sc * (z[v] + Zb[j * LD + i]);
        }
    }
    __syncthreads();
    return true;
}

// LDS of the retraction of m components (bytes): three matrices for the Jacobi
// eigensolve (rows rounded up to even) or the Newton iteration.
__host__ __device__ inline int retract_lds(int m) {
    const int jac = 3 * (m + (m & 1)) * LDM * 8;
    const int nwt = m > 8 ? 3 * 16 * ((m + 15) / 16) * kNewtonLd * 8 : 240 * 8;
    return jac > nwt ? jac : nwt;
}

// M^{-1/2} of a well-conditioned M by the Newton iteration of its size.
template <bool WAVE>
__device__ __forceinline__ bool newton_root(int m, const double* M, double* W, double* buf,
                                            double* red) {
    if constexpr (WAVE) {
        return m <= 8 && newton_inv_sqrt(m, M, W, buf);
    } else {
        if (m > 8) return newton_inv_sqrt_mfma(m, M, W, buf, red);
        return blockDim.x == 64 && newton_inv_sqrt(m, M, W, buf);
    }
}

struct StopShared {
    double rot[kMaxM];
    double lam[kMaxM];
    double fj[kMaxM];
    int nj[kMaxM];
    int live[kMaxM];
    int dead[kMaxM];
    double dsc[kMaxM];  // original-form block L1: 1/||s_j|| (0 for a dead component)
    double fterm[kMaxM];  // component j's term of F
    int nlive, ndead, rankdef, stop;
};

// Retraction coefficients for the block forms with live set L and dead set D.
template <bool WAVE = false>
__device__ void block_coefficients(int m, double* coef, double* vprev, StopShared& ss,
                                   double* A0, double* A1, double* A2, Ctrl* ctrl) {
    const int t = group_thread<WAVE>(), nt = group_size<WAVE>(), mm = m * m;
    const double* GtG = coef + 2 * mm;
    const double* GtX = coef + 3 * mm;
    const double* XtX = coef + 4 * mm;
    double* Om = coef;
    double* Ps = coef + mm;
    const int nl = ss.nlive, nd = ss.ndead;
    // every component live and G^T G well conditioned: Omega = (G^T G)^{-1/2}
    // (a solve in which the iteration once did not converge stays with Jacobi)
    if (nd == 0 && !ctrl->no_newton) {
        if (newton_root<WAVE>(m, GtG, Om, A0, ss.lam)) {
            for (int e = t; e < mm; e += nt) Ps[e] = 0.0;
            if (t == 0) ctrl->ndead = 0;
            group_sync<WAVE>();
            return;
        }
        group_sync<WAVE>();
        if (t == 0) ctrl->no_newton = 1;
    }
    for (int e = t; e < 2 * mm; e += nt) coef[e] = 0.0;
    // W_L = (G_L^T G_L)^{-1/2}
    const bool warm = (nd == 0) && ctrl->warm;
    for (int e = t; e < nl * nl; e += nt) {
        const int i = e / nl, j = e % nl;
        A0[i * LDM + j] = GtG[ss.live[i] * m + ss.live[j]];
        if (warm) A1[i * LDM + j] = vprev[i * m + j];
    }
    group_sync<WAVE>();
    if (warm) {
        // A0 <- V0^T M V0 with the previous pass's eigenvectors V0: the Gram matrix
        // changes little between passes, so this is nearly diagonal already
        lds_gemm<false, false, WAVE>(nl, A0, A1, A2);
        lds_gemm<true, false, WAVE>(nl, A1, A2, A0);
    }
    jacobi_eig<WAVE>(A0, A1, nl, ss.rot, warm);

    if (nd == 0) {
        for (int e = t; e < nl * nl; e += nt) {
            const int i = e / nl, j = e % nl;
            vprev[i * m + j] = A1[i * LDM + j];
        }
    }
    int rd1 = 0;
    inv_sqrt_from_eig<WAVE>(A0, A1, A2, nl, ss.lam, &ss.rankdef);

    rd1 = ss.rankdef;
    group_sync<WAVE>();
    // Omega[L,L] = W_L
    for (int e = t; e < nl * nl; e += nt) {
        const int i = e / nl, j = e % nl;
        Om[ss.live[i] * m + ss.live[j]] = A2[i * LDM + j];
    }
    if (nd > 0) {
        // C = W_L^T (G^T X)[L, D]   (nl x nd) -> A0
        group_sync<WAVE>();
        for (int e = t; e < nl * nd; e += nt) {
            const int a = e / nd, d = e % nd;
            double s = 0.0;
            for (int l = 0; l < nl; ++l) s += A2[l * LDM + a] * GtX[ss.live[l] * m + ss.dead[d]];
            A0[a * LDM + d] = s;
        }
        group_sync<WAVE>();
        // H^T H = (X^T X)[D,D] - C^T C -> A1
        for (int e = t; e < nd * nd; e += nt) {
            const int d1 = e / nd, d2 = e % nd;
            double s = XtX[ss.dead[d1] * m + ss.dead[d2]];
            for (int a = 0; a < nl; ++a) s -= A0[a * LDM + d1] * A0[a * LDM + d2];
            A1[d1 * LDM + d2] = s;
        }
        group_sync<WAVE>();
        // W_L C  (nl x nd) -> keep in Om scratch rows?  compute into A0 in place:
        // B = W_L C; needs W_L (A2) and C (A0): write B into Ps temporarily.
        for (int e = t; e < nl * nd; e += nt) {
            const int a = e / nd, d = e % nd;
            double s = 0.0;
            for (int l = 0; l < nl; ++l) s += A2[a * LDM + l] * A0[l * LDM + d];
            Ps[a * m + d] = s;  // temporary (nl x nd, leading dim m)
        }
        group_sync<WAVE>();
        // W_D = (H^T H)^{-1/2}: eig of A1 into (A1, A0), inverse root into A2
        for (int e = t; e < nd * nd; e += nt) {
            const int i = e / nd, j = e % nd;
            A0[i * LDM + j] = A1[i * LDM + j];
        }
        group_sync<WAVE>();
        jacobi_eig<WAVE>(A0, A1, nd, ss.rot);
        inv_sqrt_from_eig<WAVE>(A0, A1, A2, nd, ss.lam, &ss.rankdef);
        // Omega[L,D] = -(W_L C) W_D ; Psi[D,D] = W_D
        double* tmp = A0;  // nl x nd product
        for (int e = t; e < nl * nd; e += nt) {
            const int a = e / nd, d = e % nd;
            double s = 0.0;
            for (int k = 0; k < nd; ++k) s += Ps[a * m + k] * A2[k * LDM + d];
            tmp[a * LDM + d] = -s;
        }
        group_sync<WAVE>();
        for (int e = t; e < mm; e += nt) Ps[e] = 0.0;
        group_sync<WAVE>();
        for (int e = t; e < nl * nd; e += nt) {
            const int a = e / nd, d = e % nd;
            Om[ss.live[a] * m + ss.dead[d]] = tmp[a * LDM + d];
        }
        for (int e = t; e < nd * nd; e += nt) {
            const int i = e / nd, j = e % nd;
            Ps[ss.dead[i] * m + ss.dead[j]] = A2[i * LDM + j];
        }
        group_sync<WAVE>();
    }
    if (t == 0) {
        ctrl->ndead = nd;
        ctrl->warm = (nd == 0) ? 1 : 0;
        if (nd > 0 || rd1 || ss.rankdef) ctrl->degenerate_seen = 1;
    }
    group_sync<WAVE>();
}

}  // namespace gpspca
