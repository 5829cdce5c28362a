// Default start and output kernels of the GP-SPCA power iteration.
//
// Default start: the m columns of largest norm, ordered by (-||a_i||, i), so
// ties go to the lower index; their polar factor (or normalization) is the
// starting point.  Selection is two-level: each workgroup keeps the sorted top m
// of its column range, one workgroup merges the sorted lists.
//
// Outputs: Z = S with unit-norm columns (a column with empty support stays
// zero), the support as packed bit words, and X copied out of the internal
// padded buffer.
#include <cfloat>

#include "gpspca_internal.h"
#include "storage.h"

namespace gpspca {

__device__ __forceinline__ bool better(double va, int64_t ia, double vb, int64_t ib) {
    if (ib < 0) return ia >= 0;
    if (ia < 0) return false;
    return va > vb || (va == vb && ia < ib);
}

__device__ __forceinline__ void wave_best(double& v, int64_t& i) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(v, o, 64);
        const int64_t oi = __shfl_xor(i, o, 64);
        if (better(ov, oi, v, i)) {
            v = ov;
            i = oi;
        }
    }
}

// m rounds of a workgroup argmax over norms [b, e), read anew in each.  The order
// "larger value, then lower index" is strict and total, so round r's winner
// is the best pair that comes after round r-1's winner in it: one comparison
// per pair and round, and any reduction order finds the same (unique) pair.
// Results in chosen_v / chosen_i (index -1 once the pairs run out).
__device__ void topm_block(int m, int64_t b, int64_t e, const double* __restrict__ val,
                           double* chosen_v, int64_t* chosen_i, double* rv, int64_t* ri) {
    const int t = threadIdx.x, nt = blockDim.x, lane = t & 63, wv = t >> 6, nw = (nt + 63) >> 6;
    double lv = INFINITY;   // the previous round's winner (none yet: every pair qualifies)
    int64_t li = -1;
    for (int r = 0; r < m; ++r) {
        double bv = -INFINITY;
        int64_t bi = -1;
        for (int64_t i = b + t; i < e; i += nt) {
            const double cv = fmax(val[i], -DBL_MAX);
            // after the previous winner in the order, and better than the best so far
            const bool after = (r == 0) || better(lv, li, cv, i);
            if (after && better(cv, i, bv, bi)) {
                bv = cv;
                bi = i;
            }
        }
        wave_best(bv, bi);
        if (lane == 0) {
            rv[wv] = bv;
            ri[wv] = bi;
        }
        __syncthreads();
        bv = rv[0];
        bi = ri[0];
        for (int w = 1; w < nw; ++w)
            if (better(rv[w], ri[w], bv, bi)) {
                bv = rv[w];
                bi = ri[w];
            }
        if (t == 0) {
            chosen_v[r] = bv;
            chosen_i[r] = bi;
        }
        lv = bv;
        li = bi;
        __syncthreads();
        if (bi < 0) {
            // pairs exhausted: the remaining rounds choose nothing
            for (int q = r + 1 + t; q < m; q += nt) {
                chosen_v[q] = -INFINITY;
                chosen_i[q] = -1;
            }
            __syncthreads();
            return;
        }
    }
}

// Largest value of the 64 lanes, by row shifts and broadcasts in the vector ALU.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
    const uint64_t u = __double_as_longlong(v);
    const int ulo = (int)(uint32_t)u, uhi = (int)(u >> 32);
    const uint32_t lo = __builtin_amdgcn_update_dpp(ulo, ulo, CTRL, ROWS, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(uhi, uhi, CTRL, ROWS, 0xF, false);
    return fmax(v, __longlong_as_double(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_max(double v) {
    v = dpp_max<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8: lane 15 of each row
    v = dpp_max<0x112, 0xF>(v);
    v = dpp_max<0x114, 0xF>(v);
    v = dpp_max<0x118, 0xF>(v);
    v = dpp_max<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_max<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, 63);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(u >> 32), 63);
    return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// Top m of the m-entry lists lv[list * m + r], list < nl <= 64 LPL, each sorted
// (-inf past its end) and of lower indices than the next list, by one wave: lane
// l keeps the heads of lists l LPL .. l LPL + LPL - 1, and each round takes the
// largest head, of the lowest list among equals.  pos[r] receives its place in
// lv, -1 once the lists run out.  A round is one maximum over the lanes and one
// LDS read, no barrier.
template <int LPL>
__device__ void merge_lists(int nl, int m, const double* lv, int* pos) {
    const int lane = threadIdx.x & 63;
    double h[LPL];
    int q[LPL];
#pragma unroll
    for (int u = 0; u < LPL; ++u) {
        const int l = lane * LPL + u;
        q[u] = 0;
        h[u] = l < nl ? lv[l * m] : -INFINITY;
    }
    for (int r = 0; r < m; ++r) {
        double b = h[0];
        int bu = 0;
#pragma unroll
        for (int u = 1; u < LPL; ++u)
            if (h[u] > b) {
                b = h[u];
                bu = u;
            }
        const double top = wave_max(b);
        if (top == -INFINITY) {
            for (int k = r + lane; k < m; k += 64) pos[k] = -1;
            return;
        }
        const uint64_t eq = __ballot(b == top);
        if (lane == __ffsll((unsigned long long)eq) - 1) {
            const int l = lane * LPL + bu;
#pragma unroll
            for (int u = 0; u < LPL; ++u)
                if (u == bu) {
                    pos[r] = l * m + q[u];
                    ++q[u];
                    h[u] = q[u] < m ? lv[l * m + q[u]] : -INFINITY;
                }
        }
    }
}

constexpr int kTopLane = 8;                    // norms per lane
constexpr int64_t kTopRange = 256 * kTopLane;  // norms per workgroup

// Top m of norms[b, e), sorted; at most kTopRange of them: each wave takes a
// quarter, each lane consecutive norms of it in registers, and a round takes
// the largest of the lanes' largest (the lowest lane, the first norm among
// equals, so the lowest index).  The four waves run without barriers and wave 0
// merges their lists.  The rounds are a serial chain, here of about 200 cycles
// each; as reductions over the workgroup of (norm, index) pairs by cross-lane
// reads through LDS with two barriers a round, they took 33 instead of 12 us (both
// kernels 88 and 20) at n = 20011, m = 16 and 128 and 41 (420 and 67) at n = 100000,
// m = 64.  A norm that is not a number counts as the lowest.  Longer ranges (n > 524288) are re-read every round.
__global__ __launch_bounds__(256) void k_topm_local(int64_t n, int m, const double* __restrict__ norms,
                                                    double* __restrict__ cv, int64_t* __restrict__ ci) {
    const int64_t b = n * blockIdx.x / gridDim.x, e = n * (blockIdx.x + 1) / gridDim.x;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (e - b > kTopRange) {
        __shared__ double rv[256];
        __shared__ int64_t ri[256];
        __shared__ double chv[kMaxM];
        __shared__ int64_t chi[kMaxM];
        topm_block(m, b, e, norms, chv, chi, rv, ri);
        for (int r = t; r < m; r += blockDim.x) {
            cv[(size_t)blockIdx.x * m + r] = chv[r];
            ci[(size_t)blockIdx.x * m + r] = chi[r];
        }
        return;
    }
    __shared__ double lv[4 * kMaxM];
    __shared__ int64_t li[4 * kMaxM];
    __shared__ int pos[kMaxM];
    const int64_t len = e - b;
    const int64_t wb = b + len * wv / 4, we = b + len * (wv + 1) / 4;
    const int per = (int)((we - wb + 63) / 64);          // <= kTopLane
    const int64_t lb = wb + (int64_t)lane * per;
    double v[kTopLane];
#pragma unroll
    for (int u = 0; u < kTopLane; ++u)
        v[u] = (u < per && lb + u < we) ? fmax(norms[lb + u], -DBL_MAX) : -INFINITY;
    for (int r = 0; r < m; ++r) {
        double best = v[0];
        int bu = 0;
#pragma unroll
        for (int u = 1; u < kTopLane; ++u)
            if (v[u] > best) {
                best = v[u];
                bu = u;
            }
        const double top = wave_max(best);
        if (top == -INFINITY) {
            for (int k = r + lane; k < m; k += 64) lv[wv * m + k] = -INFINITY;
            break;
        }
        const uint64_t eq = __ballot(best == top);
        if (lane == __ffsll((unsigned long long)eq) - 1) {
            lv[wv * m + r] = best;
            li[wv * m + r] = lb + bu;
#pragma unroll
            for (int u = 0; u < kTopLane; ++u)
                if (u == bu) v[u] = -INFINITY;
        }
    }
    __syncthreads();
    if (wv == 0) merge_lists<1>(4, m, lv, pos);
    __syncthreads();
    for (int r = t; r < m; r += blockDim.x) {
        const int k = pos[r];
        cv[(size_t)blockIdx.x * m + r] = k < 0 ? -INFINITY : lv[k];
        ci[(size_t)blockIdx.x * m + r] = k < 0 ? -1 : li[k];
    }
}

// The lists of at most 256 workgroups, staged in LDS by 1024 threads.
__global__ __launch_bounds__(1024) void k_topm_final(int nl, int m, const double* __restrict__ cv,
                                                     const int64_t* __restrict__ ci,
                                                     int64_t* __restrict__ idx) {
    extern __shared__ double lists[];
    __shared__ int pos[kMaxM];
    for (int k = threadIdx.x; k < nl * m; k += blockDim.x) lists[k] = cv[k];
    __syncthreads();
    if (threadIdx.x < 64) merge_lists<4>(nl, m, lists, pos);
    __syncthreads();
    for (int r = threadIdx.x; r < m; r += blockDim.x) idx[r] = pos[r] < 0 ? -1 : ci[pos[r]];
}

hipError_t launch_topm(const Plan& pl, const double* norms, double* cand_v, int64_t* cand_i,
                       int64_t* idx, hipStream_t st) {
    static const bool lds_once =
        ((void)hipFuncSetAttribute((const void*)k_topm_final, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   256 * kMaxM * (int)sizeof(double)),
         (void)hipGetLastError(), true);   // advisory: no sticky error is left behind
    (void)lds_once;
    if (pl.topm_grid > 256 || pl.m > kMaxM) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_topm_local, dim3(pl.topm_grid), dim3(256), 0, st, pl.n, pl.m, norms,
                       cand_v, cand_i);
    hipLaunchKernelGGL(k_topm_final, dim3(1), dim3(1024),
                       sizeof(double) * (size_t)pl.topm_grid * pl.m, st, pl.topm_grid, pl.m,
                       cand_v, cand_i, idx);
    return hipGetLastError();
}

// g64[j*p + r] = A[r, idx[j]] in FP64 (dequantized and scaled for 16/8-bit storage).
__global__ void k_gather(PassParams pp, int dtype, const int64_t* __restrict__ idx,
                         double* __restrict__ g64) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)pp.m * pp.p) return;
    const int j = (int)(e / pp.p), r = (int)(e % pp.p);
    const int64_t c = idx[j];
    double v;
    if (dtype == GPSPCA_BF16)
        v = (double)bf16_value(pp.Abf[c * pp.lda + r]) * (double)column_scale(pp, c);
    else if (dtype == GPSPCA_F8E4M3)
        v = (double)e4m3_value(pp.Af8[c * pp.lda + r]) * (double)column_scale(pp, c);
    else
        v = (double)pp.A[c * pp.lda + r];
    g64[e] = v;
}

hipError_t launch_gather(const Plan& pl, const PassParams& pp, const int64_t* idx, double* g64,
                         hipStream_t st) {
    const int64_t ne = (int64_t)pl.m * pl.p;
    hipLaunchKernelGGL(k_gather, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, pp,
                       pl.dtype, idx, g64);
    return hipGetLastError();
}

// Support words and per-block sums of s^2 per component.  S is row-major
// (n x m): thread t takes component t % m of word blockIdx.x * (256 / m) + t / m,
// so each load instruction of a wave reads consecutive components of a row.
// Bound by latency: one row at a time it took 10 instead of 4.8 us at n = 20011,
// m = 16.
__global__ __launch_bounds__(256) void k_fin_support(int64_t n, int m, const float* __restrict__ S,
                                                     uint32_t* __restrict__ support,
                                                     double* __restrict__ fin,
                                                     const Ctrl* __restrict__ ctrl) {
    if (ctrl && ctrl->abort) return;
    __shared__ double red[256];
    const int t = threadIdx.x;
    const int wpb = 256 / m, j = t % m, k = t / m;
    const int64_t nw = (n + 31) / 32;
    const int64_t w = (int64_t)blockIdx.x * wpb + k;
    double ss = 0.0;
    if (k < wpb && w < nw) {
        uint32_t bits = 0;
        const int64_t i0 = w * 32;
        const int cnt = (int)((n - i0) < 32 ? (n - i0) : 32);
        // every load of the word is in flight together (rows past the last one
        // re-read it and count as zero)
        float s[32];
#pragma unroll
        for (int b = 0; b < 32; ++b) s[b] = S[(i0 + (b < cnt ? b : cnt - 1)) * m + j];
#pragma unroll
        for (int b = 0; b < 32; ++b) {
            const float v = b < cnt ? s[b] : 0.f;
            bits |= (v != 0.f ? 1u : 0u) << b;
            ss += (double)v * (double)v;
        }
        if (support) support[(size_t)j * nw + w] = bits;
    }
    red[t] = ss;
    __syncthreads();
    // per component, a fixed pairwise tree over the block's words
    for (int h = 1; h < wpb; h <<= 1) {
        if (k < wpb && (k & (2 * h - 1)) == 0 && k + h < wpb) red[t] += red[t + h * m];
        __syncthreads();
    }
    if (k == 0) fin[(size_t)blockIdx.x * m + j] = red[t];
}

// 1 / ||s_j|| from the per-block sums; grid (components), 256 threads: strided
// per-thread sums in block order, then a fixed tree.
__global__ __launch_bounds__(256) void k_fin_norm(int m, int nblk, const double* __restrict__ fin,
                                                  double* __restrict__ invn) {
    __shared__ double red[256];
    const int j = blockIdx.x, t = threadIdx.x;
    double s = 0.0;
    for (int b = t; b < nblk; b += 256) s += fin[(size_t)b * m + j];
    red[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
    }
    if (t == 0) invn[j] = red[0] > 0.0 ? 1.0 / sqrt(red[0]) : 0.0;
}

// Z[i + j*n] = S[i*m + j] * invn[j]  (invn == nullptr: plain transpose).  A
// workgroup transposes 64 rows of S through LDS: rows are read as one
// contiguous block, and each column j of Z is written as 64 consecutive
// values.
__global__ __launch_bounds__(256) void k_fin_z(int64_t n, int m, const float* __restrict__ S,
                                               const double* __restrict__ invn,
                                               float* __restrict__ Z,
                                               const Ctrl* __restrict__ ctrl) {
    if (ctrl && ctrl->abort) return;
    __shared__ float tile[64 * (kMaxM + 1)];
    const int t = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * 64;
    const int rows = (int)((n - i0) < 64 ? (n - i0) : 64);
    const int ld = m + 1;
    for (int e = t; e < rows * m; e += 256) tile[(e / m) * ld + e % m] = S[i0 * m + e];
    __syncthreads();
    for (int e = t; e < 64 * m; e += 256) {
        const int j = e >> 6, ii = e & 63;
        if (ii < rows) {
            const float s = tile[ii * ld + j];
            Z[(size_t)j * n + i0 + ii] = invn ? (float)((double)s * invn[j]) : s;
        }
    }
}

// ctrl (may be NULL): of a solve whose persistent kernel may have given up.  It runs
// again then, and its start X0 may lie in an output: nothing is written.
hipError_t launch_finalize(const Plan& pl, const float* S, double* fin, double* invn, float* Z,
                           uint32_t* support, const Ctrl* ctrl, hipStream_t st) {
    if (invn) {
        hipLaunchKernelGGL(k_fin_support, dim3(pl.fin_grid), dim3(256), 0, st, pl.n, pl.m, S,
                           support, fin, ctrl);
        hipLaunchKernelGGL(k_fin_norm, dim3(pl.m), dim3(256), 0, st, pl.m, pl.fin_grid, fin, invn);
    }
    if (Z)
        hipLaunchKernelGGL(k_fin_z, dim3((unsigned)((pl.n + 63) / 64)), dim3(256), 0, st, pl.n,
                           pl.m, S, invn, Z, ctrl);
    return hipGetLastError();
}

// Xout (p x m, leading dim p) <- Xint (leading dim ldx)
__global__ void k_copy_x(int m, int p, int ldx, const float* __restrict__ Xi, float* __restrict__ Xo) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)m * p) return;
    const int j = (int)(e / p), r = (int)(e % p);
    Xo[e] = Xi[(size_t)j * ldx + r];
}

// The same from the iterate of the last pass, X_{n_iter - 1}, which sits in
// Xa (n_iter odd) or Xb (n_iter even); nothing when no pass was made or the
// persistent kernel gave up.
__global__ void k_copy_x_last(int m, int p, int ldx, const float* __restrict__ Xa,
                              const float* __restrict__ Xb, const Ctrl* __restrict__ ctrl,
                              float* __restrict__ Xo) {
    const int ni = ctrl->n_iter;
    if (ni < 1 || ctrl->abort) return;
    const float* Xi = ((ni - 1) & 1) ? Xb : Xa;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)m * p) return;
    const int j = (int)(e / p), r = (int)(e % p);
    Xo[e] = Xi[(size_t)j * ldx + r];
}

hipError_t launch_copy_x_last(const Plan& pl, const float* Xa, const float* Xb, const Ctrl* ctrl,
                              float* Xout, hipStream_t st) {
    const int64_t ne = (int64_t)pl.m * pl.p;
    hipLaunchKernelGGL(k_copy_x_last, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, pl.m,
                       (int)pl.p, pl.ldx, Xa, Xb, ctrl, Xout);
    return hipGetLastError();
}

hipError_t launch_copy_x(const Plan& pl, const float* Xint, float* Xout, hipStream_t st) {
    const int64_t ne = (int64_t)pl.m * pl.p;
    hipLaunchKernelGGL(k_copy_x, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, pl.m,
                       (int)pl.p, pl.ldx, Xint, Xout);
    return hipGetLastError();
}

}  // namespace gpspca

namespace gpspca {

// Ascending list of the columns whose support bit is set for at least one
// component (the columns a frozen-support pass has to read).  One workgroup;
// each thread owns one 32-column word per round, and a workgroup prefix sum of
// the word populations places the thread's columns.
__global__ __launch_bounds__(1024) void k_mask_list(const uint32_t* __restrict__ mask,
                                                    int64_t words, int m, int64_t n,
                                                    int* __restrict__ list,
                                                    int* __restrict__ nlist) {
    __shared__ int wave_tot[16];
    __shared__ int base_s;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (t == 0) base_s = 0;
    __syncthreads();
    for (int64_t w0 = 0; w0 < words; w0 += 1024) {
        const int64_t wi = w0 + t;
        uint32_t u = 0;
        if (wi < words) {
            for (int j = 0; j < m; ++j) u |= mask[(int64_t)j * words + wi];
            if (wi == words - 1 && (n & 31)) u &= (1u << (n & 31)) - 1u;
        }
        const int c = __popc(u);
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        if (lane == 63) wave_tot[wv] = incl;
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < 16; ++w) {
            const int v = wave_tot[w];
            if (w < wv) before += v;
            total += v;
        }
        int pos = base_s + before + incl - c;
        while (u) {
            const int b = __ffs(u) - 1;
            list[pos++] = (int)(wi * 32 + b);
            u &= u - 1u;
        }
        __syncthreads();
        if (t == 0) base_s += total;
        __syncthreads();
    }
    if (t == 0) *nlist = base_s;
}

hipError_t launch_mask_list(const uint32_t* mask, int64_t words, int m, int64_t n, int* list,
                            int* nlist, hipStream_t st) {
    hipLaunchKernelGGL(k_mask_list, dim3(1), dim3(1024), 0, st, mask, words, m, n, list, nlist);
    return hipGetLastError();
}

}  // namespace gpspca
