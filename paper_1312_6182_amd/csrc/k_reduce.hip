// Reduction, retraction and stopping kernels of the GP-SPCA power iteration.
//
// After a pass has produced per-workgroup partials of the ascent direction G
// (FP32) and per-wave objective partials (FP64), these kernels:
//   k_reduce_partials  sum the G partials in a fixed order (FP64 accumulation),
//   k_gram             finish G (FP64), and per row block the Gram matrices
//                      G^T G, G^T X_k, X_k^T X_k,
//   k_stop             (one workgroup) sum the objective F_k in fixed order, apply
//                      the stopping rule, and compute the retraction
//                      X_{k+1} = G Omega + X_k Psi:
//                        m = 1   Omega = 1/||g||           (unit sphere)
//                        block   Omega = (G^T G)^{-1/2}    (polar factor on the
//                                Stiefel manifold), in FP64 by a Newton-Schulz
//                                iteration, by a cyclic Jacobi eigen-
//                                decomposition where that does not converge;
//                        dead components (empty support) are completed by the
//                        polar factor of the previous columns projected off the
//                        live part, expressed through the same Gram matrices,
//   k_apply            X_{k+1} = G Omega + X_k Psi, rounded to FP32.
// Every reduction runs in a fixed order, so results are bitwise reproducible.
#include "gpspca_internal.h"
#include "retract.h"

namespace gpspca {

// Allow dynamic LDS beyond 64 KB (gfx950 has 160 KB per CU).
static void set_lds_limit(const void* fn) {
    (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipGetLastError();  // the attribute is advisory; do not leave a sticky error behind
}

// ---------------------------------------------------------------------------
__global__ void k_fill_zero(uint32_t* __restrict__ p, size_t words) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t st) {
    const size_t words = bytes / 4;
    if (words == 0) return hipSuccess;
    size_t blocks = (words + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<uint32_t*>(ptr), words);
    return hipGetLastError();
}

__device__ __forceinline__ void ctrl_reset_fields(Ctrl* ctrl, int max_iter, double tol) {
    ctrl->k = 0;
    ctrl->done = 0;
    ctrl->status = GPSPCA_OK;
    ctrl->n_iter = 0;
    ctrl->ndead = 0;
    ctrl->degenerate_seen = 0;
    ctrl->max_iter = max_iter;
    ctrl->warm = 0;
    ctrl->nact = 0;
    ctrl->no_newton = 0;
    ctrl->bar = 0;
    ctrl->abort = 0;
    ctrl->tol = tol;
    ctrl->last_F = 0.0;
}

// Start of a solve in one launch: the control block reset (thread 0 of
// workgroup 0), the listed buffers cleared, and g64[j p + r] = X0[j ldx0 + r]
// in FP64 for j < m (m = 0: no X0).
__global__ __launch_bounds__(256) void k_start(Ctrl* ctrl, int max_iter, double tol, StartZero z,
                                               int m, int p, const float* __restrict__ X0,
                                               int ldx0, double* __restrict__ g64) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctrl_reset_fields(ctrl, max_iter, tol);
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (int b = 0; b < z.n; ++b) {
        uint32_t* ptr = z.ptr[b];
        const size_t w = z.words[b];
        for (size_t i = i0; i < w; i += step) ptr[i] = 0u;
    }
    const size_t ne = (size_t)m * p;
    for (size_t e = i0; e < ne; e += step) {
        const size_t j = e / p, r = e % p;
        g64[e] = (double)X0[j * ldx0 + r];
    }
}

hipError_t launch_start(Ctrl* ctrl, int max_iter, double tol, const StartZero& z, int m, int p,
                        const float* X0, int ldx0, double* g64, hipStream_t st) {
    size_t most = X0 ? (size_t)m * p : 0;
    for (int i = 0; i < z.n; ++i) most = z.words[i] > most ? z.words[i] : most;
    size_t blocks = (most + 255) / 256;
    blocks = blocks < 1 ? 1 : blocks > 4096 ? 4096 : blocks;
    hipLaunchKernelGGL(k_start, dim3((unsigned)blocks), dim3(256), 0, st, ctrl, max_iter, tol, z,
                       X0 ? m : 0, p, X0, ldx0, g64);
    return hipGetLastError();
}

__global__ void k_ctrl_reset(Ctrl* ctrl, int max_iter, double tol) {
    if (threadIdx.x == 0) ctrl_reset_fields(ctrl, max_iter, tol);
}

hipError_t launch_ctrl_reset(Ctrl* ctrl, int max_iter, double tol, hipStream_t st) {
    hipLaunchKernelGGL(k_ctrl_reset, dim3(1), dim3(64), 0, st, ctrl, max_iter, tol);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// l1[y][e] = sum_{c in chunk y} gpart[c][e]  (e < m*ldx), skipping untouched
// partials; chunks are contiguous ranges of the partial index.
__global__ __launch_bounds__(256) void k_reduce_partials(const float* __restrict__ gpart,
                                                         const int* __restrict__ touched,
                                                         int npart, int nsplit, int64_t ne,
                                                         double* __restrict__ l1,
                                                         const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    const int y = blockIdx.y;
    const int c0 = (int)((int64_t)npart * y / nsplit), c1 = (int)((int64_t)npart * (y + 1) / nsplit);
    // this split's touched partials as an ascending list in LDS, built once
    // (a partial that no workgroup wrote is neither read nor added)
    __shared__ int plist[1024];
    __shared__ int wcnt[4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const bool staged = touched && (c1 - c0) <= 1024;
    int nlist = 0;
    if (staged) {
        for (int b = 0; b < c1 - c0; b += 256) {
            const int i = b + t;
            const bool on = i < c1 - c0 && touched[c0 + i] != 0;
            const uint64_t bal = __ballot(on);
            if (lane == 0) wcnt[wv] = __popcll(bal);
            __syncthreads();
            int before = nlist;
            for (int w = 0; w < wv; ++w) before += wcnt[w];
            if (on) plist[before + __popcll(bal & ((1ull << lane) - 1ull))] = c0 + i;
            nlist += wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
            __syncthreads();
        }
    }
    const int64_t e = (int64_t)blockIdx.x * 256 + t;
    if (e >= ne) return;
    double s = 0.0;
    int c = c0;
    if (staged) {
        // in list order (ascending c); the loads of 8 partials are issued
        // together (past the end the last one is re-read and not added)
        for (int q = 0; q < nlist; q += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = gpart[(size_t)plist[q + u < nlist ? q + u : nlist - 1] * ne + e];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q + u < nlist) s += (double)v[u];
        }
        c = c1;
    } else if (!touched) {
        for (; c + 4 <= c1; c += 4) {
            const float v0 = gpart[(size_t)c * ne + e];
            const float v1 = gpart[(size_t)(c + 1) * ne + e];
            const float v2 = gpart[(size_t)(c + 2) * ne + e];
            const float v3 = gpart[(size_t)(c + 3) * ne + e];
            s += (double)v0;
            s += (double)v1;
            s += (double)v2;
            s += (double)v3;
        }
    }
    for (; c < c1; ++c)
        if (!touched || touched[c]) s += (double)gpart[(size_t)c * ne + e];
    l1[(size_t)y * ne + e] = s;
}

hipError_t launch_reduce_partials(const Plan& pl, const float* gpart, const int* touched,
                                  double* l1, const Ctrl* ctrl, hipStream_t st) {
    const int64_t ne = (int64_t)pl.m * pl.ldx;
    dim3 grid((unsigned)((ne + 255) / 256), (unsigned)pl.red_split);
    hipLaunchKernelGGL(k_reduce_partials, grid, dim3(256), 0, st, gpart, touched, pl.npart,
                       pl.red_split, ne, l1, ctrl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// G^T G, G^T X and X^T X (with_x; else zeros) of one row block held in LDS (gt,
// xt: leading dim ld >= m, rows up to the next multiple of 16 past nr zero) on the
// FP64 matrix cores: a wave takes 16 x 16 tiles of the products in turn, the upper
// ones of the two symmetric products, 4 rows per v_mfma_f64_16x16x4_f64 (lane l:
// row l / 16, components l % 16 of both sides; entry v of the result is component
// 4 v + l / 16 against l % 16) in two alternating sums.  Components past m repeat
// the last one and are not stored.  One thread per entry, walking the rows,
// spent its time on the LDS reads of that chain.
__device__ __forceinline__ void gram_products(const double* gt, const double* xt, int ld, int nr,
                                              int m, bool with_x, double* __restrict__ out) {
    using d4 = __attribute__((ext_vector_type(4))) double;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int nt = (m + 15) / 16, up = nt * (nt + 1) / 2, mm = m * m;
    const int ntask = with_x ? 2 * up + nt * nt : up;
    for (int q = wv; q < ntask; q += nwv) {
        const int which = q < up ? 0 : q < 2 * up ? 2 : 1;
        int ti, tj;
        if (which == 1) {
            ti = (q - 2 * up) / nt;
            tj = (q - 2 * up) % nt;
        } else {
            int u = which == 0 ? q : q - up;
            ti = 0;
            while (u >= nt - ti) u -= nt - ti++;
            tj = ti + u;
        }
        const int ca = 16 * ti + li < m ? 16 * ti + li : m - 1;
        const int cb = 16 * tj + li < m ? 16 * tj + li : m - 1;
        const double* a = (which == 2 ? xt : gt) + lk * ld + ca;
        const double* b = (which == 0 ? gt : xt) + lk * ld + cb;
        d4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
        for (int r = 0; r < nr; r += 16) {
            double av[4], bv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                av[k] = a[(r + 4 * k) * ld];
                bv[k] = b[(r + 4 * k) * ld];
            }
            s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[0], bv[0], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[1], bv[1], s1, 0, 0, 0);
            s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[2], bv[2], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[3], bv[3], s1, 0, 0, 0);
        }
        s0 += s1;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * ti + 4 * v + lk, j = 16 * tj + li;
            if (i < m && j < m) {
                out[which * mm + i * m + j] = s0[v];
                if (which != 1 && ti != tj) out[which * mm + j * m + i] = s0[v];
            }
        }
    }
    if (!with_x)
        for (int e = threadIdx.x; e < 2 * mm; e += blockDim.x) out[mm + e] = 0.0;
}

// The diagonal of G^T G only (a gamma path): S row slices per component, added
// by a fixed-order tree.  red: 256 doubles; every thread of the workgroup calls.
__device__ __forceinline__ void gram_diagonal(const double* gt, int ld, int nr, int m, double* red,
                                              double* __restrict__ out) {
    const int t = threadIdx.x;
    int S = 1;
    while (2 * S * m <= 256 && S < 64) S *= 2;
    if (t < m * S) {
        const int j = t % m;
        double acc = 0.0;
        for (int r = t / m; r < nr; r += S) acc += gt[r * ld + j] * gt[r * ld + j];
        red[t] = acc;
    }
    __syncthreads();
    for (int h = S / 2; h >= 1; h /= 2) {
        if (t < m * h) red[t] += red[t + m * h];
        __syncthreads();
    }
    if (t < m) out[t * m + t] = red[t];
}

// Row block r0..r0+nr: g_r = sum_y l1[y][.][r] (fixed order) -> g64 (p x m,
// leading dim p); partial Gram matrices over the block ->
// gram[blk][0|1|2][m*m] = G^T G, G^T X, X^T X.  Bound by the latency of its
// loads: four elements of a thread are in flight together.  With one element at
// a time and a thread per Gram entry it took 13.6 instead of 6.6 us at p = 1999,
// m = 16 (5 splits) and 36 instead of 28 at p = 10000, m = 64.
__global__ __launch_bounds__(256) void k_gram(const double* __restrict__ l1, int nsplit, int m,
                                              int ldx, int p, int rows, const float* __restrict__ X,
                                              int with_x, double* __restrict__ g64,
                                              double* __restrict__ gram,
                                              const Ctrl* __restrict__ ctrl) {
    if (ctrl && ctrl->done) return;
    extern __shared__ double sh[];
    __shared__ double red[256];
    constexpr int U = 4;
    const int mp = m + 1;
    double* gt = sh;                         // rows x (m+1)
    double* xt = sh + (size_t)rows * mp;     // rows x (m+1)
    const int r0 = blockIdx.x * rows;
    const int nr = (p - r0 < rows) ? p - r0 : rows;
    const int t = threadIdx.x;
    const size_t ne = (size_t)m * ldx;
    for (int e0 = t; e0 < nr * m; e0 += U * 256) {
        double s[U];
        float x[U];
        int rr[U], j[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + 256 * u < nr * m ? e0 + 256 * u : nr * m - 1;
            rr[u] = e % nr;
            j[u] = e / nr;
            x[u] = (with_x == 1) ? X[(size_t)j[u] * ldx + r0 + rr[u]] : 0.f;
        }
        if (!l1 || nsplit == 1) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                s[u] = l1 ? l1[(size_t)j[u] * ldx + r0 + rr[u]]
                          : g64[(size_t)j[u] * p + r0 + rr[u]];
        } else {
            // in order of y, four splits at a time (past the end the last one is
            // re-read and not added)
#pragma unroll
            for (int u = 0; u < U; ++u) s[u] = 0.0;
            for (int y = 0; y < nsplit; y += 4) {
                double v[U][4];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        v[u][k] = l1[(size_t)(y + k < nsplit ? y + k : nsplit - 1) * ne +
                                     (size_t)j[u] * ldx + r0 + rr[u]];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (y + k < nsplit) s[u] += v[u][k];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e0 + 256 * u < nr * m) {
                if (l1) g64[(size_t)j[u] * p + r0 + rr[u]] = s[u];
                gt[rr[u] * mp + j[u]] = s[u];
                xt[rr[u] * mp + j[u]] = (double)x[u];
            }
    }
    for (int e = nr * mp + t; e < ((nr + 15) & ~15) * mp; e += 256) gt[e] = xt[e] = 0.0;
    __syncthreads();
    double* out = gram + (size_t)blockIdx.x * 3 * m * m;
    if (with_x == 2) gram_diagonal(gt, mp, nr, m, red, out);
    else gram_products(gt, xt, mp, nr, m, with_x == 1, out);
}

hipError_t launch_gram(const Plan& pl, const double* l1, int nsplit, const float* X, int with_x,
                       double* g64, double* gram, const Ctrl* ctrl, hipStream_t st) {
    const size_t shm = (size_t)2 * pl.gram_rows * (pl.m + 1) * sizeof(double);
    static const bool lds_once = (set_lds_limit((const void*)k_gram), true);
    (void)lds_once;
    hipLaunchKernelGGL(k_gram, dim3(pl.gram_grid), dim3(256), shm, st, l1, nsplit, pl.m, pl.ldx,
                       (int)pl.p, pl.gram_rows, X, with_x, g64, gram, ctrl);
    return hipGetLastError();
}

// Final fixed-order reduction of the per-row-block Gram partials into the
// coefficient scratch: coef[2mm + e] = sum_g gram[g][e] for e < nent.
// Each workgroup owns EPB = 256 / S entries; S slices per entry sum the
// partials g = sl, sl + S, ... and a fixed-order tree adds the slices.
// Blocks past the Gram entries (fsum != NULL) each sum one component's
// objective and support-size partials: fsum[j] = sum_w fpart[j nwp + w],
// fsum[m + j] = sum_w nnzpart[j nwp + w] (thread slices in order, then a fixed
// tree), so the one-workgroup stop kernel reads 2m numbers.
__global__ __launch_bounds__(256) void k_gram_sum(int nent, int mm, int ngram, int S,
                                                  const double* __restrict__ gram,
                                                  double* __restrict__ coef,
                                                  const double* __restrict__ fpart,
                                                  const int* __restrict__ nnzpart, int nwp,
                                                  int m, double* __restrict__ fsum,
                                                  const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ double red[256];
    __shared__ long long redc[256];
    const int t = threadIdx.x, epb = 256 / S;
    const int nblk = (nent + epb - 1) / epb;
    if ((int)blockIdx.x >= nblk) {
        const int j = blockIdx.x - nblk;
        double sf = 0.0;
        long long sc = 0;
        for (int w0 = t; w0 < nwp; w0 += 8 * 256) {
            double v[8];
            int c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int w = w0 + u * 256;
                const int wc = w < nwp ? w : nwp - 1;
                v[u] = fpart[(size_t)j * nwp + wc];
                c[u] = nnzpart[(size_t)j * nwp + wc];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (w0 + u * 256 < nwp) {
                    sf += v[u];
                    sc += c[u];
                }
        }
        red[t] = sf;
        redc[t] = sc;
        __syncthreads();
        for (int hh = 128; hh >= 1; hh >>= 1) {
            if (t < hh) {
                red[t] += red[t + hh];
                redc[t] += redc[t + hh];
            }
            __syncthreads();
        }
        if (t == 0) {
            fsum[j] = red[0];
            fsum[m + j] = (double)redc[0];
        }
        return;
    }
    const int el = t % epb, sl = t / epb;
    const int e = blockIdx.x * epb + el;
    double s = 0.0;
    if (e < nent) {
        // in order of g; the loads of 8 terms are issued together (indices past
        // the end re-read the last term and are not added)
        const double* gp = gram + e;
        for (int g0 = sl; g0 < ngram; g0 += 8 * S) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int g = g0 + u * S;
                v[u] = gp[(size_t)(g < ngram ? g : ngram - 1) * 3 * mm];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (g0 + u * S < ngram) s += v[u];
        }
    }
    red[t] = s;
    __syncthreads();
    for (int h = S / 2; h >= 1; h /= 2) {
        if (sl < h) red[t] += red[t + h * epb];
        __syncthreads();
    }
    if (sl == 0 && e < nent) coef[2 * mm + e] = red[t];
}

hipError_t launch_gram_sum(const Plan& pl, int nent, int ngram, const double* gram, double* coef,
                           const Ctrl* ctrl, hipStream_t st, const double* fpart,
                           const int* nnzpart, double* fsum) {
    const int mm = pl.m * pl.m;
    // slices per entry: enough to shorten the serial chains, while keeping at
    // least a few workgroups busy
    int S = 1;
    while (S < 64 && S * 8 <= ngram && (nent * 2 * S + 255) / 256 <= 64) S *= 2;
    const int epb = 256 / S;
    const int blocks = (nent + epb - 1) / epb + (fsum ? pl.m : 0);
    hipLaunchKernelGGL(k_gram_sum, dim3(blocks), dim3(256), 0, st, nent, mm, ngram, S, gram, coef,
                       fpart, nnzpart, pl.nwave_part, pl.m, fsum, ctrl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fused partial reduction + Gram for m <= 16: one workgroup per 64 rows.
// Thread (row rr, slice sl) sums the partials c = sl, sl + NSL, ... of its row for
// every component, the slices are added in order (fixed order), the row of G is
// written in FP64, and the block's contributions to G^T G, G^T X, X^T X (or only
// the diagonal of G^T G, with_x == 2) go to gram[block].  Bound by the latency of
// the partials' loads, 4 partials per thread in flight: few row blocks take a
// workgroup per CU with 16 slices (8 for m > 8, whose sums fill the LDS).  4 slices
// and a thread per Gram entry took 8.0 instead of 5.5 us at p = 800, n = 8000, m = 5
// and 9.9 instead of 6.5 at 10000 x 100000, m = 8.
template <int MB, int NSL>
__global__ __launch_bounds__(64 * NSL) void k_reduce_gram(const float* __restrict__ gpart,
                                                     const int* __restrict__ touched, int npart,
                                                     int m, int ldx, int p,
                                                     const float* __restrict__ X, int with_x,
                                                     double* __restrict__ g64,
                                                     double* __restrict__ gram,
                                                     const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    constexpr int MP = MB + 1, T = 64 * NSL;
    extern __shared__ double sh[];
    double* const part = sh;                    // NSL x 64 x MP
    double* const gt = sh + NSL * 64 * MP;      // 64 x MP
    double* const xt = gt + 64 * MP;
    __shared__ int plist[1024];
    __shared__ int wcnt[NSL];
    const int t = threadIdx.x, rr = t & 63, sl = t >> 6;
    const int r0 = blockIdx.x * 64;
    const int r = r0 + rr;
    const int nr = (p - r0 < 64) ? p - r0 : 64;
    const size_t stride = (size_t)m * ldx;
    // ascending list of the partials that hold data (all of them without flags),
    // built in parallel so that the sums below never wait on a flag
    int nlist = 0;
    for (int c0 = 0; c0 < npart; c0 += T) {
        const int c = c0 + t;
        const bool on = c < npart && (!touched || touched[c] != 0);
        const uint64_t bal = __ballot(on);
        if (rr == 0) wcnt[sl] = __popcll(bal);
        __syncthreads();
        int before = nlist;
#pragma unroll
        for (int w = 0; w < NSL; ++w) {
            before += w < sl ? wcnt[w] : 0;
            nlist += wcnt[w];
        }
        const int at = before + __popcll(bal & ((1ull << rr) - 1ull));
        if (on && at < 1024) plist[at] = c;
        __syncthreads();
    }
    double g[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) g[j] = 0.0;
    // component offsets: components >= m re-read component m - 1 (a valid
    // address) and are dropped by a select, so the loads stay unconditional and
    // are issued together instead of one branch and one wait per component
    size_t joff[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) joff[j] = (size_t)(j < m ? j : m - 1) * ldx + r;
    if (r < p && nlist <= 1024) {
        for (int e = sl; e < nlist; e += 4 * NSL) {
            float v[4][MB];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int eu = e + u * NSL < nlist ? e + u * NSL : nlist - 1;
                const float* src = gpart + (size_t)plist[eu] * stride;
#pragma unroll
                for (int j = 0; j < MB; ++j) v[u][j] = src[joff[j]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (e + u * NSL < nlist) {
#pragma unroll
                    for (int j = 0; j < MB; ++j) g[j] += (j < m) ? (double)v[u][j] : 0.0;
                }
        }
    } else if (r < p) {
        // more than 1024 partials: walk the flags directly
        for (int c = sl; c < npart; c += NSL) {
            if (touched && !touched[c]) continue;
            float v[MB];
            const float* src = gpart + (size_t)c * stride;
#pragma unroll
            for (int j = 0; j < MB; ++j) v[j] = src[joff[j]];
#pragma unroll
            for (int j = 0; j < MB; ++j) g[j] += (j < m) ? (double)v[j] : 0.0;
        }
    }
#pragma unroll
    for (int j = 0; j < MB; ++j) part[(sl * 64 + rr) * MP + j] = g[j];
    __syncthreads();
    for (int j = sl; j < MB; j += NSL) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < NSL; ++w) v += part[(w * 64 + rr) * MP + j];
        gt[rr * MP + j] = v;
        if (r < p && j < m) g64[(size_t)j * p + r] = v;
        xt[rr * MP + j] = (with_x == 1 && r < p && j < m) ? (double)X[(size_t)j * ldx + r] : 0.0;
    }
    __syncthreads();
    double* out = gram + (size_t)blockIdx.x * 3 * m * m;
    if (with_x == 2) gram_diagonal(gt, MP, nr, m, part, out);
    else gram_products(gt, xt, MP, nr, m, with_x == 1, out);
}

template <int MB, int NSL>
static void launch_reduce_gram_t(const Plan& pl, const float* gpart, const int* touched,
                                 const float* X, int with_x, double* g64, double* gram,
                                 const Ctrl* ctrl, hipStream_t st) {
    static const bool lds_once = (set_lds_limit((const void*)k_reduce_gram<MB, NSL>), true);
    (void)lds_once;
    hipLaunchKernelGGL((k_reduce_gram<MB, NSL>), dim3((unsigned)((pl.p + 63) / 64)),
                       dim3(64 * NSL), sizeof(double) * (NSL + 2) * 64 * (MB + 1), st, gpart,
                       touched, pl.npart, pl.m, pl.ldx, (int)pl.p, X, with_x, g64, gram, ctrl);
}

hipError_t launch_reduce_gram(const Plan& pl, const float* gpart, const int* touched,
                              const float* X, int with_x, double* g64, double* gram,
                              const Ctrl* ctrl, hipStream_t st) {
    // up to 256 row blocks there is a CU for each
    const bool wide = pl.p <= 64 * 256;
#define GPSPCA_RG(MB, NSL)                                                                     \
    (wide ? launch_reduce_gram_t<MB, NSL>(pl, gpart, touched, X, with_x, g64, gram, ctrl, st)  \
          : launch_reduce_gram_t<MB, 4>(pl, gpart, touched, X, with_x, g64, gram, ctrl, st))
    if (pl.m <= 1) GPSPCA_RG(1, 16);
    else if (pl.m <= 2) GPSPCA_RG(2, 16);
    else if (pl.m <= 4) GPSPCA_RG(4, 16);
    else if (pl.m <= 8) GPSPCA_RG(8, 16);
    else GPSPCA_RG(16, 8);
#undef GPSPCA_RG
    return hipGetLastError();
}

// s, c = sum of fp[w], cp[w] over w = sl, sl + step, ... < nwp, in that
// order.  The loads of B terms are issued together (indices past the end
// re-read the last term and add 0, which leaves the non-negative sums as they
// were), instead of one dependent load at a time.
template <int B>
__device__ __forceinline__ void slice_sum(const double* __restrict__ fp,
                                          const int* __restrict__ cp, int nwp, int sl, int step,
                                          double* s_out, int* c_out) {
    double s = 0.0;
    int c = 0;
    for (int w0 = sl; w0 < nwp; w0 += B * step) {
        double fv[B];
        int cv[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int w = w0 + u * step;
            const int wc = w < nwp ? w : nwp - 1;
            fv[u] = fp[wc];
            cv[u] = cp[wc];
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const bool in = w0 + u * step < nwp;
            s += in ? fv[u] : 0.0;
            c += in ? cv[u] : 0;
        }
    }
    *s_out = s;
    *c_out = c;
}

// Objective of a pass, its trace entry and the stopping rule, by the whole
// workgroup: per-component terms f_j and support sizes from the fixed-order
// sums of the wave partials, F, and the rule (F = 0, the relative change
// below tol, or the last allowed pass).  Fills ss (terms, live and dead
// components, stop) and the control block; returns the stop flag.
// kGiven: fsum is always given (the branch that sums the partials is left out).
template <bool kGiven = false>
__device__ int stop_rule(int m, int nwp, const double* __restrict__ fpart,
                         const int* __restrict__ nnzpart, double* __restrict__ trace,
                         double* __restrict__ fcomp, int exact, Ctrl* __restrict__ ctrl,
                         StopShared& ss, const double* __restrict__ fsum = nullptr) {
    const int t = threadIdx.x, nt = blockDim.x;
    const int k = ctrl->k;
    // the control fields the stopping rule needs, loaded up front so their
    // latency overlaps the sums
    const double last_F = ctrl->last_F, tol = ctrl->tol;
    const int max_iter = ctrl->max_iter, deg_seen = ctrl->degenerate_seen;

    // per-component objective and support size: summed already (fsum, by the
    // Gram-sum kernel), or here by tpc (a power of two <= 64) lanes of one
    // wave per component, each summing a strided slice, the slices combined by
    // a fixed butterfly (fixed order)
    if (kGiven || fsum) {
        for (int j = t; j < m; j += nt) {
            ss.fj[j] = fsum[j];
            ss.nj[j] = (int)fsum[m + j];
        }
    } else {
        int tpc = 64;
        while (tpc > 1 && tpc * m > nt) tpc >>= 1;
        for (int j0 = 0; j0 < m; j0 += nt / tpc) {
            const int j = j0 + t / tpc, sl = t % tpc;
            double s = 0.0;
            int c = 0;
            if (j < m) slice_sum<32>(fpart + (size_t)j * nwp, nnzpart + (size_t)j * nwp, nwp, sl, tpc,
                                 &s, &c);
            for (int o = tpc / 2; o >= 1; o >>= 1) {
                s += __shfl_xor(s, o, 64);
                c += __shfl_xor(c, o, 64);
            }
            if (sl == 0 && j < m) {
                ss.fj[j] = s;
                ss.nj[j] = c;
            }
        }
    }
    __syncthreads();
    // per-component terms in parallel (original form of block L1: ||s_j||)
    for (int j = t; j < m; j += nt) {
        const double fj = ss.fj[j];
        ss.fterm[j] = exact ? sqrt(fj) : fj;
        ss.dsc[j] = (exact && fj > 0.0) ? 1.0 / sqrt(fj) : 0.0;
        fcomp[j] = fj;
        reinterpret_cast<int64_t*>(fcomp + m)[j] = ss.nj[j];
    }
    __syncthreads();
    if (t == 0) {
        double F = 0.0;
        int nl = 0, nd = 0;
        for (int j = 0; j < m; ++j) {
            F += ss.fterm[j];
            if (ss.nj[j] > 0) ss.live[nl++] = j;
            else ss.dead[nd++] = j;
        }
        ss.nlive = nl;
        ss.ndead = nd;
        trace[k] = F;
        int stop = 0, status = GPSPCA_OK;
        int degenerate = deg_seen;
        if (!isfinite(F)) {
            stop = 1;
            status = GPSPCA_ENONFINITE;
        } else if (F == 0.0) {
            stop = 1;
            degenerate = 1;
            ctrl->degenerate_seen = 1;
        } else if (k >= 1 && fabs(F - last_F) < tol * fabs(last_F)) {
            stop = 1;
        } else if (k + 1 >= max_iter) {
            stop = 1;
            status = GPSPCA_MAXITER;
        }
        if (stop) {
            if (status >= 0 && degenerate) status = GPSPCA_DEGENERATE;
            ctrl->status = status;
            ctrl->done = 1;
            ctrl->n_iter = k + 1;
        }
        ctrl->last_F = F;
        ss.stop = stop;
    }
    __syncthreads();
    return ss.stop;
}

// m = 1: ||g||^2 as the sum of the ngram Gram partials (entry 0 of each
// 3-entry block; strided per-thread sums, a fixed butterfly in each wave, the
// waves in order), 1/||g|| into coef, and the check that it is finite.
// Returns 1/||g|| to every thread, or 0 when the pass failed.  red: at least
// blockDim.x / 64 doubles of LDS.
__device__ double unit_scale(const double* __restrict__ gram, int ngram,
                             double* __restrict__ coef, int k, Ctrl* __restrict__ ctrl,
                             double* red) {
    const int t = threadIdx.x, nt = blockDim.x;
    double sg = 0.0;
    for (int g = t; g < ngram; g += nt) sg += gram[(size_t)3 * g];
    sg = wave_sum_d(sg);
    if ((t & 63) == 0) red[t >> 6] = sg;
    __syncthreads();
    if (t == 0) {
        double g2 = 0.0;
        for (int u = 0; u < (nt + 63) / 64; ++u) g2 += red[u];
        coef[2] = g2;
        const double om = 1.0 / sqrt(g2);
        coef[0] = om;
        coef[1] = 0.0;
        ctrl->ndead = 0;
        const int bad = (!(g2 > 0.0) || !isfinite(om)) ? 1 : 0;
        if (bad) {
            ctrl->status = GPSPCA_ENONFINITE;
            ctrl->done = 1;
            ctrl->n_iter = k + 1;
        }
        red[0] = bad ? 0.0 : om;
    }
    __syncthreads();
    return red[0];
}

// One workgroup: objective, trace, stopping rule, retraction coefficients.
// m = 1: ||g||^2 is summed here from the ngram Gram partials (no k_gram_sum),
// and with Xn given the retraction x_{k+1} = g / ||g|| is written here too
// (rows < p, FP32), in place of a separate apply launch.
__global__ __launch_bounds__(1024) void k_stop(int m, int nwp, const double* __restrict__ fpart,
                       const int* __restrict__ nnzpart, double* __restrict__ vprev,
                       double* __restrict__ trace, double* __restrict__ coef,
                       double* __restrict__ fcomp, const double* __restrict__ gram, int ngram,
                       int exact, const double* __restrict__ g64, float* __restrict__ Xn, int p,
                       const double* __restrict__ fsum, Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ StopShared ss;
    __shared__ double red[1024];
    extern __shared__ double dyn[];
    double* A0 = dyn;
    // three matrices of m rows rounded up to even (jacobi_eig pads odd sizes)
    const int mr = m + (m & 1);
    double* A1 = dyn + (size_t)mr * LDM;
    double* A2 = dyn + (size_t)2 * mr * LDM;
    const int t = threadIdx.x, nt = blockDim.x;
    const int k = ctrl->k;
    if (stop_rule(m, nwp, fpart, nnzpart, trace, fcomp, exact, ctrl, ss, m > 1 ? fsum : nullptr))
        return;

    const int mm = m * m;
    if (m == 1) {
        const double om = unit_scale(gram, ngram, coef, k, ctrl, red);
        if (Xn && om != 0.0)
            for (int r = t; r < p; r += nt) Xn[r] = (float)(g64[r] * om);
    } else {
        if (exact) {
            // direction G D, D = Diag(1/||s_j||): G^T G <- D G^T G D, G^T X <- D G^T X
            for (int e = t; e < mm; e += nt) {
                const int a = e / m, b = e % m;
                coef[2 * mm + e] *= ss.dsc[a] * ss.dsc[b];
                coef[3 * mm + e] *= ss.dsc[a];
            }
            __syncthreads();
        }
        block_coefficients(m, coef, vprev, ss, A0, A1, A2, ctrl);
        if (exact) {
            // X_{k+1} = (G D) Omega + X_k Psi: row l of Omega takes 1/||s_l||
            __syncthreads();
            for (int e = t; e < mm; e += nt) coef[e] *= ss.dsc[e / m];
            __syncthreads();
        }
        // finiteness of the coefficients (every thread checks its share)
        int bad = 0;
        for (int e = t; e < 2 * mm; e += nt) bad |= isfinite(coef[e]) ? 0 : 1;
        if (__syncthreads_or(bad) && t == 0) {
            ctrl->status = GPSPCA_ENONFINITE;
            ctrl->done = 1;
            ctrl->n_iter = k + 1;
            ctrl->warm = 0;
        }
        __syncthreads();
    }
    if (t == 0 && !ctrl->done) {
        ctrl->k = k + 1;
        ctrl->nact = 0;   // the next pass counts its active columns afresh
    }
}

// Single unit (m = 1) with the retraction written here: stopping rule, ||g||^2
// from the Gram partials and x_{k+1} = g / ||g|| (rows < p, FP32).  Wave 0
// sums the objective and support-size partials (lane l the partials l, l + 64,
// ..., then a fixed butterfly) while waves 1.. load their rows of g (kX1Rows
// each: rows u, u + nt - 64, ... for u = t - 64), so that the latency of both
// overlaps; rows past kX1Rows * (nt - 64), if any, are read afterwards.
constexpr int kX1Rows = 22;   // 22 * 960 >= 20480, the largest p of the fused pass
__global__ __launch_bounds__(1024) void k_stop_x1(int nwp, const double* __restrict__ fpart,
                                                  const int* __restrict__ nnzpart,
                                                  double* __restrict__ trace,
                                                  double* __restrict__ coef,
                                                  double* __restrict__ fcomp,
                                                  const double* __restrict__ gram, int ngram,
                                                  int exact, const double* __restrict__ g64,
                                                  float* __restrict__ Xn, int p,
                                                  Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ StopShared ss;
    __shared__ double red[16];
    __shared__ double fs[2];
    const int t = threadIdx.x, nt = blockDim.x, lane = t & 63;
    const int u0 = t - 64, ust = nt - 64;
    double gx[kX1Rows];
    if (t < 64) {
        double sf;
        int sc;
        slice_sum<8>(fpart, nnzpart, nwp, lane, 64, &sf, &sc);
        for (int o = 32; o >= 1; o >>= 1) {
            sf += __shfl_xor(sf, o, 64);
            sc += __shfl_xor(sc, o, 64);
        }
        if (lane == 0) {
            fs[0] = sf;
            fs[1] = (double)sc;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kX1Rows; ++i) {
            const int r = u0 + i * ust;
            gx[i] = r < p ? g64[r] : 0.0;
        }
    }
    __syncthreads();
    const int k = ctrl->k;
    if (stop_rule<true>(1, nwp, fpart, nnzpart, trace, fcomp, exact, ctrl, ss, fs)) return;
    const double om = unit_scale(gram, ngram, coef, k, ctrl, red);
    if (om != 0.0) {
        if (t >= 64) {
#pragma unroll
            for (int i = 0; i < kX1Rows; ++i) {
                const int r = u0 + i * ust;
                if (r < p) Xn[r] = (float)(gx[i] * om);
            }
        }
        for (int r = kX1Rows * ust + t; r < p; r += nt) Xn[r] = (float)(g64[r] * om);
    }
    if (t == 0 && !ctrl->done) {
        ctrl->k = k + 1;
        ctrl->nact = 0;
    }
}

// m = 1 after the fused pass (one partial g per workgroup, every one written):
// g = the sum of the partials and the Gram partials of ||g||^2 in one launch.
// A workgroup owns kRm1Rows rows; slice sl (threads sl kRm1Rows .. + kRm1Rows
// - 1) of its kRm1Slices sums the contiguous range sl of the partials (all
// loads of a batch issued together), wave 0 adds the ranges in order, writes g
// (FP64) and the block's sum of g_r^2 (a fixed butterfly) as gram[3 * block].  Rows past p re-read row
// p - 1 and are dropped.
constexpr int kRm1Slices = 1024 / kRm1Rows, kRm1Batch = 16;
__global__ __launch_bounds__(1024) void k_reduce_m1(const float* __restrict__ gpart, int npart,
                                                    int ldx, int p, double* __restrict__ g64,
                                                    double* __restrict__ gram,
                                                    const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ double part[kRm1Slices][kRm1Rows];
    const int t = threadIdx.x, rr = t % kRm1Rows, sl = t / kRm1Rows;
    const int r = blockIdx.x * kRm1Rows + rr;
    const int rc = r < p ? r : p - 1;
    const int c0 = (int)((int64_t)npart * sl / kRm1Slices);
    const int c1 = (int)((int64_t)npart * (sl + 1) / kRm1Slices);
    double s = 0.0;
    for (int c = c0; c < c1; c += kRm1Batch) {
        float v[kRm1Batch];
#pragma unroll
        for (int u = 0; u < kRm1Batch; ++u) {
            const int cu = c + u < c1 ? c + u : c1 - 1;
            v[u] = gpart[(size_t)cu * ldx + rc];
        }
#pragma unroll
        for (int u = 0; u < kRm1Batch; ++u) s += (c + u < c1) ? (double)v[u] : 0.0;
    }
    part[sl][rr] = s;
    __syncthreads();
    if (t < 64) {   // wave 0: lanes t < kRm1Rows finish the rows, the rest add 0
        const bool own = t < kRm1Rows && r < p;
        double g = 0.0;
        if (t < kRm1Rows) {
            g = part[0][rr];
#pragma unroll
            for (int u = 1; u < kRm1Slices; ++u) g += part[u][rr];
        }
        if (own) g64[r] = g;
        const double g2 = wave_sum_d(own ? g * g : 0.0);
        if (t == 0) gram[(size_t)3 * blockIdx.x] = g2;
    }
}

hipError_t launch_reduce_m1(const Plan& pl, const float* gpart, double* g64, double* gram,
                            const Ctrl* ctrl, hipStream_t st) {
    hipLaunchKernelGGL(k_reduce_m1, dim3((unsigned)((pl.p + kRm1Rows - 1) / kRm1Rows)), dim3(1024), 0, st,
                       gpart, pl.npart, pl.ldx, (int)pl.p, g64, gram, ctrl);
    return hipGetLastError();
}

hipError_t launch_stop(const Plan& pl, const double* fpart, const int* nnzpart,
                       const double* gram, double* trace, double* coef, double* fcomp,
                       double* vprev, const double* g64, float* Xn, double* fsum, Ctrl* ctrl,
                       hipStream_t st) {
    if (pl.m > 1) {
        hipError_t e = launch_gram_sum(pl, 3 * pl.m * pl.m, pl.gram_blocks, gram, coef, ctrl, st,
                                       fpart, nnzpart, fsum);
        if (e != hipSuccess) return e;
    }
    if (pl.m == 1 && Xn) {
        hipLaunchKernelGGL(k_stop_x1, dim3(1), dim3(1024), 0, st, pl.nwave_part, fpart, nnzpart,
                           trace, coef, fcomp, gram, pl.gram_blocks, pl.exact, g64, Xn,
                           (int)pl.p, ctrl);
        return hipGetLastError();
    }
    // threads: the Jacobi steps of m = 64 have 32 x 32 blocks plus 64 x 32 rotated pairs of V;
    // m = 1 needs no eigen-solver: one wave makes every barrier free
    const int threads = pl.m > 1 ? jacobi_threads(pl.m) : 64;
    const size_t shm = (pl.m > 1) ? (size_t)retract_lds(pl.m) : 0;
    static const bool lds_once = (set_lds_limit((const void*)k_stop), true);
    (void)lds_once;
    hipLaunchKernelGGL(k_stop, dim3(1), dim3(threads), shm, st, pl.m, pl.nwave_part, fpart,
                       nnzpart, vprev, trace, coef, fcomp, gram, pl.gram_blocks, pl.exact,
                       g64, nullptr, (int)pl.p, fsum, ctrl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gamma path: m independent single-unit problems (column j has its own gamma).
// Per column: objective trace, stopping rule, and the sphere retraction
// x_j <- g_j / ||g_j||; a column whose rule fired is frozen (Psi_jj = 1), so
// its x, and with it S, F and Z, stay those of its stopping pass.
// fsum: objective and support size per column, summed by k_gram_sum in its own
// workgroups (summed here, by one workgroup from 2048 partials a column, this
// kernel took 11 us at m = 16 and 16 at m = 32 instead of 4.5 and 4.8).
__global__ __launch_bounds__(256) void k_stop_path(int m, double* __restrict__ trace,
                            double* __restrict__ coef, double* __restrict__ fcomp,
                            const double* __restrict__ fsum,
                            PathState* __restrict__ ps, Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ int nfrozen;
    const int t = threadIdx.x, nt = blockDim.x, mm = m * m;
    const int k = ctrl->k;
    const int max_iter = ctrl->max_iter;
    const double tol = ctrl->tol;
    if (t == 0) nfrozen = 0;
    for (int e = t; e < 2 * mm; e += nt) coef[e] = 0.0;  // Omega, Psi (the summed Gram is at 2mm)
    __syncthreads();
    for (int j = t; j < m; j += nt) {
        const double F = fsum[j];
        fcomp[j] = F;
        reinterpret_cast<int64_t*>(fcomp + m)[j] = (int64_t)fsum[m + j];
        PathState st = ps[j];
        if (!st.frozen) {
            trace[(size_t)j * max_iter + k] = F;
            int stop = 0, status = GPSPCA_OK;
            if (!isfinite(F)) {
                stop = 1;
                status = GPSPCA_ENONFINITE;
            } else if (F == 0.0) {
                stop = 1;
                st.degenerate = 1;
            } else if (k >= 1 && fabs(F - st.last_F) < tol * fabs(st.last_F)) {
                stop = 1;
            } else if (k + 1 >= max_iter) {
                stop = 1;
                status = GPSPCA_MAXITER;
            }
            if (stop) {
                st.frozen = 1;
                st.n_iter = k + 1;
                st.status = (status >= 0 && st.degenerate) ? GPSPCA_DEGENERATE : status;
            }
            st.last_F = F;
            ps[j] = st;
        }
        const double g2 = coef[2 * mm + (size_t)j * m + j];
        if (st.frozen) {
            coef[mm + j * m + j] = 1.0;
            atomicAdd(&nfrozen, 1);
        } else {
            coef[j * m + j] = 1.0 / sqrt(g2);
        }
    }
    __syncthreads();
    if (t == 0) {
        if (nfrozen == m) {
            ctrl->done = 1;
            ctrl->n_iter = k + 1;
        } else {
            ctrl->ndead = nfrozen > 0 ? 1 : 0;
            ctrl->k = k + 1;
        }
        ctrl->last_F = 0.0;
        ctrl->nact = 0;   // the next pass counts its active columns afresh
    }
}

hipError_t launch_stop_path(const Plan& pl, const double* fpart, const int* nnzpart,
                            const double* gram, double* trace, double* coef, double* fcomp,
                            double* fsum, PathState* ps, Ctrl* ctrl, hipStream_t st) {
    hipError_t e = launch_gram_sum(pl, pl.m * pl.m, pl.gram_blocks, gram, coef, ctrl, st, fpart,
                                   nnzpart, fsum);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_stop_path, dim3(1), dim3(256), 0, st, pl.m, trace, coef, fcomp, fsum, ps,
                       ctrl);
    return hipGetLastError();
}

// X[:, j] <- X[:, 0] for 1 <= j < m (rows < p)
__global__ void k_bcast_col0(int m, int p, int ldx, float* __restrict__ X) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)(m - 1) * p) return;
    const int j = 1 + (int)(e / p), r = (int)(e % p);
    X[(size_t)j * ldx + r] = X[r];
}

hipError_t launch_bcast_col0(const Plan& pl, float* X, hipStream_t st) {
    if (pl.m < 2) return hipSuccess;
    const int64_t ne = (int64_t)(pl.m - 1) * pl.p;
    hipLaunchKernelGGL(k_bcast_col0, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, pl.m,
                       (int)pl.p, pl.ldx, X);
    return hipGetLastError();
}

// Column-wise normalization of a starting point (gamma path): Omega =
// diag(1/||x_j||); a zero column fails with GPSPCA_EINVAL.
__global__ void k_project_diag(int m, double* __restrict__ coef, Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    const int t = threadIdx.x, mm = m * m;
    for (int e = t; e < 2 * mm; e += blockDim.x) coef[e] = 0.0;
    __syncthreads();
    for (int j = t; j < m; j += blockDim.x) {
        const double g2 = coef[2 * mm + (size_t)j * m + j];
        const double om = 1.0 / sqrt(g2);
        coef[j * m + j] = om;
        if (!(g2 > 0.0) || !isfinite(om)) {
            ctrl->status = GPSPCA_EINVAL;
            ctrl->done = 1;
        }
    }
    if (t == 0) ctrl->ndead = 0;
}

hipError_t launch_project_diag(const Plan& pl, const double* gram, double* coef, Ctrl* ctrl,
                               hipStream_t st) {
    hipError_t e = launch_gram_sum(pl, pl.m * pl.m, pl.gram_grid, gram, coef, ctrl, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_project_diag, dim3(1), dim3(256), 0, st, pl.m, coef, ctrl);
    return hipGetLastError();
}

// Projection of a starting point onto the feasible set: Omega = (G^T G)^{-1/2}
// (or 1/||g||); a rank-deficient start fails with GPSPCA_EINVAL.
__global__ __launch_bounds__(1024) void k_project(int m, double* __restrict__ coef, Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ StopShared ss;
    extern __shared__ double dyn[];
    double* A0 = dyn;
    // three matrices of m rows rounded up to even (jacobi_eig pads odd sizes)
    const int mr = m + (m & 1);
    double* A1 = dyn + (size_t)mr * LDM;
    double* A2 = dyn + (size_t)2 * mr * LDM;
    const int t = threadIdx.x, nt = blockDim.x, mm = m * m;
    if (m == 1) {
        if (t == 0) {
            const double g2 = coef[2];
            coef[0] = 1.0 / sqrt(g2);
            coef[1] = 0.0;
            if (!(g2 > 0.0) || !isfinite(coef[0])) {
                ctrl->status = GPSPCA_EINVAL;
                ctrl->done = 1;
            }
        }
        return;
    }
    if (newton_root<false>(m, coef + 2 * mm, coef, A0, ss.lam)) {
        for (int e = t; e < mm; e += nt) coef[mm + e] = 0.0;
        if (t == 0) {
            ctrl->ndead = 0;
            ctrl->warm = 0;
        }
        return;
    }
    for (int e = t; e < mm; e += nt) {
        const int i = e / m, j = e % m;
        A0[i * LDM + j] = coef[2 * mm + e];
    }
    __syncthreads();
    jacobi_eig(A0, A1, m, ss.rot);
    inv_sqrt_from_eig(A0, A1, A2, m, ss.lam, &ss.rankdef);
    for (int e = t; e < mm; e += nt) {
        const int i = e / m, j = e % m;
        coef[e] = A2[i * LDM + j];
        coef[mm + e] = 0.0;
    }
    if (t == 0) {
        ctrl->ndead = 0;
        ctrl->warm = 0;
        if (ss.rankdef) {
            ctrl->status = GPSPCA_EINVAL;
            ctrl->done = 1;
        }
    }
}

hipError_t launch_project(const Plan& pl, const double* gram, double* coef, Ctrl* ctrl,
                          hipStream_t st) {
    hipError_t e = launch_gram_sum(pl, pl.m * pl.m, pl.gram_grid, gram, coef, ctrl, st);
    if (e != hipSuccess) return e;
    const int threads = jacobi_threads(pl.m);
    const size_t shm = (pl.m > 1) ? (size_t)retract_lds(pl.m) : 0;
    static const bool lds_once = (set_lds_limit((const void*)k_project), true);
    (void)lds_once;
    hipLaunchKernelGGL(k_project, dim3(1), dim3(threads), shm, st, pl.m, coef, ctrl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// X_{k+1}[r, j] = sum_l G[r, l] Omega[l, j] + sum_l X_k[r, l] Psi[l, j]
// grid (row blocks of 256, columns j): one output element per thread.
__global__ __launch_bounds__(256) void k_apply(int m, int p, int ldx,
                                               const double* __restrict__ g64,
                                               const float* __restrict__ Xk,
                                               const double* __restrict__ coef,
                                               float* __restrict__ Xn,
                                               float* __restrict__ Xil, int diag,
                                               const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ double om[kMaxM];
    __shared__ double ps[kMaxM];
    const int t = threadIdx.x, j = blockIdx.y, mm = m * m;
    const bool dead = ctrl->ndead > 0;
    for (int l = t; l < m; l += 256) {
        om[l] = coef[l * m + j];
        ps[l] = dead ? coef[mm + l * m + j] : 0.0;
    }
    __syncthreads();
    const int r = blockIdx.x * 256 + t;
    if (r >= p) return;
    double acc = 0.0;
    int l = diag ? m : 0;  // gamma path: Omega and Psi are diagonal
    if (diag) {
        acc = g64[(size_t)j * p + r] * om[j];
        if (dead) acc += (double)Xk[(size_t)j * ldx + r] * ps[j];
    }
    for (; l + 4 <= m; l += 4) {  // in order of l, 4 loads issued together
        double gv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) gv[u] = g64[(size_t)(l + u) * p + r];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += gv[u] * om[l + u];
    }
    for (; l < m; ++l) acc += g64[(size_t)l * p + r] * om[l];
    if (dead && !diag)
        for (int l = 0; l < m; ++l) acc += (double)Xk[(size_t)l * ldx + r] * ps[l];
    Xn[(size_t)j * ldx + r] = (float)acc;
    if (Xil)
        Xil[((size_t)((j >> 4) * (ldx >> 2) + (r >> 2)) * 16 + (j & 15)) * 4 + (r & 3)] = (float)acc;
}

// The same for m > 16 (full Omega and Psi): grid (row blocks of 256, groups of
// 16 components); each thread reads its row of G once and keeps 16 outputs,
// summing over l in the same order as k_apply (bitwise the same result), so G
// is read m / 16 instead of m times.
__global__ __launch_bounds__(256) void k_apply16(int m, int p, int ldx,
                                                 const double* __restrict__ g64,
                                                 const float* __restrict__ Xk,
                                                 const double* __restrict__ coef,
                                                 float* __restrict__ Xn, float* __restrict__ Xil,
                                                 const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    __shared__ double om[kMaxM][16];
    __shared__ double ps[kMaxM][16];
    const int t = threadIdx.x, jb = blockIdx.y * 16, mm = m * m;
    const int nj = (m - jb < 16) ? m - jb : 16;
    const bool dead = ctrl->ndead > 0;
    for (int e = t; e < m * 16; e += 256) {
        const int l = e >> 4, jj = e & 15;
        const int j = jb + (jj < nj ? jj : nj - 1);
        om[l][jj] = coef[l * m + j];
        ps[l][jj] = dead ? coef[mm + l * m + j] : 0.0;
    }
    __syncthreads();
    const int r = blockIdx.x * 256 + t;
    if (r >= p) return;
    double acc[16];
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) acc[jj] = 0.0;
    int l = 0;
    for (; l + 4 <= m; l += 4) {  // 4 loads issued together
        double gv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) gv[u] = g64[(size_t)(l + u) * p + r];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) acc[jj] += gv[u] * om[l + u][jj];
    }
    for (; l < m; ++l) {
        const double gv = g64[(size_t)l * p + r];
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) acc[jj] += gv * om[l][jj];
    }
    if (dead)
        for (int l2 = 0; l2 < m; ++l2) {
            const double xv = (double)Xk[(size_t)l2 * ldx + r];
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) acc[jj] += xv * ps[l2][jj];
        }
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
        if (jj >= nj) break;
        const int j = jb + jj;
        const float v = (float)acc[jj];
        Xn[(size_t)j * ldx + r] = v;
        if (Xil)
            Xil[((size_t)((j >> 4) * (ldx >> 2) + (r >> 2)) * 16 + (j & 15)) * 4 + (r & 3)] = v;
    }
}

hipError_t launch_apply(const Plan& pl, const double* g64, const float* Xk, const double* coef,
                        float* Xn, float* Xil_n, const Ctrl* ctrl, hipStream_t st) {
    const int p = (int)pl.p;
    if (pl.m > 16 && !pl.path) {
        hipLaunchKernelGGL(k_apply16, dim3((p + 255) / 256, (pl.m + 15) / 16), dim3(256), 0, st,
                           pl.m, p, pl.ldx, g64, Xk, coef, Xn, Xil_n, ctrl);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_apply, dim3((p + 255) / 256, pl.m), dim3(256), 0, st, pl.m, p, pl.ldx,
                       g64, Xk, coef, Xn, Xil_n, pl.path, ctrl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Deflated single-unit components.  P = I - Q Q^T with Q (p x k, leading dim
// p, FP64) the earlier components.
//
// k_deflate: out = P x / ||P x|| in FP64 from FP64 x, to FP32; one workgroup
// of 1024 threads.  Every sum is a fixed-order butterfly
// within each wave followed by the 16 wave sums added in wave order, eight dot
// products per barrier.  P x = 0 gives 0 (the next pass then has F = 0 and
// stops).  scratch == x is allowed: each thread reads and writes only its
// own rows.

__global__ __launch_bounds__(1024) void k_deflate(int p, int k, const double* __restrict__ Q,
                                                  const double* x, float* __restrict__ out,
                                                  double* scratch,
                                                  const Ctrl* __restrict__ ctrl) {
    if (ctrl && ctrl->done) return;
    constexpr int NW = 16;
    __shared__ double wpart[8][NW];
    __shared__ double c[kMaxM + 1];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int j0 = 0; j0 < k; j0 += 8) {
        const int nj = (k - j0 < 8) ? k - j0 : 8;
        double d[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) d[u] = 0.0;
        // basis vectors past the last re-read vector j0 + nj - 1 (a valid
        // address) and are dropped by a select: the 8 loads are issued together
        size_t qo[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) qo[u] = (size_t)(j0 + (u < nj ? u : nj - 1)) * p;
        for (int r = t; r < p; r += 1024) {
            const double xr = x[r];
            double q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = Q[qo[u] + r];
#pragma unroll
            for (int u = 0; u < 8; ++u) d[u] += (u < nj) ? q[u] * xr : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double v = wave_sum_d(d[u]);
            if (lane == 0) wpart[u][w] = v;
        }
        __syncthreads();
        if (t < nj) {
            double v = 0.0;
            for (int i = 0; i < NW; ++i) v += wpart[t][i];
            c[j0 + t] = v;
        }
        __syncthreads();
    }
    double s2 = 0.0;
    for (int r = t; r < p; r += 1024) {
        double y = x[r];
        int j = 0;
        for (; j + 4 <= k; j += 4) {
            double q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = Q[(size_t)(j + u) * p + r];
#pragma unroll
            for (int u = 0; u < 4; ++u) y -= q[u] * c[j + u];
        }
        for (; j < k; ++j) y -= Q[(size_t)j * p + r] * c[j];
        scratch[r] = y;
        s2 += y * y;
    }
    s2 = wave_sum_d(s2);
    if (lane == 0) wpart[0][w] = s2;
    __syncthreads();
    if (t == 0) {
        double v = 0.0;
        for (int i = 0; i < NW; ++i) v += wpart[0][i];
        c[kMaxM] = v;
    }
    __syncthreads();
    const double nrm2 = c[kMaxM];
    const double inv = nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 0.0;
    for (int r = t; r < p; r += 1024) out[r] = (float)(scratch[r] * inv);
}

hipError_t launch_deflate(int p, int k, const double* Q, const double* x, float* out,
                          double* scratch, const Ctrl* ctrl, hipStream_t st) {
    hipLaunchKernelGGL(k_deflate, dim3(1), dim3(1024), 0, st, p, k, Q, x, out, scratch, ctrl);
    return hipGetLastError();
}

// k_defl_norms: ||P a_i|| = sqrt(||a_i||^2 - sum_j (q_j^T a_i)^2) in FP64 for
// every column of the FP32 matrix (one wave per column at a time; the column
// is read k + 1 times, from cache after the first): the default start of a
// deflated component.  Each lane sums its rows lane, lane + 64, ... in order;
// the loads of 8 such rows are issued together (rows past p re-read row p - 1
// and add 0), instead of one dependent load per row.
__global__ __launch_bounds__(256) void k_defl_norms(const float* __restrict__ A, int64_t lda,
                                                    int p, int64_t n, int k,
                                                    const double* __restrict__ Q,
                                                    double* __restrict__ norms) {
    constexpr int U = 8;
    const int lane = threadIdx.x & 63;
    const int64_t nw = (int64_t)gridDim.x * 4;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += nw) {
        const float* a = A + i * lda;
        double ss = 0.0;
        for (int r0 = lane; r0 < p; r0 += 64 * U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = r0 + 64 * u;
                v[u] = a[r < p ? r : p - 1];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) ss += (r0 + 64 * u < p) ? (double)v[u] * v[u] : 0.0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        double dd = 0.0;
        for (int j = 0; j < k; ++j) {
            const double* q = Q + (size_t)j * p;
            double d = 0.0;
            for (int r0 = lane; r0 < p; r0 += 64 * U) {
                float v[U];
                double qv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = r0 + 64 * u;
                    const int rc = r < p ? r : p - 1;
                    v[u] = a[rc];
                    qv[u] = q[rc];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) d += (r0 + 64 * u < p) ? qv[u] * v[u] : 0.0;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
            dd += d * d;
        }
        if (lane == 0) norms[i] = sqrt(fmax(ss - dd, 0.0));
    }
}

hipError_t launch_defl_norms(const float* A, int64_t lda, int p, int64_t n, int k,
                             const double* Q, double* norms, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_defl_norms, dim3(grid), dim3(256), 0, st, A, lda, p, n, k, Q, norms);
    return hipGetLastError();
}

// Q[:, k] = x (FP32 -> FP64)
__global__ void k_append_basis(int p, const float* __restrict__ x, double* __restrict__ q) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r < p) q[r] = (double)x[r];
}

hipError_t launch_append_basis(int p, const float* x, double* q, hipStream_t st) {
    hipLaunchKernelGGL(k_append_basis, dim3((p + 255) / 256), dim3(256), 0, st, p, x, q);
    return hipGetLastError();
}

// One thread per (block, quad, component): a 16-byte vector of 4 rows.
__global__ __launch_bounds__(256) void k_x_interleave(int mpad, int ldx,
                                                      const float* __restrict__ X,
                                                      float* __restrict__ Xil) {
    const int nq = ldx >> 2;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)nq * mpad) return;
    const int c = (int)(e % 16);
    const int64_t bq = e / 16;             // b * nq + q
    const int q = (int)(bq % nq), b = (int)(bq / nq);
    const float4 v = *reinterpret_cast<const float4*>(X + (size_t)(16 * b + c) * ldx + 4 * q);
    *reinterpret_cast<float4*>(Xil + (size_t)e * 4) = v;
}

hipError_t launch_x_interleave(const Plan& pl, const float* X, float* Xil, hipStream_t st) {
    const int64_t ne = (int64_t)(pl.ldx / 4) * pl.mpad;
    hipLaunchKernelGGL(k_x_interleave, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st,
                       pl.mpad, pl.ldx, X, Xil);
    return hipGetLastError();
}

// g64[j*p + r] = X0[j*ldx0 + r]
__global__ void k_load_g64(int m, int p, const float* __restrict__ X0, int ldx0,
                           double* __restrict__ g64) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)m * p) return;
    const int j = (int)(e / p), r = (int)(e % p);
    g64[e] = (double)X0[(size_t)j * ldx0 + r];
}

hipError_t launch_load_g64(const Plan& pl, const float* X0, int ldx0, double* g64,
                           hipStream_t st) {
    const int64_t ne = (int64_t)pl.m * pl.p;
    hipLaunchKernelGGL(k_load_g64, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, pl.m,
                       (int)pl.p, X0, ldx0, g64);
    return hipGetLastError();
}

}  // namespace gpspca
