// k_small: every pass of a solve on a small matrix in one launch.
//
// On a small matrix a pass is latency: 3 to 6 launches of 4-16 us each, while
// its arithmetic takes one.  Here nb <= 64 workgroups of 8 waves hold their
// columns in LDS (FP32, what 146 KB leave beside the other arrays: up to about 135
// KB each, 8.5 MB in all) for the whole solve and meet at grid barriers.  A read from L2 instead is bound by the 64
// bytes per clock of a CU's cache: at 400 x 4000 it took 25 us per pass against 12.
//
//   1  y = A^T X and the threshold for the workgroup's tiles of 16 columns, then
//      its partial of G = A S N over the tiles with an active column; m = 1 by
//      vector FMAs, more components on v_mfma_f32_16x16x4_f32
//   -  barrier
//   2  the partials of G summed in FP64 in a fixed order: every workgroup all of
//      G when that is little to read (one barrier per pass), else each a share
//      that it writes back, with a second barrier before all of G is read
//   3  in every workgroup alike: the objective, the stopping rule and the
//      retraction (m = 1 and gamma paths: g / ||g||, deflated: P g / ||P g||,
//      blocks: the polar factor, its small matrices on one wave), X_{k+1}
//      into LDS.  Equal inputs in equal order give every workgroup the same X
//      and the same decision, so neither has to be communicated.
//
// Sums are FP32 over 8 to 16 rows (4 to 16 columns) and FP64 above that, so that
// the results are as close to FP64 as those of the separate launches, whose
// chains are shorter than a workgroup's here: with FP32 alone the X and Z of a
// pass were 1.1 to 2 times further off.  It costs 1.3 us per pass at 200 x 2000,
// m = 5, and 0.2 at m = 1.
//
// Per pass, as separate launches -> here: 100 x 1000, m = 1: 20 -> 8 us; 200 x 2000,
// m = 5: 56 -> 22; 400 x 4000, m = 1, deflated: 27 -> 13.  What is left is the
// latency of the barrier (1.5-3 us), of reading the partials (2-4) and of the
// dependent steps in between.
//
// What the workgroups exchange (partials, objective terms, G) goes through
// device-scope relaxed atomic stores and loads, which write through and read
// past the XCDs' L2 caches; each wave waits for its stores to be acknowledged
// before its workgroup's arrival is counted.  So no cache is written back or
// invalidated: with acquire / release fences two barriers cost 45 us.
//
// The barriers need every workgroup resident.  The host admits no more
// workgroups of such solves at once than the CUs of each XCD can hold, one per
// CU, and none on a stream that is kept off some CUs (gpspca_abi.cpp), and a wait that lasts 100 ms ends the kernel
// with Ctrl::abort set: the host then runs the passes as separate launches, and
// the thread's next solves as well.
#include "corr.h"
#include "gpspca_internal.h"
#include "retract.h"
#include "storage.h"

#include <algorithm>

namespace gpspca {

static_assert(offsetof(Ctrl, bar) % 8 == 0 && offsetof(Ctrl, abort) == offsetof(Ctrl, bar) + 4,
              "read as one word");

namespace {

typedef float f4c __attribute__((ext_vector_type(4)));
typedef float f4cu __attribute__((ext_vector_type(4), aligned(4)));
typedef double d4c __attribute__((ext_vector_type(4)));

constexpr int kSmT = 512, kSmW = 8;
constexpr int kSmallLds = 146 * 1024;       // dynamic LDS of a workgroup

template <typename T>
__device__ __forceinline__ void put(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T get(const T* p) {
    return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct SmallArgs {
    float* x0;
    float* x1;
    float* S;
    float* gpart;
    double* fpart;
    int* nnzpart;
    double* g64;
    double* trace;
    double* vprev;
    PathState* ps;
    Ctrl* ctrl;
    const double* Q;
    int defl_k, exact, path, nb, whole, passes;
    uint32_t bar0;      // arrivals counted by earlier launches of the solve
    int64_t wait;       // limit of a barrier's wait, in ticks of the 100 MHz clock
};

// LDS of a workgroup, in bytes (offsets from the start).
struct SmallLds {
    int a, sq, g, jac, coef, x, gp, w, act, total;
};

__host__ __device__ inline SmallLds small_lds(int p, int m, int path, int64_t n, int nb) {
    SmallLds L;
    const int nq4 = ((p + 3) / 4 + 3) / 4 * 4;
    const int64_t ntile = (n + 15) / 16;
    const int tw = (int)((ntile + nb - 1) / nb);
    const bool block = m > 1 && !path;
    L.sq = nq4 | 1;   // odd: 16 columns' quads at one row fall on different banks
    int o = 0;
    L.a = o;    o += 16 * L.sq * 16 * tw;
    L.g = o;    o += 8 * p * m;
    L.jac = o;  o += block ? retract_lds(m) : 0;
    L.coef = o; o += block ? 6 * m * m * 8 : 0;
    L.x = o = (o + 15) / 16 * 16; o += 16 * nq4 * m;
    L.gp = o;   o += m == 1 ? 16 * kSmT : 4 * kSmW * 64 * m;
    L.w = o;    o += 4 * tw * 16 * m;
    L.act = o;  o += 4 * tw;
    L.total = (o + 15) / 16 * 16;
    return L;
}

// Rows 4q .. 4q+3 of a column; rows past p are 0.
template <int ST>
__device__ __forceinline__ f4c quad_full(const void* colv, int q) {
    if constexpr (ST == kStF32)
        return *reinterpret_cast<const f4cu*>(static_cast<const float*>(colv) + 4 * q);
    else {
        const qf4 v = load_quad_st<ST>(colv, q, q + 1, 4 * q + 4);
        return f4c{v.x, v.y, v.z, v.w};
    }
}
template <int ST>
__device__ __forceinline__ f4c quad_edge(const void* colv, int q, int nqf, int p) {
    if (q < nqf) return quad_full<ST>(colv, q);
    if (4 * q >= p) return f4c{0.f, 0.f, 0.f, 0.f};
    if constexpr (ST == kStF32) {
        const float* c = static_cast<const float*>(colv) + 4 * q;
        f4c v = f4c{c[0], 0.f, 0.f, 0.f};
        if (4 * q + 1 < p) v.y = c[1];
        if (4 * q + 2 < p) v.z = c[2];
        return v;
    } else {
        const qf4 v = load_quad_st<ST>(colv, q, nqf, p);
        return f4c{v.x, v.y, v.z, v.w};
    }
}

// Every wave's stores acknowledged, then every workgroup's arrival.  False when
// the wait ran out (the same answer for every thread of the workgroup).
__device__ bool grid_barrier(Ctrl* ctrl, uint32_t target, int64_t limit, int* flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(&ctrl->bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int64_t began = wall_clock64();
        int ok = 1;
        for (;;) {
            // arrivals and the abort flag in one read
            const uint64_t v = get(reinterpret_cast<const uint64_t*>(&ctrl->bar));
            if ((int32_t)((uint32_t)v - target) >= 0) break;
            if ((v >> 32) || wall_clock64() - began > limit) {
                put(&ctrl->abort, 1);
                ok = 0;
                break;
            }
        }
        *flag = ok;
    }
    __syncthreads();
    return *flag != 0;
}

template <int ST, int MB, bool BLOCK>
__global__ __launch_bounds__(kSmT, 2) void k_small(PassParams pp, SmallArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ StopShared ss;
    __shared__ Ctrl lc;                    // this workgroup's copy of the control block
    __shared__ PathState lps[16];
    __shared__ double fw[kSmW][16];        // objective terms of the waves, then sums
    __shared__ int nw[kSmW][16];
    __shared__ double red[kSmT];
    __shared__ double nrm[kMaxM + 1];
    __shared__ int flag, sfrozen;

    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int lj = lane & 15, lk = lane >> 4;
    const int m = pp.m, p = pp.p, ldx = pp.ldx, nb = a.nb, wg = blockIdx.x;
    const int64_t n = pp.n;
    const SmallLds L = small_lds(p, m, a.path, n, nb);
    f4c* const Al = reinterpret_cast<f4c*>(lds + L.a);         // [column][quad], stride L.sq
    double* const Gd = reinterpret_cast<double*>(lds + L.g);
    double* const jac = reinterpret_cast<double*>(lds + L.jac);
    double* const coef = reinterpret_cast<double*>(lds + L.coef);
    float* const Xl = reinterpret_cast<float*>(lds + L.x);     // [quad][component][4]
    float* const gp = reinterpret_cast<float*>(lds + L.gp);    // [wave][component][64 rows]
    float* const Sw = reinterpret_cast<float*>(lds + L.w);     // [column][component]
    uint32_t* const actm = reinterpret_cast<uint32_t*>(lds + L.act);

    if (t == 0) lc = *a.ctrl;
    __syncthreads();
    if (lc.done) return;
    const int64_t ntile = (n + 15) / 16;
    const int64_t tb = ntile * wg / nb, te = ntile * (wg + 1) / nb;
    const int tw = (int)(te - tb);
    const int nqf = p >> 2, nq = (p + 3) >> 2;
    const int nq4 = (nq + 3) / 4 * 4;
    const int nsteps = nq4 / 4, sq = L.sq;
    const bool l0 = pp.l0 != 0;
    const int cj = lj < m ? lj : m - 1;
    const float muj = pp.muf[cj];
    const double mud = pp.mu[cj], gamd = pp.gam[cj];
    const int mm = m * m;
    const int k0 = lc.k;

    // this workgroup's columns, as FP32, for the whole solve; zero past p and n
    for (int e = t; e < tw * 16 * sq; e += kSmT) {
        const int c = e / sq, q = e - c * sq;
        const int64_t col = 16 * tb + c;
        Al[e] = col < n && q < nq ? quad_edge<ST>(column_ptr<ST>(pp, col), q, nqf, p)
                                  : f4c{0.f, 0.f, 0.f, 0.f};
    }
    {
        const float* xk = (k0 & 1) ? a.x1 : a.x0;
        for (int e = t; e < 4 * nq4 * m; e += kSmT) {
            const int r = (e / (4 * m)) * 4 + (e & 3), j = (e >> 2) % m;
            Xl[e] = r < p ? xk[(size_t)j * ldx + r] : 0.f;
        }
        if (a.path)
            for (int j = t; j < m; j += kSmT) lps[j] = a.ps[j];
        else if (lc.warm)
            for (int e = t; e < mm; e += kSmT) coef[5 * mm + e] = a.vprev[e];
    }
    __syncthreads();

    uint32_t arrived = a.bar0;
    bool stop = false;
    int k = k0;
    for (int pass = 0; pass < a.passes; ++pass) {
        // With one barrier per pass a workgroup may write its next partials while
        // another still reads these: two sets, in turn.  (With two barriers, the
        // second has every reader past them.)
        const int set = a.whole ? pass & 1 : 0;
        float* const gpart = a.gpart + (size_t)set * nb * m * ldx;
        double* const fpart = a.fpart + (size_t)set * nb * m;
        int* const nnzpart = a.nnzpart + (size_t)set * nb * m;
        // ---- 1: correlation and threshold of this workgroup's tiles
        double f_acc = 0.0;
        int nnz_acc = 0;
        if (m == 1) {
            // vector FMAs: a lane takes every fourth quad of one column; with fewer
            // tiles than waves, several waves share a tile's rows
            const int parts = tw < kSmW ? kSmW / (tw > 0 ? tw : 1) : 1;
            for (int i = wv; i < tw * parts; i += kSmW) {
                const int tl = i % tw, part = i / tw;
                const f4c* ac = Al + (tl * 16 + lj) * sq + lk;
                const int sa = nsteps * part / parts, sz = nsteps * (part + 1) / parts;
                double yd = 0.0;
#pragma unroll 2
                for (int s0 = sa; s0 < sz; s0 += 4) {   // 4 quads per FP32 sum
                    f4c acc = f4c{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool in = s0 + u < sz;
                        const int s = in ? s0 + u : sz - 1;
                        const f4c x = *reinterpret_cast<const f4c*>(Xl + 4 * (4 * s + lk));
                        const f4c av = ac[4 * s];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[e] = __builtin_fmaf(in ? av[e] : 0.f, x[e], acc[e]);
                    }
                    yd += (double)((acc[0] + acc[1]) + (acc[2] + acc[3]));
                }
                yd += __shfl_xor(yd, 16, 64);
                yd += __shfl_xor(yd, 32, 64);
                // at most 128 partial sums, or one per column
                if (lk == 0 && parts > 1)
                    reinterpret_cast<double*>(gp)[(tl * 16 + lj) * parts + part] = yd;
                else if (lk == 0)
                    gp[tl * 16 + lj] = (float)yd;
            }
            __syncthreads();
            for (int c = t; c < tw * 16; c += kSmT) {
                float y;
                if (parts > 1) {
                    const double* yp = reinterpret_cast<const double*>(gp) + c * parts;
                    double yd = yp[0];
                    for (int i = 1; i < parts; ++i) yd += yp[i];
                    y = (float)yd;
                } else {
                    y = gp[c];
                }
                float s = 0.f;
                const int64_t col = 16 * tb + c;
                if (col < n) {
                    const float sc = ST == kStF32 ? 1.0f : column_scale(pp, col);
                    double fv;
                    if (threshold(l0, mud, gamd, ST == kStF32 ? y : sc * y, s, fv)) {
                        f_acc += fv;
                        nnz_acc += 1;
                    }
                }
                Sw[c] = s;
            }
            f_acc = wave_sum_s(f_acc);
            nnz_acc = wave_sum_s(nnz_acc);
        } else {
        for (int tl = wv; tl < tw; tl += kSmW) {
            const int64_t c0 = 16 * (tb + tl);
            const f4c* ac = Al + (tl * 16 + lj) * sq + lk;
            d4c tot = d4c{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
            for (int s = 0; s < nsteps; ++s) {   // 8 rows per FP32 sum
                const f4c x = *reinterpret_cast<const f4c*>(Xl + 4 * ((4 * s + lk) * m + cj));
                const f4c av = ac[4 * s];
                f4c c[2];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    c[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        av[e], x[e], e < 2 ? f4c{0.f, 0.f, 0.f, 0.f} : c[e & 1], 0, 0, 0);
                tot += __builtin_convertvector(c[0] + c[1], d4c);
            }
            const f4c y = __builtin_convertvector(tot, f4c);
            uint32_t mask = 0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t c = c0 + 4 * lk + v;
                bool on = false;
                if (lj < m) {
                    float s = 0.f;
                    if (c < n) {
                        const float sc = ST == kStF32 ? 1.0f : column_scale(pp, c);
                        double fv;
                        on = threshold(l0, mud, gamd, ST == kStF32 ? y[v] : sc * y[v],
                                         s, fv);
                        if (on) {
                            f_acc += fv;
                            nnz_acc += 1;
                        }
                    }
                    Sw[(tl * 16 + 4 * lk + v) * m + lj] = s;
                }
                const uint64_t b = __ballot(on);
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if ((b >> (16 * g)) & 0xFFFFull) mask |= 1u << (4 * g + v);
            }
            if (lane == 0) actm[tl] = mask;
        }
        f_acc += __shfl_xor(f_acc, 16, 64);
        nnz_acc += __shfl_xor(nnz_acc, 16, 64);
        f_acc += __shfl_xor(f_acc, 32, 64);
        nnz_acc += __shfl_xor(nnz_acc, 32, 64);
        }
        if (lane < 16) {
            fw[wv][lane] = f_acc;
            nw[wv][lane] = nnz_acc;
        }
        __syncthreads();
        if (t < m) {
            double f = 0.0;
            int c = 0;
            for (int w = 0; w < kSmW; ++w) {
                f += fw[w][t];
                c += nw[w][t];
            }
            if (nb > 1) {
                put(fpart + (size_t)t * nb + wg, f);
                put(nnzpart + (size_t)t * nb + wg, c);
            } else {
                ss.fj[t] = f;
                ss.nj[t] = c;
            }
        }

        // ---- 1b: this workgroup's partial of G
        if (m == 1) {
            // a thread takes a quad of rows of a range of columns
            const int nsp = nq < kSmT ? (kSmT / nq < 8 ? kSmT / nq : 8) : 1;
            for (int q0 = 0; q0 < nq; q0 += kSmT) {
                const int q = nsp > 1 ? t % nq : q0 + t, sp = nsp > 1 ? t / nq : 0;
                if (q < nq && sp < nsp) {
                    d4c tot = d4c{0.0, 0.0, 0.0, 0.0};
                    const int ca = tw * 16 * sp / nsp, cz = tw * 16 * (sp + 1) / nsp;
                    for (int c0 = ca; c0 < cz; c0 += 8) {   // 4 columns per FP32 sum
                        f4c g[2];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            if (u % 4 == 0) g[u / 4] = f4c{0.f, 0.f, 0.f, 0.f};
                            const int c = c0 + u < cz ? c0 + u : cz - 1;
                            const float sw = c0 + u < cz ? Sw[c] : 0.f;
                            float w = muj * sw;
                            if constexpr (ST != kStF32) {
                                const int64_t col = 16 * tb + c;
                                w *= column_scale(pp, col < n ? col : n - 1);
                            }
                            // an inactive column has weight 0 and may hold anything
                            const f4c av = Al[c * sq + q];
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                g[u / 4][e] = __builtin_fmaf(w, sw != 0.f ? av[e] : 0.f, g[u / 4][e]);
                        }
                        tot += __builtin_convertvector(g[0], d4c) + __builtin_convertvector(g[1], d4c);
                    }
                    *reinterpret_cast<f4c*>(gp + 4 * (nsp > 1 ? sp * nq + q : t)) =
                        __builtin_convertvector(tot, f4c);
                }
                __syncthreads();
                const int len = nsp > 1 ? 4 * nq : 4 * (nq - q0 < kSmT ? nq - q0 : kSmT);
                for (int e = t; e < len; e += kSmT) {
                    const int r = 4 * q0 + e;
                    float v[8];
                    double g = 0.0;
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = gp[(i < nsp ? i : 0) * 4 * nq + e];
#pragma unroll
                    for (int i = 0; i < 8; ++i) g += i < nsp ? (double)v[i] : 0.0;
                    if (r < p) {
                        if (nb > 1) put(gpart + (size_t)wg * ldx + r, (float)g);
                        else Gd[r] = g;
                    }
                }
                __syncthreads();
            }
        } else {
        // matrix cores, 64 rows per wave; with fewer row blocks than waves the tiles
        // are split over csp waves
        const int nrb = (p + 63) / 64;
        const int csp = nrb < kSmW ? kSmW / nrb : 1;
        for (int rb0 = 0; rb0 < nrb; rb0 += kSmW) {
            const int rb = csp > 1 ? wv % nrb : rb0 + wv;
            const int cs = csp > 1 ? wv / nrb : 0;
            if (rb < nrb && cs < csp) {
                const int ta = tw * cs / csp, tz = tw * (cs + 1) / csp;
                const int q = 16 * rb + lj < sq ? 16 * rb + lj : sq - 1;   // rows past p are dropped
                d4c tot[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) tot[e] = d4c{0.0, 0.0, 0.0, 0.0};
                for (int t0 = ta; t0 < tz; t0 += 2) {   // 16 columns per FP32 sum
                    f4c acc[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[h][e] = f4c{0.f, 0.f, 0.f, 0.f};
                        const int tl = t0 + h;
                        if (tl >= tz) continue;
                        const uint32_t mask = __builtin_amdgcn_readfirstlane(actm[tl]);
                        if (mask == 0) continue;
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const int c = tl * 16 + 4 * g + lk;
                            // an inactive column has weight 0 and may hold anything
                            const bool in = (mask >> (4 * g + lk)) & 1u;
                            const f4c av = Al[c * sq + q];
                            float w = muj * Sw[c * m + cj];
                            if constexpr (ST != kStF32) {
                                const int64_t col = 16 * tb + c;
                                w *= column_scale(pp, col < n ? col : n - 1);
                            }
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[h][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    in ? av[e] : 0.f, w, acc[h][e], 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        tot[e] += __builtin_convertvector(acc[0][e] + acc[1][e], d4c);
                }
                if (lj < m) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            gp[(wv * m + lj) * 64 + 16 * lk + 4 * v + e] = (float)tot[e][v];
                }
            }
            __syncthreads();
            const int nr = csp > 1 ? nrb : (nrb - rb0 < kSmW ? nrb - rb0 : kSmW);
            for (int e = t; e < nr * m * 64; e += kSmT) {
                const int row = e & 63, j = (e >> 6) % m, b = (e >> 6) / m;
                const int r = 64 * (rb0 + b) + row;
                if (r >= p) continue;
                float v[kSmW];
                double g = 0.0;
#pragma unroll
                for (int c = 0; c < kSmW; ++c)
                    v[c] = gp[(((c < csp ? c : 0) * nrb + b) * m + j) * 64 + row];
#pragma unroll
                for (int c = 0; c < kSmW; ++c) g += c < csp ? (double)v[c] : 0.0;
                if (nb > 1) put(gpart + ((size_t)wg * m + j) * ldx + r, (float)g);
                else Gd[j * p + r] = g;
            }
            __syncthreads();
        }
        }

        // ---- 2: G summed over the workgroups
        if (nb > 1) {
            arrived += nb;
            if (!grid_barrier(a.ctrl, arrived, a.wait, &flag)) return;
            const int cnt = p * m;
            const int e0 = a.whole ? 0 : (int)((int64_t)cnt * wg / nb);
            const int e1 = a.whole ? cnt : (int)((int64_t)cnt * (wg + 1) / nb);
            const int len = e1 - e0;
            int nsl = len > 0 && len < kSmT ? kSmT / len : 1;
            nsl = nsl < nb ? nsl : nb;
            // objective terms: component j's by one wave (fixed order); the first
            // loads are in flight with those of the partials
            double f0 = 0.0;
            int c0 = 0;
            if (wv < m && lane < nb) {
                f0 = get(fpart + (size_t)wv * nb + lane);
                c0 = get(nnzpart + (size_t)wv * nb + lane);
            }
            for (int b0 = 0; b0 < len; b0 += kSmT) {
                const int idx = nsl > 1 ? t % len : b0 + t;
                const int sl = nsl > 1 ? t / len : 0;
                double s = 0.0;
                if (idx < len && sl < nsl) {
                    const int e = e0 + idx, j = e / p, r = e % p;
                    const int w0 = nb * sl / nsl, w1 = nb * (sl + 1) / nsl;
                    const float* src = gpart + (size_t)j * ldx + r;
                    for (int w = w0; w < w1; w += 16) {
                        float v[16];
#pragma unroll
                        for (int u = 0; u < 16; ++u) {
                            const int wc = w + u < w1 ? w + u : w1 - 1;
                            v[u] = get(src + (size_t)wc * m * ldx);
                        }
#pragma unroll
                        for (int u = 0; u < 16; ++u) s += w + u < w1 ? (double)v[u] : 0.0;
                    }
                }
                if (nsl > 1) {
                    red[t] = s;
                    __syncthreads();
                    if (t < len)
                        for (int u = 1; u < nsl; ++u) s += red[u * len + t];
                }
                if (idx < len && sl == 0) {
                    if (a.whole) Gd[e0 + idx] = s;
                    else put(a.g64 + e0 + idx, s);
                }
                if (nsl > 1) break;
            }
            for (int j = wv; j < m; j += kSmW) {
                if (j != wv) {
                    f0 = lane < nb ? get(fpart + (size_t)j * nb + lane) : 0.0;
                    c0 = lane < nb ? get(nnzpart + (size_t)j * nb + lane) : 0;
                }
                const double f = wave_sum_s(f0);
                const int c = wave_sum_s(c0);
                if (lane == 0) {
                    ss.fj[j] = f;
                    ss.nj[j] = c;
                }
            }
            if (!a.whole) {
                arrived += nb;
                if (!grid_barrier(a.ctrl, arrived, a.wait, &flag)) return;
                for (int b0 = t; b0 < cnt; b0 += 8 * kSmT) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int e = b0 + u * kSmT;
                        v[u] = get(a.g64 + (e < cnt ? e : cnt - 1));
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (b0 + u * kSmT < cnt) Gd[b0 + u * kSmT] = v[u];
                }
            }
        }
        __syncthreads();

        // ---- 3: objective, stopping rule
        if (a.path) {
            if (t == 0) sfrozen = 0;
            __syncthreads();
            if (t < m) {
                PathState st = lps[t];
                const double F = ss.fj[t];
                if (!st.frozen) {
                    if (wg == 0) a.trace[(size_t)t * lc.max_iter + k] = F;
                    int halt = 0, status = GPSPCA_OK;
                    if (!isfinite(F)) {
                        halt = 1;
                        status = GPSPCA_ENONFINITE;
                    } else if (F == 0.0) {
                        halt = 1;
                        st.degenerate = 1;
                    } else if (k >= 1 && fabs(F - st.last_F) < lc.tol * fabs(st.last_F)) {
                        halt = 1;
                    } else if (k + 1 >= lc.max_iter) {
                        halt = 1;
                        status = GPSPCA_MAXITER;
                    }
                    if (halt) {
                        st.frozen = 1;
                        st.n_iter = k + 1;
                        st.status = (status >= 0 && st.degenerate) ? GPSPCA_DEGENERATE : status;
                    }
                    st.last_F = F;
                    lps[t] = st;
                }
                if (st.frozen) atomicAdd(&sfrozen, 1);
            }
            __syncthreads();
            if (t == 0) {
                ss.stop = sfrozen == m;
                if (ss.stop) {
                    lc.done = 1;
                    lc.n_iter = k + 1;
                }
                lc.last_F = 0.0;
            }
        } else if (t == 0) {
            double F = 0.0;
            int nl = 0, nd = 0;
            for (int j = 0; j < m; ++j) {
                const double fj = ss.fj[j];
                F += a.exact ? sqrt(fj) : fj;
                ss.dsc[j] = (a.exact && fj > 0.0) ? 1.0 / sqrt(fj) : 0.0;
                if (ss.nj[j] > 0) ss.live[nl++] = j;
                else ss.dead[nd++] = j;
            }
            ss.nlive = nl;
            ss.ndead = nd;
            if (wg == 0) a.trace[k] = F;
            int halt = 0, status = GPSPCA_OK;
            int degenerate = lc.degenerate_seen;
            if (!isfinite(F)) {
                halt = 1;
                status = GPSPCA_ENONFINITE;
            } else if (F == 0.0) {
                halt = 1;
                degenerate = 1;
                lc.degenerate_seen = 1;
            } else if (k >= 1 && fabs(F - lc.last_F) < lc.tol * fabs(lc.last_F)) {
                halt = 1;
            } else if (k + 1 >= lc.max_iter) {
                halt = 1;
                status = GPSPCA_MAXITER;
            }
            if (halt) {
                if (status >= 0 && degenerate) status = GPSPCA_DEGENERATE;
                lc.status = status;
                lc.done = 1;
                lc.n_iter = k + 1;
            }
            lc.last_F = F;
            ss.stop = halt;
        }
        __syncthreads();
        if (ss.stop) {
            stop = true;
            break;
        }

        // ---- 3b: retraction
        if constexpr (!BLOCK) {   // m = 1 or a path
            if (a.defl_k > 0) {
                // g <- P g, P = I - Q Q^T: the dot products first, then the update
                for (int j = wv; j < a.defl_k; j += kSmW) {
                    double d = 0.0;
                    for (int r = lane; r < p; r += 64) d += a.Q[(size_t)j * p + r] * Gd[r];
                    d = wave_sum_s(d);
                    if (lane == 0) nrm[j] = d;
                }
                __syncthreads();
                for (int r = t; r < p; r += kSmT) {
                    double y = Gd[r];
                    for (int j = 0; j < a.defl_k; ++j) y -= a.Q[(size_t)j * p + r] * nrm[j];
                    Gd[r] = y;
                }
                __syncthreads();
            }
            for (int j = wv; j < m; j += kSmW) {
                double s = 0.0;
                for (int r = lane; r < p; r += 64) {
                    const double g = Gd[j * p + r];
                    s += g * g;
                }
                s = wave_sum_s(s);
                if (lane == 0) nrm[j] = s;
            }
            __syncthreads();
            if (!a.path) {
                const double g2 = nrm[0], om = 1.0 / sqrt(g2);
                if (a.defl_k == 0 && (!(g2 > 0.0) || !isfinite(om))) {
                    if (t == 0) {
                        lc.status = GPSPCA_ENONFINITE;
                        lc.done = 1;
                        lc.n_iter = k + 1;
                    }
                    __syncthreads();
                    stop = true;
                    break;
                }
                // a deflated direction that vanishes leaves x = 0: the next pass has F = 0
                const double sc = g2 > 0.0 ? om : 0.0;
                for (int r = t; r < p; r += kSmT) Xl[4 * (r >> 2) + (r & 3)] = (float)(Gd[r] * sc);
            } else {
                for (int e = t; e < p * m; e += kSmT) {
                    const int j = e / p, r = e % p;
                    if (!lps[j].frozen)
                        Xl[4 * ((r >> 2) * m + j) + (r & 3)] =
                            (float)(Gd[e] * (1.0 / sqrt(nrm[j])));
                }
            }
        } else {
            // G^T G, and with a dead component G^T X and X^T X: one entry per wave
            const int np = m * (m + 1) / 2;
            for (int e = wv; e < np; e += kSmW) {
                int i = 0, rem = e;
                while (rem >= m - i) {
                    rem -= m - i;
                    ++i;
                }
                const int j = i + rem;
                double s = 0.0;
                for (int r = lane; r < p; r += 64) s += Gd[i * p + r] * Gd[j * p + r];
                s = wave_sum_s(s);
                if (lane == 0) coef[2 * mm + i * m + j] = coef[2 * mm + j * m + i] = s;
            }
            if (ss.ndead > 0) {
                for (int e = wv; e < mm; e += kSmW) {
                    const int i = e / m, j = e % m;
                    double s = 0.0, x = 0.0;
                    for (int r = lane; r < p; r += 64) {
                        const double xj = (double)Xl[4 * ((r >> 2) * m + j) + (r & 3)];
                        s += Gd[i * p + r] * xj;
                        x += (double)Xl[4 * ((r >> 2) * m + i) + (r & 3)] * xj;
                    }
                    s = wave_sum_s(s);
                    x = wave_sum_s(x);
                    if (lane == 0) {
                        coef[3 * mm + e] = s;
                        coef[4 * mm + e] = x;
                    }
                }
            }
            __syncthreads();
            if (wv == 0) {
                if (a.exact) {
                    for (int e = lane; e < mm; e += 64) {
                        coef[2 * mm + e] *= ss.dsc[e / m] * ss.dsc[e % m];
                        if (ss.ndead > 0) coef[3 * mm + e] *= ss.dsc[e / m];
                    }
                    group_sync<true>();
                }
                const int mr = m + (m & 1);
                block_coefficients<true>(m, coef, coef + 5 * mm, ss, jac, jac + mr * LDM,
                                         jac + 2 * mr * LDM, &lc);
                int bad = 0;
                for (int e = lane; e < mm; e += 64) {
                    if (a.exact) coef[e] *= ss.dsc[e / m];
                    bad |= isfinite(coef[e]) && isfinite(coef[mm + e]) ? 0 : 1;
                }
                if (__any(bad) && lane == 0) {
                    lc.status = GPSPCA_ENONFINITE;
                    lc.done = 1;
                    lc.n_iter = k + 1;
                    lc.warm = 0;
                }
            }
            __syncthreads();
            if (lc.done) {
                stop = true;
                break;
            }
            const bool dead = lc.ndead > 0;
            for (int r = t; r < p; r += kSmT) {
                double gv[MB], xo[MB];
                float* const xr = Xl + 4 * (r >> 2) * m + (r & 3);
#pragma unroll
                for (int l = 0; l < MB; ++l) {
                    const int lc_ = l < m ? l : m - 1;
                    gv[l] = Gd[lc_ * p + r];
                    xo[l] = dead ? (double)xr[4 * lc_] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < MB; ++j) {
                    if (j >= m) continue;
                    double s = 0.0;
#pragma unroll
                    for (int l = 0; l < MB; ++l) s += l < m ? gv[l] * coef[l * m + j] : 0.0;
                    if (dead) {
#pragma unroll
                        for (int l = 0; l < MB; ++l) s += l < m ? xo[l] * coef[mm + l * m + j] : 0.0;
                    }
                    xr[4 * j] = (float)s;
                }
            }
        }
        ++k;
        __syncthreads();
    }

    // ---- state: the iterate (X_k of the stopping pass, or the next one), S of
    // the last pass, the control block
    if (stop) {
        for (int e = t; e < tw * 16 * m; e += kSmT) {
            const int64_t c = 16 * tb + e / m;
            if (c < n) a.S[c * m + e % m] = Sw[e];
        }
    }
    if (wg == 0) {
        float* xk = (k & 1) ? a.x1 : a.x0;
        for (int e = t; e < p * m; e += kSmT) {
            const int j = e / p, r = e % p;
            xk[(size_t)j * ldx + r] = Xl[4 * ((r >> 2) * m + j) + (r & 3)];
        }
        if (a.path)
            for (int j = t; j < m; j += kSmT) a.ps[j] = lps[j];
        else if (m > 1)
            for (int e = t; e < mm; e += kSmT) a.vprev[e] = coef[5 * mm + e];
        if (t == 0) {
            a.ctrl->k = k;
            a.ctrl->done = lc.done;
            a.ctrl->status = lc.status;
            a.ctrl->n_iter = lc.n_iter;
            a.ctrl->ndead = lc.ndead;
            a.ctrl->degenerate_seen = lc.degenerate_seen;
            a.ctrl->warm = lc.warm;
            a.ctrl->no_newton = lc.no_newton;
            a.ctrl->last_F = lc.last_F;
        }
    }
}

}  // namespace

// Workgroups of the solve (0: it is not taken) and whether each sums all of G.
int small_workgroups(const Plan& pl, int* whole) {
    if (pl.m > (pl.path ? 16 : 8) || pl.restricted) return 0;
    const int64_t ntile = (pl.n + 15) / 16;
    static_assert(kSmallWgs <= 64, "one lane per workgroup's objective term");
    // the columns alone in 64 bits first (64 bytes of LDS per row and tile at least):
    // small_lds counts in 32
    if ((ntile + kSmallWgs - 1) / kSmallWgs * 64 * pl.p > kSmallLds) return 0;
    const int most = std::min(kSmallWgs, std::min(pl.npart, pl.nwave_part) / 2);   // two sets
    // tiles per workgroup that give its waves work, then what its LDS holds
    int nb = (int)std::min<int64_t>(most, (ntile + kSmallTiles - 1) / kSmallTiles);
    nb = std::max(nb, 1);
    while (nb < most && small_lds((int)pl.p, pl.m, pl.path, pl.n, nb).total > kSmallLds) ++nb;
    if (small_lds((int)pl.p, pl.m, pl.path, pl.n, nb).total > kSmallLds) return 0;
    *whole = (int64_t)nb * pl.p * pl.m <= kSmallWhole ? 1 : 0;
    return nb;
}

hipError_t launch_small(const Plan& pl, const PassParams& pp, float* x0, float* x1, float* S,
                        float* gpart, double* fpart, int* nnzpart, double* g64, double* trace,
                        double* vprev, PathState* ps, Ctrl* ctrl, int passes, uint32_t bar0,
                        int64_t wait_ticks, hipStream_t st) {
    SmallArgs a{x0, x1, S, gpart, fpart, nnzpart, g64, trace, vprev, ps, ctrl, pl.defl_q,
                pl.defl_k, pl.exact, pl.path, pl.small_nb, pl.small_whole, passes, bar0, wait_ticks};
    const int lds = small_lds((int)pl.p, pl.m, pl.path, pl.n, pl.small_nb).total;
    const dim3 grid(pl.small_nb), block(kSmT);
#define GPSPCA_SMK(ST, MB, BLOCK)                                                              \
    do {                                                                                       \
        static const hipError_t limit = hipFuncSetAttribute(                                   \
            (const void*)k_small<ST, MB, BLOCK>, hipFuncAttributeMaxDynamicSharedMemorySize,   \
            kSmallLds);                                                                        \
        if (limit != hipSuccess) (void)hipGetLastError();                                      \
        GPSPCA_LAUNCH_TIMED((k_small<ST, MB, BLOCK>), grid, block, lds, st, pp, a);            \
    } while (0)
#define GPSPCA_SM(ST)                                              \
    do {                                                           \
        if (pl.m == 1 || pl.path) GPSPCA_SMK(ST, 1, false);        \
        else GPSPCA_SMK(ST, 8, true);                              \
    } while (0)
    if (pl.dtype == GPSPCA_BF16) GPSPCA_SM(kStBF16);
    else if (pl.dtype == GPSPCA_F8E4M3) GPSPCA_SM(kStF8);
    else GPSPCA_SM(kStF32);
#undef GPSPCA_SMK
#undef GPSPCA_SM
    return hipGetLastError();
}

}  // namespace gpspca
