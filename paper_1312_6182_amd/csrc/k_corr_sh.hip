// k_corr_sh: correlation + threshold of the block forms and gamma paths, for
// every storage type of A and every alignment of its columns.
//
//   y_ij = a_i^T x_j (Table 1), then the soft / hard threshold, S, a per-column
//   activity flag and the objective partials.
//
// A pass cannot do without one read of A, so everything here serves the
// stream: A goes from HBM into registers by 16-byte loads, 4 (256 bytes per
// column) or 8 (128 bytes) column segments per instruction, and each register is
// loaded again for a later stage as soon as it has been handed to LDS.  A wave
// so keeps 8-16 KB in flight at all times, about 100 KB per CU, without LDS space
// or barriers of its own.  Register loads at 4-byte alignment also cover columns
// that a DMA into LDS cannot take.  The loads are ordinary ones: columns start
// in the middle of 128-byte lines, and nontemporal loads read a line that two
// stages share twice (without arithmetic, 10000 x 100000: 5.7 against 6.2 TB/s).
//
//   - one workgroup of 8 waves per CU; it owns whole tiles of 16 columns,
//     split evenly over its waves (at most 4 tiles per wave and round);
//   - rows are streamed in stages of SB bytes per column.  A wave writes a
//     pair of tiles to its own LDS region (16-byte slots XOR-swizzled by the
//     column, so that writes and operand reads are free of bank conflicts) and
//     reads the operands back; LDS operations of one wave are in order, so the
//     region needs no second copy;
//   - X is staged once per stage for all 8 waves, double-buffered, one barrier
//     per stage.  In the bfloat16 modes its three parts x = x1 + x2 + x3 are
//     made there, once per workgroup instead of once per wave.
//
// Times (10000 x 100000 unless stated; in brackets the kernels that served these
// before): FP32, 64 components 950 us (one wave per workgroup, parts of X made
// by every wave: 1245); FP32, 32 components 757 us (LDS DMA, 16x16x4 products:
// 759 + 9 for its leftover tiles); e4m3, 32 components 296 us (372); odd leading
// dimension, FP32: 12 components 756 us, 32 components 913, 64 components 1145
// (n = 100000, p = 10001), 1999 x 20011, 12 components 39 us (two vector-ALU
// launches of 37); bfloat16 2003 x 20021, 16 components 34 us (38).
// At 64 components the six part products are the bound, with the conversions
// on two waves per SIMD to overlap them; the totals take 35 us, for an error of
// 2.7e-7 instead of 1.6e-6 at p = 10000 (in registers, added to after every stage:
// 75 us, 3.4e-7).  Below that, HBM and the latency of the stages.
// Modes (the arithmetic stays FP32-accurate in each):
//   0  FP32 A, v_mfma_f32_16x16x4_f32 (at most 2 component groups: at 4 the
//      FP32 matrix cores, not HBM, are the bound);
//   1  FP32 A split exactly into three bfloat16 parts, six part products on
//      v_mfma_f32_16x16x32_bf16 (the three dropped ones are below 2^-23 of a
//      product, FP32's own rounding of it);
//   2  bfloat16 codes, three products with the parts of X;
//   3  e4m3 codes widened to bfloat16 (exact), as mode 2.
// Rows past the last full 16-byte slot are added by FP32 FMAs at the end.  A
// correlation that comes out non-finite is computed again by plain FP32 FMAs:
// the parts of an infinity or of a value near the FP32 limit are NaN, and in
// every mode the slots of the last stage past a column's end repeat its last
// full slot against zeros of X, where an infinity gives NaN.
#include "corr.h"
#include "gpspca_internal.h"
#include "storage.h"

#include <algorithm>
#include <type_traits>

namespace gpspca {

namespace {

typedef float f4s __attribute__((ext_vector_type(4)));
typedef double d4s __attribute__((ext_vector_type(4)));
typedef __bf16 bf8s __attribute__((ext_vector_type(8)));
typedef uint32_t u4s __attribute__((ext_vector_type(4)));
typedef uint32_t u4sa __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kShWaves = 8;
constexpr int kShThreads = 64 * kShWaves;
constexpr int kShTiles = 4;   // tiles per wave and round, at most
constexpr int kShFlush = 4;   // stages per accumulator
constexpr int kShLdsTiles = 3;   // tiles of a wave whose totals are in LDS (mode 1)

template <int MODE, int J, int SB>
struct Sh {
    static constexpr int ES = MODE <= 1 ? 4 : MODE == 2 ? 2 : 1;   // bytes per element
    static constexpr int EPS = 16 / ES;                             // rows per slot
    static constexpr int NS = SB / 16;                              // slots per column and stage
    static constexpr int NL = NS / 4;                               // loads per tile and stage
    static constexpr int RS = SB / ES;                              // rows per stage
    static constexpr int KS = RS / 32;                              // bfloat16 contraction steps
    static constexpr int XItems = MODE == 0 ? RS / 4 * 16 * J : KS * J * 64;
    static constexpr int XI = (XItems + kShThreads - 1) / kShThreads;
    static constexpr int XBytes = MODE == 0 ? RS * 16 * J * 4 : RS * 16 * J * 6;
    static constexpr int AWave = 2 * 16 * SB;                       // a pair of tiles
    static constexpr int Tot = MODE == 1 ? kShLdsTiles * J * 1024 : 0;   // totals of a wave
    static constexpr int Lds = 2 * XBytes + kShWaves * AWave;
    static_assert(Lds + kShWaves * Tot <= 160 * 1024, "LDS of a CU");
};

__device__ __forceinline__ uint32_t sh_pack_hi(float lo, float hi) {
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

__device__ __forceinline__ bf8s sh_widen8(uint32_t w0, uint32_t w1) {
    const qf2 a = e4m3_pair(w0, false), b = e4m3_pair(w0, true);
    const qf2 c = e4m3_pair(w1, false), d = e4m3_pair(w1, true);
    return __builtin_bit_cast(bf8s, u4s{sh_pack_hi(a.x, a.y), sh_pack_hi(b.x, b.y),
                                        sh_pack_hi(c.x, c.y), sh_pack_hi(d.x, d.y)});
}

template <int MODE>
__device__ __forceinline__ float sh_elem(const uint8_t* col, int r) {
    if constexpr (MODE <= 1) return reinterpret_cast<const float*>(col)[r];
    else if constexpr (MODE == 2) return bf16_value(reinterpret_cast<const uint16_t*>(col)[r]);
    else return e4m3_value(col[r]);
}

// One round of one wave: its NT tiles of 16 columns from c0 (columns at or past
// cend are clamped and their results dropped).  Every wave of the workgroup
// takes part in the staging of X and in the barriers, NT = 0 included.
// D stages of A are in flight in registers.
template <int MODE, int J, int SB, int FINE, int NT, int D>
__device__ __forceinline__ void sh_round(const PassParams& pp, int64_t c0, int64_t cend, int wv,
                                         uint8_t* __restrict__ lds, const float* __restrict__ X,
                                         const float* __restrict__ Xil, double* f_acc,
                                         int* nnz_acc, float* __restrict__ S,
                                         uint8_t* __restrict__ act) {
    using T = Sh<MODE, J, SB>;
    constexpr int UN = D > 2 ? D : 2;          // stages per trip of the unrolled loop
    constexpr int NA = NT > 0 ? NT : 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int lj = lane & 15, lk = lane >> 4;
    const int p = pp.p, m = pp.m;
    const int nsf = p / T::EPS;                // full slots per column
    const int nst = (nsf + T::NS - 1) / T::NS; // stages
    const int nxq = nsf * (T::EPS / 4);        // row quads of X that full slots cover
    const int nqx = pp.ldx >> 2;               // quads of the X buffers; the last is zero
    const uint8_t* Ab = MODE <= 1 ? reinterpret_cast<const uint8_t*>(pp.A)
                      : MODE == 2 ? reinterpret_cast<const uint8_t*>(pp.Abf) : pp.Af8;
    const int64_t colbytes = pp.lda * T::ES;

    // load i of a tile: column 64/NS i + lane / NS, slot lane % NS
    const int lslot = lane % T::NS, lcol = lane / T::NS;
    const uint8_t* tb[NA];
    uint32_t voff[NA][T::NL];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int64_t ct = c0 + 16 * t;
        tb[t] = Ab + ct * colbytes;
#pragma unroll
        for (int i = 0; i < T::NL; ++i) {
            int64_t c = ct + (64 / T::NS) * i + lcol;
            c = c < cend ? c : cend - 1;
            voff[t][i] = (uint32_t)((c - ct) * colbytes);
        }
    }
    u4s areg[D][NA][T::NL];
    auto slot_off = [&](int st) {
        const int sl = T::NS * st + lslot;
        return 16u * (uint32_t)(sl < nsf ? sl : nsf - 1);
    };
    auto load_tile = [&](int t, uint32_t so, u4s (&dst)[T::NL]) {
#pragma unroll
        for (int i = 0; i < T::NL; ++i)
            dst[i] = *reinterpret_cast<const u4sa*>(tb[t] + (size_t)(voff[t][i] + so));
    };

    // X items of this thread
    f4s xreg[2][T::XI][2];
    auto load_x = [&](int st, f4s (&dst)[T::XI][2]) {
#pragma unroll
        for (int k = 0; k < T::XI; ++k) {
            const int it = tid + kShThreads * k;
            if (T::XItems % kShThreads != 0 && it >= T::XItems) continue;
            if constexpr (MODE == 0) {
                const int c = it & 15, jq = it >> 4;
                const int jb = jq / (T::RS / 4);
                int q = T::RS / 4 * st + jq % (T::RS / 4);
                q = q < nxq ? q : nqx - 1;
                dst[k][0] = *reinterpret_cast<const f4s*>(Xil + ((size_t)(jb * nqx + q) * 16 + c) * 4);
            } else {
                const int rest = it >> 6, h = rest % T::KS, jb = rest / T::KS;
                const int r0 = MODE == 3 ? 64 * (h >> 1) + 16 * lk + 8 * (h & 1) : 32 * h + 8 * lk;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    int q = T::RS / 4 * st + r0 / 4 + u;
                    q = q < nxq ? q : nqx - 1;
                    dst[k][u] = *reinterpret_cast<const f4s*>(
                        Xil + ((size_t)(jb * nqx + q) * 16 + lj) * 4);
                }
            }
        }
    };
    auto store_x = [&](uint8_t* xb, const f4s (&src)[T::XI][2]) {
#pragma unroll
        for (int k = 0; k < T::XI; ++k) {
            const int it = tid + kShThreads * k;
            if (T::XItems % kShThreads != 0 && it >= T::XItems) continue;
            if constexpr (MODE == 0) {
                *reinterpret_cast<f4s*>(xb + 16 * it) = src[k][0];
            } else {
                bf8s x1, x2, x3;
                split3_bf16(src[k][0], src[k][1], x1, x2, x3);
                uint8_t* at = xb + 3072 * (it >> 6) + 16 * lane;   // (jb KS + h) x 3 parts
                *reinterpret_cast<bf8s*>(at) = x1;
                *reinterpret_cast<bf8s*>(at + 1024) = x2;
                *reinterpret_cast<bf8s*>(at + 2048) = x3;
            }
        }
    };

    // The matrix cores chain their additions (FP32 operands: one rounding per
    // row; bfloat16: one truncation per 32 rows), so an accumulator through all
    // rows would be off by sqrt(rows) roundings.  STEP: it carries 16 rows (FINE
    // == 8: 8; mode 1: 32) from zero and is added to tot in FP64.
    // Otherwise acc carries kShFlush stages before it is added to tot; with 4
    // component groups of 16/8-bit codes it is all there is.
    // Mode 1 without FINE: acc carries 2 kShFlush stages, and the totals of three
    // of a wave's four tiles are in LDS (there are no registers for them).
    constexpr bool STEP = FINE > 0, LTOT = MODE == 1 && !STEP;
    constexpr bool kTot = STEP || J < 4;
    using TotV = typename std::conditional<STEP, d4s, f4s>::type;
    f4s acc[STEP ? 1 : NA][STEP ? 1 : J];
    TotV tot[kTot ? NA : 1][kTot || LTOT ? J : 1];
    f4s* const lt = reinterpret_cast<f4s*>(lds + 2 * T::XBytes + kShWaves * T::AWave + wv * T::Tot) +
                    lane;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int jb = 0; jb < J; ++jb) {
            if constexpr (!STEP) acc[t][jb] = f4s{0.f, 0.f, 0.f, 0.f};
            if constexpr (kTot) tot[t][jb] = TotV{0, 0, 0, 0};
            else if constexpr (LTOT) {
                if (t < kShLdsTiles) lt[64 * (t * J + jb)] = f4s{0.f, 0.f, 0.f, 0.f};
                else tot[0][jb] = TotV{0, 0, 0, 0};
            }
        }
    auto flush = [&] {
        if constexpr ((kTot && !STEP) || LTOT) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int jb = 0; jb < J; ++jb) {
                    if constexpr (kTot) tot[t][jb] += acc[t][jb];
                    else if (t < kShLdsTiles) lt[64 * (t * J + jb)] += acc[t][jb];
                    else tot[0][jb] += acc[t][jb];
                    acc[t][jb] = f4s{0.f, 0.f, 0.f, 0.f};
                }
        }
    };

    uint8_t* const aw = lds + 2 * T::XBytes + wv * T::AWave;
    // slot (c, q) of a tile in the wave's region
    auto a_at = [&](int pt, int c, int q) {
        return aw + 16 * ((pt * 16 + c) * T::NS + (q ^ (c & (T::NS - 1))));
    };
    // tiles t0 .. t0 + PT - 1 of the stage whose registers are `src`: to LDS, the
    // registers loaded again for a later stage, operands back, products
    auto tiles = [&](auto pt_c, int t0, u4s (&src)[NA][T::NL], uint32_t so_next,
                     const uint8_t* xb) {
        constexpr int PT = decltype(pt_c)::value;
#pragma unroll
        for (int u = 0; u < PT; ++u)
#pragma unroll
            for (int i = 0; i < T::NL; ++i)
                *reinterpret_cast<u4s*>(a_at(u, (64 / T::NS) * i + lcol, lslot)) = src[t0 + u][i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < PT; ++u) load_tile(t0 + u, so_next, src[t0 + u]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MODE == 0) {
#pragma unroll
            for (int g = 0; g < T::RS / 16; ++g) {
                f4s a[PT];
#pragma unroll
                for (int u = 0; u < PT; ++u)
                    a[u] = *reinterpret_cast<const f4s*>(a_at(u, lj, 4 * g + lk));
#pragma unroll
                for (int jb = 0; jb < J; ++jb) {
                    const f4s x = *reinterpret_cast<const f4s*>(
                        xb + 16 * ((jb * (T::RS / 4) + 4 * g + lk) * 16 + lj));
                    constexpr int NC = FINE == 8 ? 2 : 1;
                    f4s c[NC][PT];
#pragma unroll
                    for (int u = 0; u < PT; ++u)
#pragma unroll
                        for (int h = 0; h < NC; ++h) {
                            if constexpr (STEP) c[h][u] = f4s{0.f, 0.f, 0.f, 0.f};
                            else c[h][u] = acc[t0 + u][jb];
                        }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int u = 0; u < PT; ++u)
                            c[e % NC][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], x[e],
                                                                                c[e % NC][u], 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < PT; ++u) {
                        if constexpr (STEP) {
#pragma unroll
                            for (int h = 0; h < NC; ++h)
                                tot[t0 + u][jb] += __builtin_convertvector(c[h][u], TotV);
                        } else {
                            acc[t0 + u][jb] = c[0][u];
                        }
                    }
                }
            }
        } else {
            u4s raw[PT];
#pragma unroll
            for (int h = 0; h < T::KS; ++h) {
                bf8s a1[PT], a2[PT], a3[PT];
#pragma unroll
                for (int u = 0; u < PT; ++u) {
                    if constexpr (MODE == 1) {
                        const f4s q0 = *reinterpret_cast<const f4s*>(a_at(u, lj, 8 * h + 2 * lk));
                        const f4s q1 = *reinterpret_cast<const f4s*>(a_at(u, lj, 8 * h + 2 * lk + 1));
                        split3_bf16(q0, q1, a1[u], a2[u], a3[u]);
                    } else if constexpr (MODE == 2) {
                        a1[u] = *reinterpret_cast<const bf8s*>(a_at(u, lj, 4 * h + lk));
                    } else {
                        if ((h & 1) == 0)
                            raw[u] = *reinterpret_cast<const u4s*>(a_at(u, lj, 2 * h + lk));
                        a1[u] = sh_widen8(raw[u][2 * (h & 1)], raw[u][2 * (h & 1) + 1]);
                    }
                }
#pragma unroll
                for (int jb = 0; jb < J; ++jb) {
                    const uint8_t* at = xb + 3072 * (jb * T::KS + h) + 16 * lane;
                    const bf8s x1 = *reinterpret_cast<const bf8s*>(at);
                    const bf8s x2 = *reinterpret_cast<const bf8s*>(at + 1024);
                    const bf8s x3 = *reinterpret_cast<const bf8s*>(at + 2048);
                    f4s c[PT];
#pragma unroll
                    for (int u = 0; u < PT; ++u) {
                        if constexpr (STEP) c[u] = f4s{0.f, 0.f, 0.f, 0.f};
                        else c[u] = acc[t0 + u][jb];
                    }
#define GPSPCA_SH_MM(AA, XX)                                                              \
    _Pragma("unroll") for (int u = 0; u < PT; ++u) c[u] =                                  \
        __builtin_amdgcn_mfma_f32_16x16x32_bf16(AA[u], XX, c[u], 0, 0, 0)
                    if constexpr (MODE == 1) {   // smallest terms first
                        GPSPCA_SH_MM(a3, x1);
                        GPSPCA_SH_MM(a2, x2);
                        GPSPCA_SH_MM(a1, x3);
                        GPSPCA_SH_MM(a2, x1);
                        GPSPCA_SH_MM(a1, x2);
                        GPSPCA_SH_MM(a1, x1);
                    } else {
                        GPSPCA_SH_MM(a1, x3);
                        GPSPCA_SH_MM(a1, x2);
                        GPSPCA_SH_MM(a1, x1);
                    }
#undef GPSPCA_SH_MM
#pragma unroll
                    for (int u = 0; u < PT; ++u) {
                        if constexpr (STEP) tot[t0 + u][jb] += __builtin_convertvector(c[u], TotV);
                        else acc[t0 + u][jb] = c[u];
                    }
                }
            }
        }
    };

    if (nst > 0) {
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
            for (int t = 0; t < NT; ++t) load_tile(t, slot_off(d), areg[d][t]);
        load_x(0, xreg[0]);
        load_x(1, xreg[1]);   // a stage past the last meets the zero quad
        for (int s0 = 0; s0 < nst; s0 += UN) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int s = s0 + u;
                if (s >= nst) continue;
                uint8_t* const xb = lds + (u & 1) * T::XBytes;   // UN is even
                store_x(xb, xreg[u & 1]);
                load_x(s + 2, xreg[u & 1]);
                __syncthreads();
                if constexpr (NT > 0) {
                    const uint32_t so = slot_off(s + D);
                    if constexpr (NT >= 2) tiles(std::integral_constant<int, 2>{}, 0, areg[u % D], so, xb);
                    if constexpr (NT == 4) tiles(std::integral_constant<int, 2>{}, 2, areg[u % D], so, xb);
                    if constexpr (NT == 1) tiles(std::integral_constant<int, 1>{}, 0, areg[u % D], so, xb);
                    if constexpr (NT == 3) tiles(std::integral_constant<int, 1>{}, 2, areg[u % D], so, xb);
                    if ((s + 1) % (LTOT ? 2 * kShFlush : kShFlush) == 0) flush();
                }
            }
        }
        // the next round's first stage writes the X buffer that a wave may
        // still be reading here
        __syncthreads();
        flush();
    }

    if constexpr (NT > 0) {
        const int rows_main = nsf * T::EPS;
        const bool l0 = pp.l0 != 0;
        int nact_l = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t col = c0 + 16 * t + 4 * lk + v;
                const bool cvalid = col < cend;
                const uint8_t* ac = Ab + (cvalid ? col : cend - 1) * colbytes;
                float y[J];
#pragma unroll
                for (int jb = 0; jb < J; ++jb) {
                    if constexpr (kTot) y[jb] = (float)tot[t][jb][v];
                    else if constexpr (LTOT)
                        y[jb] = t < kShLdsTiles ? lt[64 * (t * J + jb)][v] : tot[0][jb][v];
                    else y[jb] = acc[t][jb][v];
                }
                for (int r = rows_main; r < p; ++r) {
                    const float a = sh_elem<MODE>(ac, r);
#pragma unroll
                    for (int jb = 0; jb < J; ++jb)
                        y[jb] = __builtin_fmaf(a, X[(size_t)(16 * jb + lj) * pp.ldx + r], y[jb]);
                }
#pragma unroll
                for (int jb = 0; jb < J; ++jb)
                    if (!(fabsf(y[jb]) < __builtin_inff())) {
                        const float* xc = X + (size_t)(16 * jb + lj) * pp.ldx;
                        float z = 0.f;
                        for (int r = 0; r < p; ++r)
                            z = __builtin_fmaf(sh_elem<MODE>(ac, r), xc[r], z);
                        y[jb] = z;
                    }
                const float sc = (MODE >= 2 && cvalid) ? column_scale(pp, col) : 1.0f;
                bool any = false;
#pragma unroll
                for (int jb = 0; jb < J; ++jb) {
                    const int comp = 16 * jb + lj;
                    if (cvalid && comp < m) {
                        float sv;
                        double fv;
                        const bool on = threshold(l0, pp.mu[comp], pp.gam[comp],
                                                  MODE >= 2 ? sc * y[jb] : y[jb], sv, fv);
                        S[col * m + comp] = sv;
                        if (on) {
                            f_acc[jb] += fv;
                            nnz_acc[jb] += 1;
                            any = true;
                        }
                    }
                }
                const uint64_t bal = __ballot(any);
                if (cvalid && lj == 0) {
                    const int fl = ((bal >> (16 * lk)) & 0xFFFFull) ? 1 : 0;
                    act[col] = fl;
                    nact_l += fl;
                }
            }
        add_active_count(nact_l, pp.nact);
    }
}

template <int MODE, int J, int SB, int FINE>
__global__ __launch_bounds__(kShThreads, 2) void k_corr_sh(PassParams pp, const float* __restrict__ X,
                                                        const float* __restrict__ Xil,
                                                        float* __restrict__ S,
                                                        uint8_t* __restrict__ act,
                                                        double* __restrict__ fpart,
                                                        int* __restrict__ nnzpart,
                                                        const Ctrl* __restrict__ ctrl) {
    if (ctrl->done) return;
    using T = Sh<MODE, J, SB>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[T::Lds + (FINE ? 0 : kShWaves * T::Tot)];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = pp.m;
    const int64_t n = pp.n;
    const int64_t G = gridDim.x, g = blockIdx.x;
    const int64_t ntile = (n + 15) / 16;
    const int64_t tb = ntile * g / G, te = ntile * (g + 1) / G;   // this workgroup's tiles
    const int lj = lane & 15;

    double f_acc[J];
    int nnz_acc[J];
#pragma unroll
    for (int jb = 0; jb < J; ++jb) { f_acc[jb] = 0.0; nnz_acc[jb] = 0; }

    // FP64 totals of 4 component groups: two tiles are what the registers hold
    constexpr int most = FINE > 0 && J == 4 ? 2 : kShTiles;
    constexpr int per = kShWaves * most;
    for (int64_t r0 = tb; r0 < te; r0 += per) {
        // the round's tiles, split evenly over the waves
        const int64_t r1 = r0 + per < te ? r0 + per : te;
        const int64_t nt = r1 - r0;
        const int64_t w0 = r0 + nt * wv / kShWaves, w1 = r0 + nt * (wv + 1) / kShWaves;
        const int64_t c0 = 16 * w0;
        const int64_t cend = std::min<int64_t>(n, 16 * w1);
        constexpr int d1 = T::NL == 4 ? 4 : 6;
#define GPSPCA_SHR(NT, D) \
    sh_round<MODE, J, SB, FINE, NT, D>(pp, c0, cend, wv, lds, X, Xil, f_acc, nnz_acc, S, act)
        switch ((int)(w1 - w0)) {
            case 0: GPSPCA_SHR(0, 1); break;
            case 1: GPSPCA_SHR(1, d1); break;
            case 2: GPSPCA_SHR(2, (d1 == 4 ? 2 : 4)); break;
            default:
                if constexpr (most > 2) {
                    if (w1 - w0 == 3) GPSPCA_SHR(3, (d1 == 4 ? 1 : 2));
                    else GPSPCA_SHR(4, (d1 == 4 ? 1 : 2));
                }
        }
#undef GPSPCA_SHR
    }

    const int64_t W = G * kShWaves, w = g * kShWaves + wv;
#pragma unroll
    for (int jb = 0; jb < J; ++jb) {
        double f = f_acc[jb];
        int c = nnz_acc[jb];
        f += __shfl_xor(f, 16, 64);
        c += __shfl_xor(c, 16, 64);
        f += __shfl_xor(f, 32, 64);
        c += __shfl_xor(c, 32, 64);
        const int comp = 16 * jb + lj;
        if (lane < 16 && comp < m) {
            fpart[(int64_t)comp * W + w] = f;
            nnzpart[(int64_t)comp * W + w] = c;
        }
    }
}

template <int MODE, int J, int SB, int FINE = 0>
hipError_t sh_launch(const Plan& pl, const PassParams& pp, const float* X, const float* Xil,
                     float* S, uint8_t* act, double* fpart, int* nnzpart, const Ctrl* ctrl,
                     hipStream_t st) {
    GPSPCA_LAUNCH_TIMED((k_corr_sh<MODE, J, SB, FINE>), dim3(pl.corr_grid), dim3(kShThreads), 0, st,
                        pp, X, Xil, S, act, fpart, nnzpart, ctrl);
    return hipGetLastError();
}

}  // namespace

int corr_sh_grid(int64_t n, int ncu) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(ncu, (n + 15) / 16));
}
int corr_sh_waves() { return kShWaves; }

// Columns of up to 2^26 bytes: the 32-bit offsets of a tile's 16 columns.  e4m3
// with 4 component groups is left to k_corr_qw (X alone takes 96 KB of LDS per
// 128 rows: 12.7 against 12.6 ms for 12 passes at 10000 x 100000).
bool corr_sh_ok(const Plan& pl) {
    const int64_t es = pl.dtype == GPSPCA_F32 ? 4 : pl.dtype == GPSPCA_BF16 ? 2 : 1;
    return pl.lda * es <= ((int64_t)1 << 26) && !(pl.dtype == GPSPCA_F8E4M3 && pl.m > 32);
}

hipError_t launch_corr_sh(const Plan& pl, const PassParams& pp, const float* X, const float* Xil,
                          float* S, uint8_t* act, double* fpart, int* nnzpart, const Ctrl* ctrl,
                          hipStream_t st) {
    const int J = pl.m <= 16 ? 1 : pl.m <= 32 ? 2 : 4;
#define GPSPCA_SH(MODE, JJ, SB) \
    return sh_launch<MODE, JJ, SB>(pl, pp, X, Xil, S, act, fpart, nnzpart, ctrl, st)
    // FP32 columns that are not 16-byte aligned: FP64 totals, so that this kernel
    // is as close to FP64 as the vector-ALU one (k_corr), whose lanes add p / 64
    // rows each.  Relative error of a correlation, here / k_corr: 6.4e-8 / 7.2e-8
    // at p = 101, 7.9e-8 / 7.6e-8 at 201 by 16 rows (6.5e-8 by 8), 8.2e-8 / 8.3e-8 at
    // 401, 8.2e-8 / 2.3e-7 at 10001 (FP32 totals: 2.9e-7 at 1001, 3.1e-7 at 10001).
    // 8 rows cost 4 us more than 16 at 1999 x 20011, m = 12, so only short
    // columns take them.  64 components: 5e-8 to 1.2e-7 / 7e-8 to 2.3e-7 (one
    // accumulator: 4.8e-7 at 1001, 1.6e-6 at 10001).
    if (pl.dtype == GPSPCA_F32 && !pl.vec4) {
#define GPSPCA_SHF(MODE, JJ, SB, FF) \
    return sh_launch<MODE, JJ, SB, FF>(pl, pp, X, Xil, S, act, fpart, nnzpart, ctrl, st)
        if (J == 4) GPSPCA_SHF(1, 4, 128, 16);
        if (J == 1) {
            if (pl.p < 401) GPSPCA_SHF(0, 1, 256, 8);
            GPSPCA_SHF(0, 1, 256, 16);
        }
        if (pl.p < 401) GPSPCA_SHF(0, 2, 256, 8);
        GPSPCA_SHF(0, 2, 256, 16);
#undef GPSPCA_SHF
    }
    if (pl.dtype == GPSPCA_F32) {
        if (J == 1) GPSPCA_SH(0, 1, 256);
        if (J == 2) GPSPCA_SH(0, 2, 256);
        GPSPCA_SH(1, 4, 128);
    }
    if (pl.dtype == GPSPCA_BF16) {
        if (J == 1) GPSPCA_SH(2, 1, 256);
        if (J == 2) GPSPCA_SH(2, 2, 256);
        GPSPCA_SH(2, 4, 128);
    }
    if (J == 1) GPSPCA_SH(3, 1, 128);
    GPSPCA_SH(3, 2, 128);
#undef GPSPCA_SH
}

}  // namespace gpspca
