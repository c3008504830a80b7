// sk_separable.hip -- the tiled iteration on a shared cost that splits over two
// axes.
//
// A histogram over an h x w grid with a cost that adds up over the axes,
//     C[(r, c), (r', c')] = A[r, r'] + B[c, c'],
// (squared or absolute coordinate differences, or any sum of one function per
// axis) needs no d1 x d2 sweep: the logsumexp of a half-step splits exactly,
//     LSE_{r',c'}(b[r',c'] - C/lambda) = LSE_{r'}(LSE_{c'}(b[r',c'] - B/lambda) - A/lambda),
// so an iteration costs 2 w1 h2 (h1 + w2) cells per problem instead of d1 d2:
// 1.0 million against 16.8 for 64 x 64 grids, 88 thousand against 615 for
// 28 x 28 images.  The planes a problem iterates on fit the LDS of one CU, so
// one work-group runs all its iterations in one launch (sk_sep_solve).
//
// Whether a cost splits is tested on the device in every call, over every
// entry (sk_sep_guess, sk_sep_verify): nothing is assumed from sizes, and a
// cost that does not split is left to the sweeps.
//
// Line sums without an exponential per cell: with integers Lr (per output o
// and block J of BS inputs, the rounded largest exponent of the block) and
// R_J (the rounded largest input of the block),
//     sum_i 2^(x_i + L_oi) = sum_J 2^(R_J + Lr_oJ) sum_{i in J} 2^(x_i - R_J) E_oi,
//     E_oi = 2^(L_oi - Lr_oJ)   (a table made once per call),
// so a cell is one fma and a block one integer add, max and subtraction, one
// ldexp and one addition: 4 + 20/BS cycles per 64 cells against 22 for an
// exponential with a running maximum.  Scalings and sums are a float times a
// power of two held as an integer, so nothing is lost to the size of the
// potentials (thousands of units at small lambda) and an iteration takes no
// exponential and no logarithm: only the returned potentials are rounded to
// fp32.
#include <type_traits>

#include "sk_device.h"
#include "sk_internal.h"

namespace sk {
namespace {

constexpr int kSepLine = 64;  // longest line (one lane per entry)

// Lanes of a line: 16, 32 or 64.
__host__ __device__ inline int sep_lanes(int n1, int n2) {
    const int n = n1 > n2 ? n1 : n2;
    return n <= 16 ? 16 : (n <= 32 ? 32 : 64);
}
// Cells of half an iteration's line sums, and whether a pair of grid widths
// qualifies: at most half as many cells per iteration as the sweep.
__host__ __device__ inline int sep_half_cells(int w1, int h1, int w2, int h2) { return w1 * h2 * (h1 + w2); }
__host__ __device__ inline bool sep_pair_ok(int d1, int d2, int w1, int w2) {
    if (w1 < 2 || w2 < 2 || w1 > kSepLine || w2 > kSepLine || d1 % w1 || d2 % w2) return false;
    if (d1 == d2 && w1 != w2) return false;  // one grid
    const int h1 = d1 / w1, h2 = d2 / w2;
    if (h1 < 2 || h2 < 2 || h1 > kSepLine || h2 > kSepLine) return false;
    return (int64_t)4 * sep_half_cells(w1, h1, w2, h2) <= (int64_t)d1 * d2;
}

// Four line tables, each the E entries [in / 4][out][in % 4] (64 x 64 at most)
// followed by the block exponents Lr [J / 4][out][J % 4] (16 x 64 at most).
constexpr int kSepTable = kSepLine * kSepLine + 16 * kSepLine;
constexpr int kTabU1 = 0, kTabU2 = 1, kTabV1 = 2, kTabV2 = 3;  // T -> a, a -> S, S -> b, b -> T
// The cost-weighted tables of the loss: E s C 2^-kSepWeight in the place of E
// (|s C| < 2^22, see sk_sep_verify, so a product still fits the budget below).
constexpr int kTabWU = 4, kTabWV = 5, kTables = 6;
constexpr int kSepWeight = 22;
// Exponent budget: E <= 2^(kSepE0 + 1/2), inputs 2^(x - R + kSepE0), so a sum of
// 64 products stays below 2^(2 kSepE0 + 8).  With a block's exponents within
// kSepSpan bits every E is a normal number, the largest product of a block is
// at least 2^(2 kSepE0 - kSepSpan - 1), and an input that underflows was below
// 2^(kSepSpan - kSepE0 - 126) = 2^-31 of it.
constexpr int kSepE0 = 55, kSepSpan = 150;

// ---- does the cost split? ----
//
// Entry (i, j) against the entries of the first row and column of its blocks:
// in exact arithmetic C[i,j] - C[(r,0),(r',0)] - C[(0,c),(0,c')] + C[0,0] = 0.
// The four entries are fp32 roundings of costs that may themselves have been
// computed in fp32, so each may be off by 2^-23 of its value; nothing larger
// passes.  (NaN and infinities fail the comparison.)
__device__ __forceinline__ bool sep_entry_ok(float cij, float ca, float cb, float c00) {
    const double d = ((double)cij - (double)ca) - ((double)cb - (double)c00);
    const double t = 1.1920928955078125e-7 * ((fabs((double)cij) + fabs((double)ca)) +
                                              (fabs((double)cb) + fabs((double)c00)));
    return fabs(d) <= t && t < 1e30;
}

// One work-group: every pair of widths (w1 | d1, w2 | d2) is tried on 16
// entries; of the pairs that pass, the one with the fewest cells goes on to
// sk_sep_verify.
constexpr int kGuessThreads = 1024;
__global__ __launch_bounds__(kGuessThreads) void sk_sep_guess(const float *C, int d1, int d2, int32_t *mode) {
    __shared__ unsigned best;
    if (threadIdx.x == 0) best = 0xffffffffu;
    __syncthreads();
    const float c00 = C[0];
    for (int u = threadIdx.x; u < kSepLine * kSepLine; u += kGuessThreads) {
        const int w1 = u / kSepLine + 1, w2 = u % kSepLine + 1;
        if (!sep_pair_ok(d1, d2, w1, w2)) continue;
        bool ok = true;
#pragma unroll
        for (int n = 1; n <= 16; ++n) {
            const int i = (int)(((uint64_t)(2654435769u * (uint32_t)n) * (uint32_t)d1) >> 32);
            const int j = (int)(((uint64_t)(1779033703u * (uint32_t)n + 977u) * (uint32_t)d2) >> 32);
            const int r = i / w1, q = j / w2;
            const float cij = C[(size_t)i * d2 + j], ca = C[(size_t)(r * w1) * d2 + q * w2];
            const float cb = C[(size_t)(i - r * w1) * d2 + (j - q * w2)];
            ok = ok && sep_entry_ok(cij, ca, cb, c00);
        }
        // at most 2^19 half cells above the pair's 12 bits
        if (ok) atomicMin(&best, (unsigned)sep_half_cells(w1, d1 / w1, w2, d2 / w2) << 12 | (unsigned)u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool any = best != 0xffffffffu;
        mode[0] = any ? 16 : 0;
        mode[1] = any ? (int)(best & 4095u) / kSepLine + 1 : 0;
        mode[2] = any ? (int)(best & 4095u) % kSepLine + 1 : 0;
    }
}

// Raw cost of entry (in, out) of line table t.
__device__ __forceinline__ float sep_cost(const float *C, int d2, int w1, int w2, float c00, int t, int in, int o) {
    const bool in_second = t == kTabU1 || t == kTabV2;  // the inputs belong to the second grid
    const int x = in_second ? o : in, y = in_second ? in : o;
    return t == kTabU1 || t == kTabU2 ? C[(size_t)(x * w1) * d2 + y * w2] : C[(size_t)x * d2 + y] - c00;
}
__device__ __forceinline__ void sep_table_shape(int t, int w1, int h1, int w2, int h2, int *nin, int *nout) {
    *nin = t == kTabU1 ? h2 : t == kTabU2 ? h1 : t == kTabV1 ? w1 : w2;
    *nout = t == kTabU1 ? h1 : t == kTabU2 ? h2 : t == kTabV1 ? w2 : w1;
}

// Every entry of the cost (one wavefront per row).  The first work-group also
// checks the spread of the tables' blocks: 16 inputs, else 4, else the cost is
// left to the sweeps.
__global__ __launch_bounds__(256) void sk_sep_verify(const float *C, int d1, int d2, float s, SepArgs P) {
    if (P.mode[0] == 0) return;
    const int w1 = P.mode[1], w2 = P.mode[2], h1 = d1 / w1, h2 = d2 / w2;
    const float c00 = C[0];
    bool ok = true, ok16 = true;
    if (blockIdx.x == 0) {
        for (int t = 0; t < 4; ++t) {
            int nin, nout;
            sep_table_shape(t, w1, h1, w2, h2, &nin, &nout);
            for (int u = threadIdx.x; u < 4 * nout; u += 256) {  // 16 inputs of one output
                const int o = u % nout, J = u / nout;
                float lo16 = 0.f, hi16 = 0.f;
                for (int q = 0; q < 4 && J * 16 + 4 * q < nin; ++q) {
                    float lo = 0.f, hi = 0.f;
                    for (int e = 0; e < 4 && J * 16 + 4 * q + e < nin; ++e) {
                        const float v = s * sep_cost(C, d2, w1, w2, c00, t, J * 16 + 4 * q + e, o);
                        lo = e == 0 || v < lo ? v : lo;
                        hi = e == 0 || v > hi ? v : hi;
                    }
                    ok = ok && hi - lo <= (float)kSepSpan && fabsf(hi) < 4.0e6f && fabsf(lo) < 4.0e6f;
                    lo16 = q == 0 || lo < lo16 ? lo : lo16;
                    hi16 = q == 0 || hi > hi16 ? hi : hi16;
                }
                ok16 = ok16 && hi16 - lo16 <= (float)kSepSpan;
            }
        }
        if (!ok16) atomicMin(P.mode, 4);
    }
    const int lane = threadIdx.x & 63;
    const int step_q = 64 / w2, step_c = 64 - step_q * w2;
    for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < d1; i += gridDim.x * 4) {
        const int r = i / w1, c = i - r * w1;
        const float *row = C + (size_t)i * d2, *ra = C + (size_t)(r * w1) * d2, *rb = C + (size_t)c * d2;
        int q = lane / w2, cc = lane - q * w2;
        for (int j = lane; j < d2; j += 64) {
            ok = ok && sep_entry_ok(row[j], ra[q * w2], rb[cc], c00);
            q += step_q;
            cc += step_c;
            if (cc >= w2) {
                cc -= w2;
                ++q;
            }
        }
    }
    if (!ok) atomicMin(P.mode, 0);
}

// The tables, one work-group each, thread u = one block of 4 inputs of
// one output.  Entries past the line are 0.
__global__ __launch_bounds__(256) void sk_sep_tables(const float *C, int d1, int d2, float s, SepArgs P) {
    const int bs = P.mode[0];
    if (bs == 0) return;
    const int w1 = P.mode[1], w2 = P.mode[2], h1 = d1 / w1, h2 = d2 / w2;
    const int t = blockIdx.x == kTabWU ? kTabU1 : blockIdx.x == kTabWV ? kTabV2 : blockIdx.x;
    const bool weighted = (int)blockIdx.x != t;
    const float c00 = C[0];
    int nin, nout;
    sep_table_shape(t, w1, h1, w2, h2, &nin, &nout);
    const int po = sep_lanes(nin, nout);
    float *E = P.table + blockIdx.x * kSepTable;
    int *Lr = reinterpret_cast<int *>(E + kSepLine * kSepLine);
    for (int u = threadIdx.x; u < po * po / 4; u += 256) {
        const int o = u % po, q = u / po;
        const int per = bs / 4, q0 = q / per * per;  // the block this group of 4 inputs belongs to
        float top = -3.0e38f;
        for (int x = 0; x < bs; ++x) {
            const int in = q0 * 4 + x;
            if (in < nin && o < nout) top = fmaxf(top, -s * sep_cost(C, d2, w1, w2, c00, t, in, o));
        }
        const float ref = top > -3.0e38f ? rintf(top) : 0.f;
        for (int e = 0; e < 4; ++e) {
            const int in = q * 4 + e;
            float v = 0.f;
            if (in < nin && o < nout) {
                const double sc = (double)s * (double)sep_cost(C, d2, w1, w2, c00, t, in, o);
                const double x = -sc - (double)ref;
                const double fl = floor(x);
                v = ldexpf(exp2f((float)(x - fl)), (int)fl + kSepE0);
                if (weighted) v = (float)ldexp((double)v * sc, -kSepWeight);
            }
            E[(q * po + o) * 4 + e] = v;
        }
        if (q == q0) {
            const int J = q0 / per;
            Lr[((J >> 2) * po + o) * 4 + (J & 3)] = (int)ref;
        }
    }
}

// ---- line sums ----

typedef float f4s __attribute__((ext_vector_type(4)));
typedef int i4s __attribute__((ext_vector_type(4)));

// Lane N of each 16-lane row, on all lanes of the row.
template <int N>
__device__ __forceinline__ int row_bcast(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xF, 0xF, true);
}
// Partial sums of 16 inputs: a[g] = sum_{i < 4} y_{4g+i} e[g][i], y_n being lane
// n of the lane's own 16-lane row, broadcast by the instruction itself
// (row_newbcast; the compiler folds the broadcast into a multiplication but
// not into a fused multiply-add).  The leading s_nop covers a vector write of y
// just before (two wait states until a DPP read).
__device__ __forceinline__ void fma16(float (&a)[4], float y, const f4s (&e)[4]) {
    __asm__("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %4, %5 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %1, %4, %9 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %2, %4, %13 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %3, %4, %17 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %6 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %4, %10 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %4, %14 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %4, %18 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %7 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %4, %11 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %4, %15 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %4, %19 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %8 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %4, %12 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %4, %16 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %4, %20 row_newbcast:15 row_mask:0xf bank_mask:0xf"
            : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
            : "v"(y), "v"(e[0][0]), "v"(e[0][1]), "v"(e[0][2]), "v"(e[0][3]), "v"(e[1][0]), "v"(e[1][1]), "v"(e[1][2]),
              "v"(e[1][3]), "v"(e[2][0]), "v"(e[2][1]), "v"(e[2][2]), "v"(e[2][3]), "v"(e[3][0]), "v"(e[3][1]),
              "v"(e[3][2]), "v"(e[3][3]));
}
template <int CTRL>
__device__ __forceinline__ int dppi(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int BS>
__device__ __forceinline__ int block_max(int v) {
    v = max(v, dppi<kQuadXor1>(v));
    v = max(v, dppi<kQuadXor2>(v));
    if (BS == 16) {
        v = max(v, dppi<kHalfMirror>(v));
        v = max(v, dppi<kRowRor8>(v));
    }
    return v;
}
// A value f 2^h; no mass: f = 0 and h far below any other.
constexpr int kSepNone = -(1 << 27);
struct Scaled {
    int h;
    float f;
};
__device__ __forceinline__ Scaled none() { return {kSepNone, 0.f}; }
// 2^x (x = -inf: none).
__device__ __forceinline__ Scaled scaled_exp2(float x) {
    if (!(x > neg_inf())) return {kSepNone, x < 0.f ? 0.f : x};  // NaN stays NaN
    const float r = rintf(x);
    return {(int)r, ex2(x - r)};
}
// e^x of a potential as it is returned (x = -inf: none), without another
// rounding of the size of the potential.
__device__ __forceinline__ Scaled scaled_exp(float x) {
    if (!(x > neg_inf())) return {kSepNone, x < 0.f ? 0.f : x};  // NaN stays NaN
    const double y = (double)x * 1.4426950408889634, r = rint(y);
    return {(int)r, ex2((float)(y - r))};
}
// mass / v, none where there is no mass.
__device__ __forceinline__ Scaled update(float mass, Scaled v) {
    Scaled u = {__builtin_amdgcn_frexp_expf(mass) - v.h, __builtin_amdgcn_frexp_mantf(mass) * __builtin_amdgcn_rcpf(v.f)};
    return mass > 0.f ? u : none();
}
// The natural logarithm in fp32; -inf for none.
__device__ __forceinline__ float scaled_ln(Scaled v) {
    return v.h > kSepNone ? __builtin_fmaf((float)v.h, kLn2, lg2(v.f) * kLn2) : neg_inf();
}
__device__ __forceinline__ float scaled_lg2(Scaled v) { return v.h > kSepNone ? (float)v.h + lg2(v.f) : neg_inf(); }
// v / w as a plain number.
__device__ __forceinline__ float ratio(Scaled v, Scaled w) {
    return __builtin_amdgcn_ldexpf(v.f * __builtin_amdgcn_rcpf(w.f), v.h - w.h);
}
__device__ __forceinline__ float product(Scaled v, Scaled w) { return __builtin_amdgcn_ldexpf(v.f * w.f, v.h + w.h); }
template <int N, class F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (N > 0) {
        unroll<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// One set of lines (one line per PO lanes of the wavefront): lane i of a line
// brings input x and takes output i, sum_i x_i 2^L (or its cost-weighted form).
// yb: 64 floats of the wavefront's own.
template <int PO, int BS>
__device__ __forceinline__ Scaled line_sum(const float *tab, const int *ref, float *yb, int lane, Scaled x) {
    constexpr int NB = PO / BS, NQ = PO / 16;
    const int o = lane & (PO - 1), base = lane & ~(PO - 1);
    // Table entries of the first 16 inputs and the block exponents: read ahead
    // of the dependent chain below.
    const f4s *tb = reinterpret_cast<const f4s *>(tab) + o;
    f4s e[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) e[g] = tb[g * PO];
    i4s lr[(NB + 3) / 4];
#pragma unroll
    for (int g = 0; g < (NB + 3) / 4; ++g) lr[g] = (reinterpret_cast<const i4s *>(ref) + o)[g * PO];
    const int rr = block_max<BS>(x.h);
    yb[lane] = __builtin_amdgcn_ldexpf(x.f, x.h - rr + kSepE0);
    // lane's block exponents: block J's on lane J of each 16-lane row
    const int R = NB == 1 ? rr : __builtin_amdgcn_ds_bpermute((base + BS * ((lane & 15) % NB)) << 2, rr);
    __builtin_amdgcn_wave_barrier();
    float y[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) y[q] = yb[base + 16 * q + (lane & 15)];
    // Exponents of the blocks, and their largest.
    int z[NB], m;
    unroll<NB>([&](auto j) {
        constexpr int J = decltype(j)::value;
        z[J] = (NB == 1 ? R : row_bcast<J>(R)) + lr[J / 4][J % 4];
        m = J == 0 ? z[J] : max(m, z[J]);
    });
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        float acc[4];
        fma16(acc, y[q], e);
        if (q + 1 < NQ) {
#pragma unroll
            for (int g = 0; g < 4; ++g) e[g] = tb[(4 * (q + 1) + g) * PO];
        }
        if (BS == 4) {
            const float s0 = __builtin_amdgcn_ldexpf(acc[0], z[(4 * q) % NB] - m),
                        s1 = __builtin_amdgcn_ldexpf(acc[1], z[(4 * q + 1) % NB] - m),
                        s2 = __builtin_amdgcn_ldexpf(acc[2], z[(4 * q + 2) % NB] - m),
                        s3 = __builtin_amdgcn_ldexpf(acc[3], z[(4 * q + 3) % NB] - m);
            s += (s0 + s1) + (s2 + s3);
        } else {
            const float t = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            s = NB == 1 ? t : s + __builtin_amdgcn_ldexpf(t, z[q % NB] - m);
        }
    }
    __builtin_amdgcn_wave_barrier();
    return {__builtin_amdgcn_frexp_expf(s) + (m - 2 * kSepE0), __builtin_amdgcn_frexp_mantf(s)};
}

// ---- all iterations of one problem in one work-group ----
//
// The plane [h2][ld] holds T (inputs of the u-update's line sums) and S (of
// the v-update's) in turn: a line sum reads one column (or row) and writes the
// same cells.  U takes the columns c of the first grid, V the rows r' of the
// second (u = 2^a, v = 2^b):
//   U: T[., c] -> u[., c] (u-update) -> S[c, .] = sum_r u[r, c] 2^(-A/lambda)
//   V: S[., r'] -> v[r', .] (v-update) -> T[r', .] = sum_{c'} v[r', c'] 2^(-B/lambda)
// The wavefronts take sets of lines in turn.
constexpr int kSepWaves = 16;
typedef int i2s __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Scaled get(const i2s *p) { return {(*p).x, __int_as_float((*p).y)}; }
__device__ __forceinline__ void put(i2s *p, Scaled v) { *p = i2s{v.h, __float_as_int(v.f)}; }
struct SepState {
    int w1, h1, w2, h2, ld, vld;  // row strides of the plane and of v's planes
    float *E[4];
    const int *Lr[4];
    i2s *plane;
    float *yb;
    int lane;
    const float *mu, *nu;  // of the problem, in memory (read again in every iteration: they stay in cache)
};

// start (null: none): S from these starting potentials (base 2) alone.
template <int PO, int BS>
__device__ __forceinline__ void sep_u(const SepState &S, int w, const float *start) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    for (int c0 = w * G; c0 < S.w1; c0 += kSepWaves * G) {
        const int c = c0 + lane / PO;
        const bool in1 = c < S.w1 && o < S.h1, in2 = c < S.w1 && o < S.h2;
        const int u1 = in1 ? o * S.w1 + c : 0, at = in2 ? o * S.ld + c : 0;
        Scaled u;
        if (start) {
            u = scaled_exp2(in1 ? start[u1] : neg_inf());
        } else {
            const float mui = S.mu[u1];
            const Scaled x = get(S.plane + at);
            u = update(in1 ? mui : 0.f, line_sum<PO, BS>(S.E[kTabU1], S.Lr[kTabU1], S.yb, lane, in2 ? x : none()));
        }
        const Scaled y = line_sum<PO, BS>(S.E[kTabU2], S.Lr[kTabU2], S.yb, lane, u);
        if (in2) put(S.plane + at, y);
    }
}

// What V does beside T: nothing; v kept; v kept and the iterate's error taken;
// the error alone (no T).  The error of (the current u, the old v): its columns
// sum to nu v_old / v_new, its rows fit.  Returns this lane's part.
// v is kept in `keep` and the old v read from `old` (planes [h2][vld], the same
// one or two), and as log2 in bout (null: none).
enum { kVPlain = 0, kVKeep = 1, kVKeepErr = 2, kVErr = 3 };
template <int PO, int BS>
__device__ __forceinline__ float sep_v(const SepState &S, int w, int what, const i2s *old, i2s *keep, float *bout) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    float err = 0.f;
    for (int r0 = w * G; r0 < S.h2; r0 += kSepWaves * G) {
        const int r = r0 + lane / PO;
        const bool in1 = r < S.h2 && o < S.w1, in2 = r < S.h2 && o < S.w2;
        const int at = in1 ? r * S.ld + o : 0, u2 = in2 ? r * S.w2 + o : 0;
        const float nuj = S.nu[u2];
        const Scaled x = get(S.plane + at);
        const Scaled v = update(in2 ? nuj : 0.f, line_sum<PO, BS>(S.E[kTabV1], S.Lr[kTabV1], S.yb, lane, in1 ? x : none()));
        if (what != kVPlain) {
            if (what >= kVKeepErr && in2)  // a column without mass is empty: its error is |nu|, NaN where nu is
                err += nuj > 0.f ? fabsf(__builtin_fmaf(nuj, ratio(get(old + r * S.vld + o), v), -nuj)) : fabsf(nuj);
            if (what == kVErr) continue;
            if (in2) {
                put(keep + r * S.vld + o, v);
                if (bout) bout[u2] = scaled_lg2(v);
            }
        }
        const Scaled y = line_sum<PO, BS>(S.E[kTabV2], S.Lr[kTabV2], S.yb, lane, v);
        if (in1) put(S.plane + at, y);
    }
    return err;
}

// The results of the returned iterate from its v (a plane, or log2 in bin):
// T and its B-weighted form in tw; then, per entry of the first grid, the row
// sums give u, and with T weighted by A the loss sum_ij P_ij C_ij, C = A + B.
// E[kTabV1] and E[kTabU2] hold the weighted tables by now.
template <int PO, int BS>
__device__ __forceinline__ void sep_result_v(const SepState &S, int w, const i2s *v, const float *bin, i2s *tw,
                                             float *beta) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    for (int r0 = w * G; r0 < S.h2; r0 += kSepWaves * G) {
        const int r = r0 + lane / PO;
        const bool in1 = r < S.h2 && o < S.w1, in2 = r < S.h2 && o < S.w2;
        const int u2 = in2 ? r * S.w2 + o : 0;
        Scaled x = none();
        if (in2) {
            x = bin ? scaled_exp2(bin[u2]) : get(v + r * S.vld + o);
            beta[u2] = scaled_ln(x);
        }
        const Scaled y = line_sum<PO, BS>(S.E[kTabV2], S.Lr[kTabV2], S.yb, lane, x);
        const Scaled yw = line_sum<PO, BS>(S.E[kTabV1], S.Lr[kTabV2], S.yb, lane, x);
        if (in1) {
            put(S.plane + r * S.ld + o, y);
            put(tw + r * S.vld + o, yw);
        }
    }
}
template <int PO, int BS>
__device__ __forceinline__ float sep_result_u(const SepState &S, int w, const i2s *tw, float *alpha) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    float loss = 0.f;
    for (int c0 = w * G; c0 < S.w1; c0 += kSepWaves * G) {
        const int c = c0 + lane / PO;
        const bool in1 = c < S.w1 && o < S.h1, in2 = c < S.w1 && o < S.h2;
        const int at = in2 ? o * S.ld + c : 0, wat = in2 ? o * S.vld + c : 0;
        const float mui = in1 ? S.mu[o * S.w1 + c] : 0.f;
        const Scaled x = in2 ? get(S.plane + at) : none(), xw = in2 ? get(tw + wat) : none();
        const Scaled sum = line_sum<PO, BS>(S.E[kTabU1], S.Lr[kTabU1], S.yb, lane, x);
        const Scaled sa = line_sum<PO, BS>(S.E[kTabU2], S.Lr[kTabU1], S.yb, lane, x);
        const Scaled sb = line_sum<PO, BS>(S.E[kTabU1], S.Lr[kTabU1], S.yb, lane, xw);
        if (in1) alpha[o * S.w1 + c] = scaled_ln(update(mui, sum));
        if (mui > 0.f) loss = __builtin_fmaf(mui, ratio(sa, sum) + ratio(sb, sum), loss);
    }
    return loss;
}

// The marginal error of the returned potentials.  They are rounded to fp32,
// which moves the plan's row and column sums by 2^-24 of the potentials' size, up
// to 1e-5 in all at thousands of units; the early stop measures the iterate
// itself, as in exact arithmetic.  Three sets of lines, once per problem:
//   V: T of e^beta   U: the rows' error under e^alpha, and S   V: the columns'
template <int PO, int BS>
__device__ __forceinline__ void sep_error_T(const SepState &S, int w, const float *beta) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    for (int r0 = w * G; r0 < S.h2; r0 += kSepWaves * G) {
        const int r = r0 + lane / PO;
        const bool in1 = r < S.h2 && o < S.w1, in2 = r < S.h2 && o < S.w2;
        const Scaled x = in2 ? scaled_exp(beta[r * S.w2 + o]) : none();
        const Scaled y = line_sum<PO, BS>(S.E[kTabV2], S.Lr[kTabV2], S.yb, lane, x);
        if (in1) put(S.plane + r * S.ld + o, y);
    }
}
template <int PO, int BS>
__device__ __forceinline__ float sep_error_rows(const SepState &S, int w, const float *alpha) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    float err = 0.f;
    for (int c0 = w * G; c0 < S.w1; c0 += kSepWaves * G) {
        const int c = c0 + lane / PO;
        const bool in1 = c < S.w1 && o < S.h1, in2 = c < S.w1 && o < S.h2;
        const int u1 = in1 ? o * S.w1 + c : 0, at = in2 ? o * S.ld + c : 0;
        const float mui = in1 ? S.mu[u1] : 0.f;
        const Scaled u = in1 ? scaled_exp(alpha[u1]) : none();
        const Scaled sum = line_sum<PO, BS>(S.E[kTabU1], S.Lr[kTabU1], S.yb, lane, in2 ? get(S.plane + at) : none());
        if (mui > 0.f) err += fabsf(product(u, sum) - mui);
        const Scaled y = line_sum<PO, BS>(S.E[kTabU2], S.Lr[kTabU2], S.yb, lane, u);
        if (in2) put(S.plane + at, y);
    }
    return err;
}
template <int PO, int BS>
__device__ __forceinline__ float sep_error_cols(const SepState &S, int w, const float *beta) {
    constexpr int G = 64 / PO;
    const int lane = S.lane, o = lane & (PO - 1);
    float err = 0.f;
    for (int r0 = w * G; r0 < S.h2; r0 += kSepWaves * G) {
        const int r = r0 + lane / PO;
        const bool in1 = r < S.h2 && o < S.w1, in2 = r < S.h2 && o < S.w2;
        const int u2 = in2 ? r * S.w2 + o : 0;
        const Scaled x = in1 ? get(S.plane + r * S.ld + o) : none();
        const Scaled sum = line_sum<PO, BS>(S.E[kTabV1], S.Lr[kTabV1], S.yb, lane, x);
        if (in2) err += fabsf(product(scaled_exp(beta[u2]), sum) - S.nu[u2]);
    }
    return err;
}

// Calls f(lanes of a line, block size) with both as constants.
template <int POMAX, class F>
__device__ __forceinline__ void with_shape(int po, int bs, F &&f) {
    using std::integral_constant;
    if (bs == 16) {
        if (po == 16)
            f(integral_constant<int, 16>{}, integral_constant<int, 16>{});
        else if (POMAX == 32 || po == 32)
            f(integral_constant<int, 32>{}, integral_constant<int, 16>{});
        else
            f(integral_constant<int, 64>{}, integral_constant<int, 16>{});
    } else {
        if (po == 16)
            f(integral_constant<int, 16>{}, integral_constant<int, 4>{});
        else if (POMAX == 32 || po == 32)
            f(integral_constant<int, 32>{}, integral_constant<int, 4>{});
        else
            f(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    }
}

// LDS floats of sk_sep_solve: four tables (po^2 entries and po^2 / 4 block
// exponents), the plane, v (and T weighted by the cost at the end), a second v
// where lines have at most 32 entries, and the wavefronts' buffers.
__host__ __device__ inline int sep_vplane(int w1, int h2, int w2) { return h2 * (w2 > (w1 | 1) ? w2 : (w1 | 1)); }
__host__ __device__ inline int sep_lds_floats(int w1, int h1, int w2, int h2) {
    const int pu = sep_lanes(h1, h2), pv = sep_lanes(w1, w2);
    const int tab = 2 * (pu * pu + pv * pv) * 5 / 4, planes = pu == 64 || pv == 64 ? 1 : 2;
    return tab + 2 * h2 * (w1 | 1) + planes * 2 * sep_vplane(w1, h2, w2) + kSepWaves * 65;
}

// Sum over the work-group in a fixed order; `red` holds kSepWaves floats.
__device__ __forceinline__ float group_sum(float v, float *red) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kSepWaves; ++w) s += red[w];
    return s;
}

// Every iteration of one problem whose cost splits over two axes, and its
// results, one work-group per problem.  The problem is marked as stopped after
// its K iterations: the launches that follow skip it.
// Bound by the chain of its line sums (LDS round trips and two barriers per
// iteration; 16 wavefronts on one CU) and, for 64-entry lines in blocks of 4,
// by vector issue.  Measured per iteration: 3.1 us for up to 256 problems of
// 28 x 28 (sweep and merge before: 50.9), 21 us for 64 problems of 64 x 64
// (236.9).  The rest of a call is the two empty launches per iteration, 3.3 to
// 5.4 us: more than the solve where problems are small (28 x 28: 4.0 of 7.1).
__device__ __forceinline__ void sep_table_in(float *dst, const float *src, int n) {
    for (int u = threadIdx.x; u < n / 4; u += 64 * kSepWaves)
        reinterpret_cast<f4s *>(dst)[u] = reinterpret_cast<const f4s *>(src)[u];
}

template <int POMAX>
__global__ __launch_bounds__(64 * kSepWaves, 4) void sk_sep_solve(SepArgs T) {
    extern __shared__ float lds[];
    const int bs = T.mode[0];
    if (bs == 0) return;
    SepState S;
    S.w1 = T.mode[1];
    S.w2 = T.mode[2];
    S.h1 = T.d1 / S.w1;
    S.h2 = T.d2 / S.w2;
    S.ld = S.w1 | 1;
    S.vld = S.w2 > S.ld ? S.w2 : S.ld;
    const int pu = sep_lanes(S.h1, S.h2), pv = sep_lanes(S.w1, S.w2);
    if ((pu > pv ? pu : pv) == 64 != (POMAX == 64)) return;  // the other kernel's
    float *at = lds;
#pragma unroll
    for (int t = 0; t < 4; ++t) {  // the tables: E then Lr
        const int po = t < 2 ? pu : pv;
        sep_table_in(at, T.table + t * kSepTable, po * po);
        sep_table_in(at + po * po, T.table + t * kSepTable + kSepLine * kSepLine, po * po / 4);
        S.E[t] = at;
        S.Lr[t] = reinterpret_cast<const int *>(at + po * po);
        at += po * po * 5 / 4;
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    S.yb = at + w * 64;
    at += kSepWaves * 64;
    float *red = at;
    at += kSepWaves;
    S.plane = reinterpret_cast<i2s *>(at);
    // v of two iterates (lines of up to 32), or of one: an iterate that may be
    // the returned one then also goes to memory, as log2.
    i2s *v0 = S.plane + S.h2 * S.ld, *v1 = POMAX == 32 ? v0 + sep_vplane(S.w1, S.h2, S.w2) : v0;
    const size_t p = blockIdx.x, bplane = (size_t)T.B * T.d2p;
    S.mu = T.mu + p * T.d1;
    S.nu = T.nu + p * T.d2;
    float *alpha = T.a + p * T.d1, *beta = T.beta + p * T.d2, *b = T.bbuf + p * T.d2p;
    const int n = T.n_iter;
    const bool stops = T.tol > 0.f;
    __syncthreads();
    int k = 0;
    float err = 0.f;
    for (;; ++k) {
        // Opaque to the compiler, so that no shape's addresses are kept in
        // registers across the iterations.
        S.lane = threadIdx.x & 63;
        __asm__ volatile("" : "+v"(S.lane));
        // u of iteration k (k = 0: the starting potentials) and S.
        with_shape<POMAX>(pu, bs, [&](auto po, auto bl) {
            sep_u<decltype(po)::value, decltype(bl)::value>(S, w, k == 0 ? alpha : nullptr);
        });
        __syncthreads();
        // v of iteration k + 1, which measures iterate k, and T.
        const int what = k == n ? kVErr : stops ? (k > 0 ? kVKeepErr : kVKeep) : k + 1 == n ? kVKeep : kVPlain;
        with_shape<POMAX>(pv, bs, [&](auto po, auto bl) {
            err = sep_v<decltype(po)::value, decltype(bl)::value>(
                S, w, what, k & 1 ? v1 : v0, k & 1 ? v0 : v1,
                POMAX == 64 && stops ? b + ((k + 1) & 1) * bplane : nullptr);
        });
        if (what >= kVKeepErr) {
            err = group_sum(err, red);
            if (k == n || err <= T.tol) break;
        } else {
            __syncthreads();
        }
    }
    // The weighted tables in the place of the two that the results do not need.
    __syncthreads();
    sep_table_in(S.E[kTabU2], T.table + kTabWU * kSepTable, pu * pu);
    sep_table_in(S.E[kTabV1], T.table + kTabWV * kSepTable, pv * pv);
    __syncthreads();
    // v of iterate k; the other plane takes the weighted T (of one plane, each
    // wavefront writes where it alone has read).
    const float *bin = POMAX == 64 && stops && k < n ? b + (k & 1) * bplane : nullptr;
    i2s *tw = k & 1 ? v0 : v1;
    with_shape<POMAX>(pv, bs, [&](auto po, auto bl) {
        sep_result_v<decltype(po)::value, decltype(bl)::value>(S, w, k & 1 ? v1 : v0, bin, tw, beta);
    });
    __syncthreads();
    float loss = 0.f;
    with_shape<POMAX>(pu, bs, [&](auto po, auto bl) {
        loss = sep_result_u<decltype(po)::value, decltype(bl)::value>(S, w, tw, alpha);
    });
    loss = group_sum(loss, red);
    // And back, for the error of what is returned.
    sep_table_in(S.E[kTabU2], T.table + kTabU2 * kSepTable, pu * pu);
    sep_table_in(S.E[kTabV1], T.table + kTabV1 * kSepTable, pv * pv);
    with_shape<POMAX>(pv, bs, [&](auto po, auto bl) {
        sep_error_T<decltype(po)::value, decltype(bl)::value>(S, w, beta);
    });
    __syncthreads();
    with_shape<POMAX>(pu, bs, [&](auto po, auto bl) {
        err = sep_error_rows<decltype(po)::value, decltype(bl)::value>(S, w, alpha);
    });
    __syncthreads();
    with_shape<POMAX>(pv, bs, [&](auto po, auto bl) {
        err += sep_error_cols<decltype(po)::value, decltype(bl)::value>(S, w, beta);
    });
    err = group_sum(err, red);
    if (threadIdx.x == 0) {
        T.loss[p] = (float)ldexp((double)loss / (double)T.s, kSepWeight);
        T.merr[p] = err;
        T.iters[p] = k;
        T.state[p] = k;
    }
}

template <int POMAX>
hipError_t launch_solve(const SepArgs &P, size_t lds, hipStream_t st) {
    if (lds == 0) return hipSuccess;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&sk_sep_solve<POMAX>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(sk_sep_solve<POMAX>, dim3(P.B), dim3(64 * kSepWaves), lds, st, P);
    return hipSuccess;
}

}  // namespace

bool separable_plan(int B, int d1, int d2, int n_iter, size_t table_bytes, SepArgs *P) {
    *P = SepArgs{};
    if (table_bytes < kTables * sizeof(float) * kSepTable) return false;
    // Both sides measured on the MI355X, in microseconds.  An iteration of the
    // sweeps: 10 for its two launches and 1 per 4.5e6 cells of the batch.  Of
    // the solve: 1.2 and 38e-6 per half cell of a problem (14 x 14: 1.2, 28 x 28:
    // 3.1, 64 x 64: 21.0 in blocks of 4, 16.2 in blocks of 16) for every 256
    // problems (one work-group per CU), and for the two empty launches 3.3 to 5.4
    // (whole calls' time per iteration less the solve's), taken as 3.8: at the
    // line the solve is ahead, 40 x 40, two problems, 13.1 and 15.1; 64 x 64, five
    // problems, 24.3 and 50.1.  The test of the cost, when it fails: 16, and one
    // read of the cost; it must stay below 1 % of the sweeps.
    const double cells = (double)d1 * d2, sweeps = 10.0 + cells * B / 4.5e6;
    if (n_iter * sweeps < 100.0 * (16.0 + cells / 1e6)) return false;
    int most = 0;
    for (int w1 = 2; w1 <= kSepLine; ++w1) {
        if (d1 % w1) continue;
        for (int w2 = 2; w2 <= kSepLine; ++w2) {
            if (!sep_pair_ok(d1, d2, w1, w2)) continue;
            const int h1 = d1 / w1, h2 = d2 / w2, half = sep_half_cells(w1, h1, w2, h2);
            const size_t x = sizeof(float) * sep_lds_floats(w1, h1, w2, h2);
            size_t &y = sep_lanes(h1, h2) == 64 || sep_lanes(w1, w2) == 64 ? P->lds64 : P->lds32;
            y = y > x ? y : x;
            most = most > half ? most : half;
        }
    }
    if (!most || 3.8 + (1.2 + 38e-6 * most) * ((B + 255) / 256) >= sweeps) return false;
    return true;
}

hipError_t launch_separable(const SepArgs &P, hipStream_t st) {
    hipLaunchKernelGGL(sk_sep_guess, dim3(1), dim3(kGuessThreads), 0, st, P.C, P.d1, P.d2, P.mode);
    hipLaunchKernelGGL(sk_sep_verify, dim3(P.d1 < 4096 ? (P.d1 + 3) / 4 : 1024), dim3(256), 0, st, P.C, P.d1, P.d2, P.s,
                       P);
    hipLaunchKernelGGL(sk_sep_tables, dim3(kTables), dim3(256), 0, st, P.C, P.d1, P.d2, P.s, P);
    const hipError_t e = launch_solve<32>(P, P.lds32, st);
    return e != hipSuccess ? e : launch_solve<64>(P, P.lds64, st);
}

}  // namespace sk
