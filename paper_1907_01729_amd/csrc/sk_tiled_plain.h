// sk_tiled_plain.h -- the plain form u = mu / (K v), v = nu / (K^T u) on the
// matrix cores, for large supports with a shared cost (included by
// sk_tiled.hip; TiledArgs and the helpers it uses are defined there).
//
// K = 2^(-s (C - min C)) is the same for the whole batch, so a half-step is a
// matrix product of K with all the batch's scalings.  It is taken where the
// scaled cost spans at most 64 bits (as in the resident kernels).  Every sum is
// then within [2^-64, 1] of the sum of its operand's scalings, whose product
// stays within [1, 2^64]; a sum that leaves [2^-80, 2^100] all the same (no mass
// on one side, or masses that are not finite) marks its problem, which is
// solved again in the log domain (sk_plain_finish).
//
// Masses that do not sum to one would move the scalings by the ratio of their
// sums in every iteration.  They are divided by their sums first; with masses
// f1 mu and f2 nu in the place of mu and nu the iteration gives u_k (f1/f2)^k
// and v_k f2 (f2/f1)^(k-1), which the returned potentials take back.  (Sums
// that move nothing by more than 8 bits in all are left as they are.)
//
// Scalings are not guarded (the resident kernels guard both): a small mass may
// give one below 2^-126, where it has few bits or none.  As an operand that
// does not matter: it is off by less than 2^-126, K <= 1, and the sums it goes
// into are at least 2^-80, so d of them move a sum by less than d 2^-46 of it.
// And the returned potentials are not taken from scalings but from the last
// sums, log2 mass - log2 sum (mass and sum as mantissa and exponent, so that
// nothing underflows).
//
// The launches are those of the sweeps (sweep: u-update, merge: v-update), so
// a cost out of range costs nothing per iteration: in range, every problem's
// state is kPlainState and the kernels that would skip a stopped problem run
// the products instead.
//
// fp32 products on v_mfma_f32_32x32x2_f32: a work-group takes 32 rows by 32
// problems and splits the contraction over its wavefronts, whose partial tiles
// meet in LDS.  K is kept in both orders and the scalings as [support][batch],
// all padded with zeros to multiples of 32, so every operand load is two runs
// of 128 bytes and nothing is masked; rows lie an odd number of 256-byte lines
// apart, so that a column's rows spread over the L2's channels.  Measured on
// 256 problems of 1000 x 1000: 12.5 and 13.4 us for the two launches (sweep
// and merge: 64.6 and 5.8), 4.3 of each the launch, the setup and the merge;
// the matrix cores alone would take 3.3, the loads of the operands set the pace.
#pragma once

typedef float f16v __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int32_t ordered(float x) {
    const int32_t i = __float_as_int(x);
    return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ __forceinline__ float unordered(int32_t i) { return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff); }

// Work-groups below kPlainRangeGroups: smallest and largest entry of the cost
// (one that is not finite fails the test in plain_fits through range[3]).  The
// others, one per problem: the factors f1, f2 of its masses.
constexpr int kPlainRangeGroups = 128;
__global__ __launch_bounds__(256) void sk_plain_range(TiledArgs T) {
    if (splits(T)) return;
    __shared__ float least[4], most[4];
    if (blockIdx.x >= kPlainRangeGroups) {
        const int b = (int)blockIdx.x - kPlainRangeGroups;
        float m1 = 0.f, m2 = 0.f;
        for (int i = threadIdx.x; i < T.d1; i += 256) m1 += fmaxf(T.mu[(size_t)b * T.d1 + i], 0.f);
        for (int j = threadIdx.x; j < T.d2; j += 256) m2 += fmaxf(T.nu[(size_t)b * T.d2 + j], 0.f);
        m1 = block_sum_n<256>(m1, least);
        m2 = block_sum_n<256>(m2, most);
        if (threadIdx.x != 0) return;
        const float l1 = log2f(m1), l2 = log2f(m2), f1 = 1.f / m1, f2 = 1.f / m2;
        const bool far = fabsf(l1 - l2) * (float)T.n_iter + fabsf(l1) + fabsf(l2) > 8.f;  // (NaN: not)
        const bool usable = f1 > 0.f && f2 > 0.f && f1 < __builtin_inff() && f2 < __builtin_inff();
        T.plain.factor[2 * b] = far && usable ? f1 : 1.f;
        T.plain.factor[2 * b + 1] = far && usable ? f2 : 1.f;
        return;
    }
    const size_t n = (size_t)T.d1 * T.d2, step = (size_t)kPlainRangeGroups * 256;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    bool bad = false;
    for (size_t u = (size_t)blockIdx.x * 256 + threadIdx.x; u < n; u += 8 * step) {
        float c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q] = T.C[u + q * step < n ? u + q * step : u];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            lo = fminf(lo, c[q]);
            hi = fmaxf(hi, c[q]);
            bad = bad || !(fabsf(c[q]) < __builtin_inff());
        }
    }
    const int w = threadIdx.x >> 6;
    lo = -wave_max(-lo);
    hi = wave_max(hi);
    if ((threadIdx.x & 63) == 0) {
        least[w] = lo;
        most[w] = hi;
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) {  // one pair of atomics per work-group: they meet on one line
        atomicMin(T.plain.range + 0, ordered(fminf(fminf(least[0], least[1]), fminf(least[2], least[3]))));
        atomicMax(T.plain.range + 1, ordered(fmaxf(fmaxf(most[0], most[1]), fmaxf(most[2], most[3]))));
        if (bad) atomicOr(T.plain.range + 3, 1);
    }
}
// The decision, the same in every kernel between sk_plain_range and the setup.
__device__ __forceinline__ bool plain_fits(const TiledArgs &T) {
    if (splits(T) || T.plain.range[3] != 0) return false;
    const float lo = unordered(T.plain.range[0]), hi = unordered(T.plain.range[1]);
    return T.s * (hi - lo) <= kPlainSpan;
}

// K in both orders, the masses transposed, u = 1 on the support of mu, v = 0,
// and every problem's state.  Work-groups of 32 x 32 tiles: first K's, then
// mu's and nu's (the transpose goes through LDS).
__global__ __launch_bounds__(256) void sk_plain_setup(TiledArgs T) {
    __shared__ float tile[32][33];
    if (!plain_fits(T)) return;
    const PlainArgs &P = T.plain;
    const float lo = unordered(P.range[0]);
    const int n1 = P.p1 / 32, n2 = P.p2 / 32, nb = P.pb / 32;
    const int tiles = n1 * n2 + nb * (n1 + n2);
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        const bool cost = t < n1 * n2;
        const int u = t - n1 * n2;
        const bool first = u < nb * n1;  // mu's
        const int v = first ? u : u - nb * n1;
        // tile (row, column) of a [rows][cols] source: K from C, else a mass [B][d]
        const int rows = cost ? T.d1 : T.B, cols = cost ? T.d2 : (first ? T.d1 : T.d2);
        const int nc = cost ? n2 : (first ? n1 : n2);
        const int r0 = (cost ? t / nc : v / nc) * 32, c0 = (cost ? t % nc : v % nc) * 32;
        const float *src = cost ? T.C : (first ? T.mu : T.nu);
        for (int y = ty; y < 32; y += 8) {
            const int r = r0 + y, c = c0 + tx;
            float x = 0.f;
            if (r < rows && c < cols) {
                x = src[(size_t)r * cols + c];
                if (!cost) x *= P.factor[2 * r + (first ? 0 : 1)];
                if (cost) {  // 2^(-s (C - lo)), the integer part of the exponent kept apart
                    const double e = -(double)T.s * ((double)x - (double)lo), f = floor(e);
                    x = ldexpf(exp2f((float)(e - f)), (int)f);
                    P.K[(size_t)r * P.l2 + c] = x;
                }
            } else if (cost) {
                P.K[(size_t)r * P.l2 + c] = 0.f;
            }
            tile[y][tx] = x;
        }
        __syncthreads();
        for (int y = ty; y < 32; y += 8) {
            const int r = c0 + y, c = r0 + tx;  // transposed
            const float x = tile[tx][y];
            if (cost) {
                P.Kt[(size_t)r * P.l1 + c] = x;
            } else {
                const size_t at = (size_t)r * P.lb + c;
                (first ? P.mut : P.nut)[at] = x;
                (first ? P.Ut : P.Vt)[at] = first && x > 0.f ? 1.f : 0.f;
            }
        }
        __syncthreads();
    }
    for (int b = blockIdx.x * 256 + threadIdx.x; b < T.B; b += gridDim.x * 256) {
        T.state[b] = kPlainState;
        plain_bad(P, T.B)[b] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) P.range[2] = 1;
}
__device__ __forceinline__ bool plain_taken(const TiledArgs &T) { return T.plain.range && T.plain.range[2] != 0; }

// out[m][n] = mass[m][n] / sum_k A[k][m] X[k][n] over m < M, n < N in tiles of
// 32 x 32: work-groups wg, wg + nwg, ... of NW wavefronts; lds: NW * 1024
// floats.  kd is a multiple of 32; out's rows and columns past its size keep
// 0.  SUMS: the sums take the masses' place, for the potentials.  One batch of
// loads is in flight beside a batch's products: bound by those loads (20 cycles
// per 256 bytes and CU), so loading further ahead only adds batches that are
// thrown away (15.2 us with three more, 12.7 so).
constexpr int kPlainUnroll = 8;  // matrix instructions (2 of the contraction each) per batch of loads
template <int NW, bool SUMS>
__device__ __forceinline__ void plain_product(const float *A, int lda, const float *X, float *mass, float *out,
                                              int ldx, int kd, int M, int N, int32_t *bad, float *lds, int wg,
                                              int nwg) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Consecutive work-groups go to the 8 XCDs in turn: a row tile stays on one
    // XCD, whose L2 then keeps its share of K over the iterations.
    const int nt = (N + 31) / 32, mt = (M + 31) / 32, tiles = (mt + 7) / 8 * 8 * nt;
    for (int t = wg; t < tiles; t += nwg) {
        const int mi = (t & 7) + 8 * ((t >> 3) / nt), m0 = mi * 32, n0 = (t >> 3) % nt * 32;
        if (mi >= mt) continue;  // work-group uniform
        // This wavefront's batches of the contraction: w, w + NW, ...
        constexpr int KB = 2 * kPlainUnroll;
        const float *a = A + (size_t)(lane >> 5) * lda + m0 + (lane & 31);
        const float *x = X + (size_t)(lane >> 5) * ldx + n0 + (lane & 31);
        f16v acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float av[kPlainUnroll], xv[kPlainUnroll];
        auto load = [&](int k) {
#pragma unroll
            for (int q = 0; q < kPlainUnroll; ++q) {
                av[q] = a[(size_t)(k + 2 * q) * lda];
                xv[q] = x[(size_t)(k + 2 * q) * ldx];
            }
        };
        int k = w * KB;
        if (k < kd) load(k);
        for (; k < kd; k += NW * KB) {
            float ac[kPlainUnroll], xc[kPlainUnroll];
#pragma unroll
            for (int q = 0; q < kPlainUnroll; ++q) {
                ac[q] = av[q];
                xc[q] = xv[q];
            }
            load(k + NW * KB < kd ? k + NW * KB : k);  // the next batch, in flight over this one's products
#pragma unroll
            for (int q = 0; q < kPlainUnroll; ++q)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ac[q], xc[q], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)  // row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
            lds[w * 1024 + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[r];
        __syncthreads();
        for (int u = threadIdx.x; u < 1024; u += 64 * NW) {
            const int m = m0 + (u >> 5), n = n0 + (u & 31);
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < NW; ++q) s += lds[q * 1024 + u];
            if (m < M && n < N) {
                const size_t at = (size_t)m * ldx + n;
                const float mm = mass[at];
                float v = 0.f;
                if (mm > 0.f) {
                    if (!(s >= kPlainLo && s <= kPlainHi)) bad[n] = 1;
                    v = mm * __builtin_amdgcn_rcpf(s);
                }
                out[at] = v;
                if (SUMS) mass[at] = s;
            }
        }
        __syncthreads();
    }
}
template <int NW, bool SUMS>
__device__ __forceinline__ void plain_u(const TiledArgs &T, float *lds, int wg, int nwg) {
    const PlainArgs &P = T.plain;
    plain_product<NW, SUMS>(P.Kt, P.l1, P.Vt, P.mut, P.Ut, P.lb, P.p2, T.d1, T.B, plain_bad(P, T.B), lds, wg, nwg);
}
template <int NW, bool SUMS>
__device__ __forceinline__ void plain_v(const TiledArgs &T, float *lds, int wg, int nwg) {
    const PlainArgs &P = T.plain;
    plain_product<NW, SUMS>(P.K, P.l2, P.Ut, P.nut, P.Vt, P.lb, P.p1, T.d2, T.B, plain_bad(P, T.B), lds, wg, nwg);
}
// The first v-update.
template <bool SUMS>
__global__ __launch_bounds__(512) void sk_plain_first(TiledArgs T) {
    extern __shared__ float lds[];
    if (!plain_taken(T)) return;
    plain_v<8, SUMS>(T, lds, (int)blockIdx.x, (int)gridDim.x);
}
// The last u-update (8 wavefronts, as beside the sweeps) or v-update (4, as
// beside the merges), keeping the sums.  Launches of their own: a test for the
// last one in the iteration's launches moved the sweep's code, 1.2 % on a cost
// out of range.
template <int NW, bool ROWS>
__global__ __launch_bounds__(64 * NW) void sk_plain_last(TiledArgs T) {
    extern __shared__ float lds[];
    if (!plain_taken(T)) return;
    if (ROWS)
        plain_u<NW, true>(T, lds, (int)blockIdx.x, (int)gridDim.x);
    else
        plain_v<NW, true>(T, lds, (int)blockIdx.x, (int)gridDim.x);
}

// log2(mass / sum), -inf without mass, to half a unit in the last place: the
// hardware's logarithm of a mantissa alone, added to the exponent (of the whole
// number it is off by a unit of the result, 2e-6 at 2^-20).
__device__ __forceinline__ float plain_potential(float mass, float sum) {
    if (!(mass > 0.f)) return neg_inf();
    const float q = __builtin_amdgcn_frexp_mantf(mass) * __builtin_amdgcn_rcpf(__builtin_amdgcn_frexp_mantf(sum));
    const int e = __builtin_amdgcn_frexp_expf(mass) - __builtin_amdgcn_frexp_expf(sum) + __builtin_amdgcn_frexp_expf(q);
    return (float)e + lg2(__builtin_amdgcn_frexp_mantf(q));
}
