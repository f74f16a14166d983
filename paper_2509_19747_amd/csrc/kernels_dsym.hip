// Matvec with a large stored symmetric matrix: y = A u + mu u reading the upper triangle
// once (half the bytes of the whole matrix, which bound this product), every element
// used for its row and its column.
//
// Rows and columns go in blocks of 256.  Work item (I, r): row block I against the
// column blocks J = I + r m .. I + r m + m - 1.  A wave takes 16 columns at a time, its
// 64 lanes holding four rows each: the row sums stay in registers over the item, the 16
// column sums are added over the lanes by a reduce-scatter.  The partial slots and the
// finish are those of the kernel matvec (k_ksym_mma): row sums of run r to slot I + r,
// column sums to slot I of the columns, or to slot nb inside the diagonal block, where
// only i <= j counts (i < j for the column sums).
//
// Measured against k_dense_matvec, which reads the whole matrix, in us:
//   float32: n = 5000 18.2 (17.5), 6000 21.4 (23.2), 8192 35 (39), 12000 60 (126),
//            16384 97 (180: 5.5 TB/s of the triangle), 30000 338 (700)
//   float64: n = 3001 17.5 (12.7), 4096 19.2 (21.6), 8192 62 (92), 10001 84 (322: columns
//            off 16-byte boundaries), 16384 188 (354), 30000 602 (1345)
// Below, the two launches and the fewer bytes in flight cost more than the lower
// triangle does: DENSE_SYM_MIN32, DENSE_SYM_MIN64.  Eight waves a block: with four, each
// has twice the columns to walk (float32, n = 6000: 25.3 us; 16384: 101).
#include "common.hpp"
#include "kernels.hpp"
#include "prof.hpp"

#include <algorithm>
#include <type_traits>

namespace rr {

constexpr int DS_RB = 256, DS_WAVES = 8, DS_THREADS = 64 * DS_WAVES, DS_COLS = 16, DS_BATCH = 8;

struct DsPlan {
    int nb, m;
    int items;
};
// Runs of two blocks once that leaves a block of work per compute unit (halves the row
// partials; float32, n = 7000: 24.1 us against 26.4, 16384: 98 against 107; four: 107).
static DsPlan ds_plan(int64_t n) {
    DsPlan p;
    p.nb = (int)((n + DS_RB - 1) / DS_RB);
    p.m = (int64_t)p.nb * (p.nb + 1) / 2 < 256 ? 1 : 2;
    p.items = 0;
    for (int I = 0; I < p.nb; ++I) p.items += (p.nb - I + p.m - 1) / p.m;
    return p;
}

// The lane's four rows within a row block: a 16-byte load each (float: rows 4 l .. 4 l + 3,
// double: 2 l, 2 l + 1 and 128 more), or with VEC false (columns not on 16-byte
// boundaries) one element at a time, rows l + 64 k.
template <typename TA, bool VEC>
RR_DEV int ds_row(int lane, int k) {
    if (!VEC) return lane + 64 * k;
    return sizeof(TA) == 4 ? 4 * lane + k : 128 * (k >> 1) + 2 * lane + (k & 1);
}

// NT: the triangle does not fit the last-level cache, so its loads bypass it (u and the
// partials keep their place).
template <typename TA, bool VEC, bool NT>
__global__ __launch_bounds__(DS_THREADS) void k_dense_sym(int64_t n, const TA* __restrict__ A, int64_t lda,
                                                          const double* __restrict__ u, double* __restrict__ part, int nb,
                                                          int m, const int32_t* __restrict__ stop) {
    __shared__ double rs[DS_WAVES][DS_RB];
    if (stop && *stop) return;
    int t = blockIdx.x, bi = 0;   // (at most a few hundred row blocks)
    {
        // row block of the item: counted from the end the row blocks come in groups of m
        // with ceil(k / m) runs each
        const int a0 = nb / m, r = m * (a0 * (a0 + 1) / 2) + (nb - a0 * m) * (a0 + 1) - 1 - t;
        int a = __builtin_amdgcn_readfirstlane((int)((__builtin_sqrtf(8.0f * (float)(r / m) + 1.0f) - 1.0f) * 0.5f));
        while (m * (a * (a + 1) / 2) > r) --a;
        while (m * ((a + 1) * (a + 2) / 2) <= r) ++a;
        const int rest = r - m * (a * (a + 1) / 2), b = rest / (a + 1);
        bi = nb - (a * m + b + 1);
        t = a - (rest - b * (a + 1));   // the run
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t i0 = (int64_t)bi * DS_RB;
    const bool whole = i0 + DS_RB <= n;
    double ui[4], acc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t i = i0 + ds_row<TA, VEC>(lane, k);
        ui[k] = i < n ? u[i] : 0.0;
        acc[k] = 0.0;
    }
    // one group of 16 columns; WIDE: whole rows in wide loads; EDGE: the diagonal block or
    // columns past n (the branches stand outside: loads behind them would wait singly)
    double cs[DS_COLS];
    auto group = [&](auto wide, auto edge, int64_t j0, bool diag) {
#pragma unroll
        for (int b = 0; b < DS_COLS; b += DS_BATCH) {
            TA a[DS_BATCH][4];
            double ub = 0.0;   // u of the columns, one per lane
            if constexpr (edge) ub = u[std::min<int64_t>(j0 + b + (lane & (DS_BATCH - 1)), n - 1)];
#pragma unroll
            for (int c = 0; c < DS_BATCH; ++c) {
                const int64_t j = j0 + b + c;
                const TA* col = A + i0 + (edge ? std::min<int64_t>(j, n - 1) : j) * lda;
                if constexpr (!wide) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int64_t i = ds_row<TA, VEC>(lane, k);
                        a[c][k] = col[std::min<int64_t>(i, n - 1 - i0)];
                    }
                } else if constexpr (sizeof(TA) == 4) {
                    typedef float f4v __attribute__((ext_vector_type(4)));
                    const f4v* p = reinterpret_cast<const f4v*>(col + 4 * lane);
                    const f4v v = NT ? __builtin_nontemporal_load(p) : *p;
#pragma unroll
                    for (int k = 0; k < 4; ++k) a[c][k] = v[k];
                } else {
                    typedef double d2v __attribute__((ext_vector_type(2)));
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const d2v* p = reinterpret_cast<const d2v*>(col + 128 * q + 2 * lane);
                        const d2v v = NT ? __builtin_nontemporal_load(p) : *p;
                        a[c][2 * q] = v[0];
                        a[c][2 * q + 1] = v[1];
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < DS_BATCH; ++c) {
                const int64_t j = j0 + b + c;
                double uj;
                if constexpr (edge) uj = read_lane(ub, c);
                else uj = u[j];
                double s = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double v = (double)a[c][k];
                    double vr = v, vc = v;
                    if constexpr (edge) {
                        const int64_t i = i0 + ds_row<TA, VEC>(lane, k);
                        vr = j < n && i < n && (!diag || i <= j) ? v : 0.0;
                        vc = j < n && i < n && (!diag || i < j) ? v : 0.0;
                    }
                    acc[k] = fma(vr, uj, acc[k]);
                    s = fma(vc, ui[k], s);
                }
                cs[b + c] = s;
            }
        }
    };
    const int bj1 = std::min(bi + (t + 1) * m, nb);
#pragma unroll 1
    for (int bj = bi + t * m; bj < bj1; ++bj) {
#pragma unroll 1
        for (int g = wave; g < DS_RB / DS_COLS; g += DS_WAVES) {
            const int64_t j0 = (int64_t)bj * DS_RB + g * DS_COLS;
            if (j0 >= n) break;
            using Y = std::true_type;
            using N = std::false_type;
            const bool diag = bj == bi;
            if (diag || j0 + DS_COLS > n) {
                if (VEC && whole) group(Y(), Y(), j0, diag);
                else group(N(), Y(), j0, diag);
            } else {
                if constexpr (VEC) group(Y(), N(), j0, diag);   // (rows before the last block)
                else group(N(), N(), j0, diag);
            }
            // column c's total on lanes 4 c .. 4 c + 3: halves, rows of 16, then by DPP
            double w8[8], w4[4], w2[2], w1[1];
#pragma unroll
            for (int e = 0; e < 8; ++e) w8[e] = swap32_sum(cs[e], cs[8 + e]);
#pragma unroll
            for (int e = 0; e < 4; ++e) w4[e] = swap16_sum(w8[e], w8[4 + e]);
            lane_halve<8, double, 2>(w4, w2, lane);
            lane_halve<4, double, 1>(w2, w1, lane);
            double v = w1[0] + lane_xor<2>(w1[0]);
            v = v + lane_xor<1>(v);
            const int c = lane >> 2;
            const int64_t slot = bj != bi ? bi : nb;
            if ((lane & 3) == 0 && j0 + c < n) part[slot * n + j0 + c] = v;
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) rs[wave][ds_row<TA, VEC>(lane, k)] = acc[k];
    __syncthreads();
    if (threadIdx.x < DS_RB && i0 + threadIdx.x < n) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < DS_WAVES; ++w) v += rs[w][threadIdx.x];
        part[(int64_t)(bi + t) * n + i0 + threadIdx.x] = v;
    }
}

bool dense_sym_ok(int64_t n, bool f32) { return n >= (f32 ? DENSE_SYM_MIN32 : DENSE_SYM_MIN64) && n <= (int64_t)1 << 19; }

size_t dense_sym_ws_doubles(int64_t n) { return ((size_t)((n + DS_RB - 1) / DS_RB) + 1) * (size_t)n; }

void launch_dense_matvec_sym(int dta, int64_t n, const void* A, int64_t lda, const double* u, double mu, double* y,
                             double* dot_part, double* ws, const int32_t* stop, hipStream_t st) {
    const DsPlan p = ds_plan(n);
    const size_t es = dta == DT_F32 ? 4 : 8;
    const bool vec = lda * es % 16 == 0 && (uintptr_t)A % 16 == 0;
    const bool nt = (size_t)n * n / 2 * es > (size_t)200 << 20;
    {
        ProfScope prof(dta == DT_F32 ? PROF_DENSE_MATVEC : PROF_DENSE_MATVEC64, st);
#define KDS(T, V, N) k_dense_sym<T, V, N><<<p.items, DS_THREADS, 0, st>>>(n, (const T*)A, lda, u, ws, p.nb, p.m, stop)
#define KDT(T)                                        \
    if (vec) { if (nt) KDS(T, true, true); else KDS(T, true, false); } \
    else { if (nt) KDS(T, false, true); else KDS(T, false, false); }
        if (dta == DT_F32) { KDT(float) } else { KDT(double) }
#undef KDT
#undef KDS
    }
    launch_slot_finish(n, p.nb, p.m, 1, 1, ws, 1.0, mu, u, y, dot_part, stop, st);
}

}  // namespace rr
