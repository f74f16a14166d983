// The kernel product of many columns in the working precision (the batched solve of
// more than 32 right-hand sides, Section 5.1): W = scale * K P + diag(mu_col) P with
// float32-class entries times P in float32, float32 sums over runs of 64 points added
// in float64.
//
// Both factors (the columns of P scaled by powers of two) are split exactly into three
// bf16 pieces (24 bits), and the six piece products with combined order <= 2 run on
// v_mfma_f32_32x32x16_bf16, the smallest first.  The three products left off reach 2^-24
// of the product, a rounding of float32, at worst (2^-27.5 in the mean square over random
// mantissas, above 2^-26 for 3 % of them), where a float32 MFMA leaves nothing off; the
// measured errors below include it.  Six bf16 MFMAs take 2.7 times less than the float32 ones
// they replace (v_mfma_f32_32x32x2_f32 at 142 against 2,270 TFLOP/s).  The entries'
// exponents come from the packed records of kmma.hpp.
//
// Block: eight waves, 128 rows by 64 NT columns, 32 points a step.  Wave (rt, wc)
// multiplies row tile rt with column tiles wc NT .. wc NT + NT - 1.  The kernel tile of a
// step (4 row tiles x 32 points) is formed by the waves of one half (wc), the next
// step's by the other, so that on each SIMD one wave forms while the other multiplies;
// both tiles are double-buffered in LDS, and a step costs one barrier.  The MFMAs bound
// it: 12 NT for the product and 3.5 for the entries per wave and step.  n = 20,000,
// d = 16, 256 columns: 1.26 ms (970 TFLOP/s of bf16 products) where the float32 MFMA
// kernel took 4.47; n = 5,003, 100 columns: 67 against 500 us.
//
// Error against 64 bits, by that of the float32 kernel (two CG steps on 33 to 256 columns,
// n = 1,000 to 12,000, 2 to 32 coordinates; mean over the columns): RBF 0.6 to 1.0 of it,
// Matern 0.01 to 0.7, and no more with points 30 from the origin.  A point with itself has
// distance 0, not what the pieces' rounding leaves of it, and the norms' step comes first,
// so that the sum of two close points is small when the small pieces are added: without
// these a Matern product was off by 1.2 to 1.6 times the float32 kernel's error.
#include "common.hpp"
#include "ctx.hpp"
#include "kentry.hpp"
#include "kernels.hpp"
#include "kmma.hpp"
#include "prof.hpp"

#include <algorithm>

namespace rr {

constexpr int KG_THREADS = 512, KG_WAVES = 8, KG_BM = 128, KG_BK = 32;
constexpr int64_t KG_COLS_MAX = 1024;                         // columns packed at a time
constexpr size_t KG_PART_MAX = (size_t)32 << 20;              // doubles of split partials

// Largest |P_ij| of each column over one of KG_CHUNKS row chunks.
constexpr int KG_CHUNKS = 8;
__global__ __launch_bounds__(256) void k_kgemm_colmax(int64_t n, int64_t m, const double* __restrict__ P, int64_t ldp,
                                                      double* __restrict__ part) {
    __shared__ double sh[4];
    const int64_t j = blockIdx.x, rpc = (n + KG_CHUNKS - 1) / KG_CHUNKS;
    const int64_t i1 = std::min<int64_t>(n, (blockIdx.y + 1) * rpc);
    double v = 0.0;
    for (int64_t i = blockIdx.y * rpc + threadIdx.x; i < i1; i += 256) v = fmax(v, fabs(P[i + j * ldp]));
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.y * m + j] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

// P packed for the product, each column times the power of two that brings its largest
// entry to [1, 2) (so that every piece of a normal-sized entry is a normal bf16 number,
// whatever the column's size; unscale gets the inverse): per block of 64 NT columns and step of 32 points, units
// ((piece 2 + g) 2 NT + column tile) of 64 x 16 bytes.  Lane 32 h + c of a unit holds
// column c of the tile at points 16 g + 4 h + (0..3) and 16 g + 8 + 4 h + (0..3) of the
// step, the order in which a lane of the exponents' accumulator holds its row's entries.
// Columns past m and points past n are zeros.
template <int NT>
__global__ __launch_bounds__(256) void k_kgemm_pack(int64_t n, int64_t steps, const double* __restrict__ P, int64_t ldp,
                                                    int64_t m, const double* __restrict__ colmax,
                                                    double* __restrict__ unscale, bf16x8_t* __restrict__ out) {
    // thread: one column, half h, group g of one step
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int c = (int)(e & 31), h = (int)(e >> 5 & 1), g = (int)(e >> 6 & 1);
    const int64_t s = (e >> 7) % steps;
    const int64_t ct = (e >> 7) / steps;   // column tile
    const int64_t col = ct * 32 + c, cb = ct / (2 * NT);
    if (cb * 64 * NT >= m) return;
    double mx = 0.0;
    if (col < m)
#pragma unroll
        for (int q = 0; q < KG_CHUNKS; ++q) mx = fmax(mx, colmax[q * m + col]);
    const int ex = mx > 0.0 && mx <= 1.7976931348623157e308 ? ilogb(mx) : 0;
    if (s == 0 && g == 0 && h == 0 && col < m) unscale[col] = ldexp(1.0, std::max(ex, -1000));
    bf16x8_t o[3];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int64_t j = s * KG_BK + 16 * g + (t >> 2) * 8 + 4 * h + (t & 3);
        __bf16 p[3];
        kmma_split3(j < n && col < m ? (float)ldexp(P[j + col * ldp], -std::max(ex, -1000)) : 0.0f, p);
#pragma unroll
        for (int q = 0; q < 3; ++q) o[q][t] = p[q];
    }
    bf16x8_t* dst = out + ((cb * steps + s) * (12 * NT) + ct % (2 * NT)) * 64 + 32 * h + c;
#pragma unroll
    for (int q = 0; q < 3; ++q) dst[(q * 2 + g) * (2 * NT) * 64] = o[q];
}

template <int KIND, int DM, int NT>
__global__ __launch_bounds__(KG_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_kgemm_bf16x6(
    int64_t n, int steps, int per, const bf16x8_t* __restrict__ rrec, const bf16x8_t* __restrict__ crec, float c,
    double scale, const double* __restrict__ mucol, const double* __restrict__ P, int64_t ldp, int64_t m,
    const double* __restrict__ unscale, const bf16x8_t* __restrict__ Pk, double* __restrict__ W, int64_t ldw, double* __restrict__ part) {
    constexpr int KB = KmmaShape<DM>::KB, UC = kmma_chunks<DM>(), UB = 12 * NT;
    __shared__ __attribute__((aligned(16))) bf16x8_t As[2][24 * 64];   // kernel tile pieces
    __shared__ __attribute__((aligned(16))) bf16x8_t Bs[2][UB * 64];   // P pieces
    const int lane = threadIdx.x & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int rt = wave & 3, wc = wave >> 2;
    const int s0 = blockIdx.z * per, cnt = std::min(per, steps - s0);
    const uint32_t bs_off = (uint32_t)(size_t)(__attribute__((address_space(3))) bf16x8_t*)&Bs[0][0];
    const bf16x8_t* pk = Pk + ((int64_t)blockIdx.y * steps + s0) * UB * 64;
    auto fetch = [&](int i) {
        const bf16x8_t* src = pk + (int64_t)i * UB * 64;
#pragma unroll
        for (int e0 = 0; e0 < UB; e0 += KG_WAVES) {
            const int e = e0 + wave;
            if (e < UB) lds_copy16(src + e * 64, lane, bs_off + ((i & 1) * UB + e) * 1024);
        }
    };
    bf16x8_t rr_[UC], cr[UC];
    const int64_t rtile = (int64_t)blockIdx.x * 4 + rt;
#pragma unroll
    for (int u = 0; u < UC; ++u) rr_[u] = rrec[(rtile * UC + u) * 64 + lane];
    auto load_points = [&](int i) {
#pragma unroll
        for (int u = 0; u < UC; ++u) cr[u] = crec[((int64_t)(s0 + i) * UC + u) * 64 + lane];
    };
    // the wave's 32 points x 32 rows of step i: element e of lane 32 h + r is point
    // 8 (e / 4) + 4 h + e % 4 of row r
    auto form = [&](int i) {
        f32x16_t d;
#pragma unroll
        for (int e = 0; e < 16; ++e) d[e] = 0.0f;
#pragma unroll
        for (int e = 0; e < KB; ++e) {
            const int s = (e + KB - 1) % KB;   // the norms' step first: close points cancel early
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cr[kmma_uc<DM, false>(s)], rr_[kmma_uc<DM, true>(s)], d, 0, 0, 0);
        }
        if (s0 + i == rtile)   // (uniform) a point with itself
#pragma unroll
            for (int e = 0; e < 16; ++e) d[e] = 8 * (e >> 2) + 4 * h + (e & 3) == l32 ? 0.0f : d[e];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            bf16x8_t o[3];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                __bf16 p[3];
                kmma_split3(kmma_entry<KIND>(d[8 * g + t], c), p);
#pragma unroll
                for (int q = 0; q < 3; ++q) o[q][t] = p[q];
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) As[i & 1][((q * 2 + g) * 4 + rt) * 64 + lane] = o[q];
        }
    };

    f32x16_t acc[NT];
    double acc64[NT][16];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            acc[t][e] = 0.0f;
            acc64[t][e] = 0.0;
        }
    auto flush = [&]() {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc64[t][e] += (double)acc[t][e];
                acc[t][e] = 0.0f;
            }
    };

    fetch(0);
    load_points(wc < cnt ? wc : 0);
    if (wc == 0) {
        form(0);
        if (2 < cnt) load_points(2);
    }
#pragma unroll 1
    for (int i = 0; i < cnt; ++i) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of step i has arrived
        __syncthreads();
        // the point records count as arrived here: a later wait for them would also wait
        // for the next step's copies
#pragma unroll
        for (int u = 0; u < UC; ++u) asm volatile("" : "+v"(cr[u]));
        if (i + 1 < cnt) {
            fetch(i + 1);
            if (wc == ((i + 1) & 1)) {
                form(i + 1);
                if (i + 3 < cnt) load_points(i + 3);
            }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            bf16x8_t kf[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) kf[q] = As[i & 1][((q * 2 + g) * 4 + rt) * 64 + lane];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                bf16x8_t pf[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) pf[q] = Bs[i & 1][((q * 2 + g) * (2 * NT) + wc * NT + t) * 64 + lane];
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[2], kf[0], acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[1], kf[1], acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[0], kf[2], acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[1], kf[0], acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[0], kf[1], acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf[0], kf[0], acc[t], 0, 0, 0);
            }
        }
        if (i & 1) flush();
    }
    flush();
    // element e of lane 32 h + r: column 8 (e / 4) + 4 h + e % 4 of the tile, row r
    const int64_t gr = rtile * 32 + l32;
    if (gr >= n) return;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t gc = (int64_t)blockIdx.y * (64 * NT) + (wc * NT + t) * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
            if (gc >= m) continue;
            const double v = acc64[t][e] * unscale[gc];
            if (part) part[((int64_t)blockIdx.z * m + gc) * n + gr] = v;
            else W[gr + gc * ldw] = fma(scale, v, mucol[gc] * P[gr + gc * ldp]);
        }
}

// W = scale (sum of the splits' partials, in order) + mu P.
__global__ void k_kgemm_reduce(int64_t n, int64_t m, int splits, const double* __restrict__ part, double scale,
                               const double* __restrict__ mucol, const double* __restrict__ P, int64_t ldp,
                               double* __restrict__ W, int64_t ldw) {
    const int64_t total = n * m;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e % n, j = e / n;
        double s = 0.0;
        for (int z = 0; z < splits; ++z) s += part[(int64_t)z * total + e];
        W[i + j * ldw] = fma(scale, s, mucol[j] * P[i + j * ldp]);
    }
}

// Column blocks of 128, of 64 where that leaves fewer empty columns; the points are
// split over blocks where whole rounds of the chip (a block per compute unit, two of the
// narrow ones) would otherwise be half empty.
struct KgPlan {
    int nt, cbs, splits, per;
    int64_t steps;
    // packed P, then the columns' scales and chunk maxima
    size_t packed_bytes(int64_t m) const {
        return (size_t)cbs * steps * (12 * nt) * 64 * sizeof(bf16x8_t) + (size_t)m * (1 + KG_CHUNKS) * sizeof(double);
    }
};
static KgPlan kg_plan(int64_t n, int64_t m, size_t part_cap) {
    KgPlan p;
    p.nt = (m + 63) / 64 % 2 == 1 && m <= 192 ? 1 : 2;
    p.cbs = (int)((m + 64 * p.nt - 1) / (64 * p.nt));
    p.steps = (n + KG_BK - 1) / KG_BK;
    const int64_t blocks = (n + KG_BM - 1) / KG_BM * p.cbs, slots = p.nt == 2 ? 256 : 512;
    double best = 0.0;
    p.splits = 1;
    for (int s = 1; s <= 8; ++s) {
        if (s > 1 && (p.steps < 16 * s || (size_t)s * n * m > part_cap)) break;
        const double cost = (double)((blocks * s + slots - 1) / slots) / s * (1.0 + 0.01 * (s - 1));
        if (s == 1 || cost < best) {
            best = cost;
            p.splits = s;
        }
    }
    p.per = (int)((p.steps + p.splits - 1) / p.splits);
    p.splits = (int)((p.steps + p.per - 1) / p.per);
    return p;
}

size_t kernel_matmat_ws_bytes(int64_t n, int64_t m) {
    size_t w = 0;
    // the column chunks of launch_kernel_matmat_bf16x6: whole ones and the rest
    for (const int64_t mc : {std::min(m, KG_COLS_MAX), m % KG_COLS_MAX}) {
        if (mc == 0) continue;
        const KgPlan p = kg_plan(n, mc, KG_PART_MAX);
        w = std::max(w, p.packed_bytes(mc) + (p.splits > 1 ? (size_t)p.splits * n * mc * 8 : 0));
    }
    return w;
}

void launch_kernel_matmat_bf16x6(const KernelOp& op, const double* mucol, const double* P, int64_t ldp, int64_t m,
                                 double* W, int64_t ldw, void* ws, size_t ws_bytes, hipStream_t st) {
    const float c = kernel_c32(op.kind, op.kconst);
    ProfScope prof(PROF_KERNEL_MATMAT, st);
    for (int64_t c0 = 0; c0 < m; c0 += KG_COLS_MAX) {
        const int64_t mc = std::min(KG_COLS_MAX, m - c0);
        // (a workspace made for more columns holds this chunk's packed P; its splits take
        // what is left)
        const size_t pkb = kg_plan(op.n, mc, 0).packed_bytes(mc);
        RR_REQUIRE(ws_bytes >= pkb, "workspace too small for the wide kernel product");
        const KgPlan p = kg_plan(op.n, mc, std::min(KG_PART_MAX, (ws_bytes - pkb) / sizeof(double)));
        bf16x8_t* pk = (bf16x8_t*)ws;
        double* part = p.splits > 1 ? (double*)((char*)ws + pkb) : nullptr;
        double* unscale = (double*)(pk + (size_t)p.cbs * p.steps * (12 * p.nt) * 64);
        double* colmax = unscale + mc;
        const double* Pc = P + c0 * ldp;
        double* Wc = W + c0 * ldw;
        k_kgemm_colmax<<<dim3((unsigned)mc, KG_CHUNKS), 256, 0, st>>>(op.n, mc, Pc, ldp, colmax);
        const unsigned pg = (unsigned)(((int64_t)p.cbs * 2 * p.nt * p.steps * 128 + 255) / 256);
        if (p.nt == 2) k_kgemm_pack<2><<<pg, 256, 0, st>>>(op.n, p.steps, Pc, ldp, mc, colmax, unscale, pk);
        else k_kgemm_pack<1><<<pg, 256, 0, st>>>(op.n, p.steps, Pc, ldp, mc, colmax, unscale, pk);
        const dim3 grid((unsigned)((op.n + KG_BM - 1) / KG_BM), (unsigned)p.cbs, (unsigned)p.splits);
#define KGL(K, DD, N)                                                                                            \
    k_kgemm_bf16x6<K, DD, N><<<grid, KG_THREADS, 0, st>>>(op.n, (int)p.steps, p.per, (const bf16x8_t*)op.rrec,    \
                                                          (const bf16x8_t*)op.crec, c, op.scale, mucol + c0, Pc, \
                                                          ldp, mc, unscale, pk, Wc, ldw, part)
#define KGN(K, DD)                        \
    if (p.nt == 2) { KGL(K, DD, 2); }     \
    else { KGL(K, DD, 1); }
#define KGD(K)                       \
    switch (op.dm) {                 \
        case 4: KGN(K, 4) break;     \
        case 8: KGN(K, 8) break;     \
        case 16: KGN(K, 16) break;   \
        default: KGN(K, 32) break;   \
    }
        if (op.kind == 1) { KGD(1) } else { KGD(2) }
#undef KGD
#undef KGN
#undef KGL
        if (part) {
            const int64_t g = std::min<int64_t>((op.n * mc + 255) / 256, 16384);
            k_kgemm_reduce<<<(unsigned)g, 256, 0, st>>>(op.n, mc, p.splits, part, op.scale, mucol + c0, Pc, ldp, Wc, ldw);
        }
    }
}

}  // namespace rr
