// Symmetric kernel matvec with the pair terms on bf16 MFMA:
// Y = scale * K U + mu U for NR = 1 or 2 columns (the PCG operator of kernel
// ridge regression, Section 7.2.2, and the two-column power iterations of the
// shift estimates).
//
// The exponent of each entry is the product of two augmented point records on
// bf16 MFMA, with float32-class accuracy (kmma.hpp).
//
// Rows are grouped in blocks of 256 (8 waves x 32 rows).  Unit (I, r, s)
// covers row block I against the column blocks J of run r (J = I + r m, ..., up to
// m of them, J < nb), restricted to the s-th of S column ranges.  Each pair (i, j)
// is evaluated once and its entry feeds y_i (row sums in registers) and y_j
// (column sums: the lane's 16 rows, then the two half-waves, then the eight waves
// in a fixed order): off the diagonal blocks by construction, and inside a
// diagonal block because wave w forms only the column tiles >= w and, in its own
// 32 x 32 tile, only the pairs with row <= column.  So the operator is exactly
// symmetric.
//
// Partial slots (float64, n per slot and column): the row sums of unit (I, r, s) go
// to slot (I + r) S + s of the rows of I; column sums from row block I < J to slot
// I S of the columns (exactly one range s covers a column); column sums inside the
// diagonal block to slot nb S.  So row i of block b owns slots p S for p < b, the
// slots from b S to (b + R_b) S (R_b = ceil((nb - b) / m) runs) and slot nb S, each
// written by exactly one unit, and the finish adds them in that order (bitwise
// reproducible, whatever the number of blocks that run the units).
//
// What bounds it: the vector ALU with the matrix cores beside it.  A 32 x 32 tile is 16
// exp2, 16 widenings and 32 float64 FMAs per lane and column (about 340 cycles of a
// SIMD) and seven MFMAs (230); the tile loop alone, from registers and LDS, runs at 537
// cycles a tile with four waves per SIMD and at 735 for two columns with two, and no
// order of its instructions (MFMAs ahead, interleaved, exponentials first, priorities)
// was faster on a warm chip.  The rest is kept off it: u of the rows stays in registers
// for a row block, records are packed once per operator and copied to LDS beside the
// products, the work is a few long blocks per compute unit, and the unit's place is
// computed, not searched.  n = 50,000, d = 16, one column: 0.40 ms (0.52 before, both
// under the tracer); two columns at n = 32,768: 0.26 ms (0.45); four: 0.51 (0.66).
// With 17 to 32 coordinates the variants of four waves a SIMD spill (24 registers for one
// RBF column, 12 Matern, 11 and 14 for two float columns), and the reloads wait for the
// copies in flight: little is gained there at large n (a whole product of one column,
// n = 50,000, d = 32: 0.81 ms, 0.82 with a block a unit; n = 20,000: 0.173, 0.218).
//
#include "common.hpp"
#include "group.hpp"
#include "kentry.hpp"
#include "kernels.hpp"
#include "kmma.hpp"
#include "prof.hpp"

#include <algorithm>
#include <type_traits>

namespace rr {

constexpr int KM_WAVES = 8;
constexpr int KM_THREADS = 64 * KM_WAVES;
constexpr int KM_RB = 32 * KM_WAVES;   // rows (and columns) per block
constexpr int KM_CT = KM_RB / 32;      // column tiles per block
constexpr int KM_MAX_SLOTS = 2048;     // partial slots per row (bounds the workspace)
constexpr int KM_MAX_RUN = 8;          // column blocks per run
constexpr int KM_STAGE = 4;            // column tiles per stage of an item

// Units (I, r, s): row block I, run r of up to m column blocks starting at
// I + r m, column range s of S (S > 1 only with m = 1, for small n).
struct KmmaPlan {
    int nb, m, S;
    int64_t units;
};

static KmmaPlan kmma_plan(int64_t n) {
    KmmaPlan p;
    p.nb = (int)((n + KM_RB - 1) / KM_RB);
    const int64_t tiles = (int64_t)p.nb * (p.nb + 1) / 2;
    p.m = (int)std::min<int64_t>(KM_MAX_RUN, std::max<int64_t>(1, tiles / 4096));
    int S = 1;
    while (p.m == 1 && S < KM_CT / 2 && tiles * S < 1024) S *= 2;   // a few items per compute unit
    p.S = S;
    int64_t runs = 0;
    for (int I = 0; I < p.nb; ++I) runs += (p.nb - I + p.m - 1) / p.m;
    p.units = runs * S;
    return p;
}

// Blocks of the launch.  A block runs consecutive units one after the other, so that the
// next unit's records arrive during this one and a row block is set up once for all the
// units the block has of it: with a block a unit, that setup and the launch took as long
// as the unit itself (n = 32,768, two columns: 13 of 21 us).  The blocks fill the chip
// once: two per compute unit for one column (or float sums), one for pairs of columns in
// float64 (wide).  One column of a Matern kernel keeps a block per unit: its longer
// entries hide the setup beside the other block, and uneven shares then cost more
// (n = 20,001, d = 3: 172 against 187 us, float64 357 against 393; RBF at n = 24,000,
// d = 8: 110 against 94).
static int kmma_blocks(const KmmaPlan& p, int kind, int nr, bool wide) {
    if (kind == 2 && !wide) return (int)p.units;
    const int64_t slots = wide ? 256 : 512, pairs = nr > 2 ? nr / 2 : 1;
    return (int)std::min(p.units, std::max<int64_t>(1, slots / pairs));
}
// First unit of block g of G: base = units / G each, and the rest spread evenly.
RR_DEV int kmma_first_unit(int g, int G, int units) {
    if (G == units) return g;
    const int base = units / G;
    return g * base + g * (units - base * G) / G;
}

// (row block, run) of run number t in the order of kmma_plan (row block 0 first).
// Counted from the end, the row blocks with k = nb - I column blocks left come in
// groups of m with ceil(k / m) runs each, so the group is a triangular root (a search
// over the row blocks is up to nb scalar steps).
RR_DEV void kmma_run_of(int t, int nb, int m, int& bi, int& run) {
    const int A = nb / m;
    const int r = m * (A * (A + 1) / 2) + (nb - A * m) * (A + 1) - 1 - t;   // run number from the end
    int a = __builtin_amdgcn_readfirstlane((int)((__builtin_sqrtf(8.0f * (float)(r / m) + 1.0f) - 1.0f) * 0.5f));
    while (m * (a * (a + 1) / 2) > r) --a;   // (the float root may be off by one)
    while (m * ((a + 1) * (a + 2) / 2) <= r) ++a;
    const int rest = r - m * (a * (a + 1) / 2), b = rest / (a + 1);
    bi = nb - (a * m + b + 1);
    run = a - (rest - b * (a + 1));
}

// The stages of a block's units in order: unit (bi, run, sr) covers the column tiles
// [tile, tile + ts) of stage q of nq; the first and last stages of a row block's stretch
// are where its rows are set up and where the unit's row sums leave.
struct KmmaWalk {
    int nb, m, S, ts, left;        // left: units to go, this one included
    int bi, run, sr, q, nq;
    RR_DEV void unit() {
        q = 0;
        nq = S > 1 ? (KM_CT / S) / ts : std::min(m, nb - bi - run * m) * (KM_CT / ts);
    }
    RR_DEV void start(int g, int G, int nb_, int m_, int S_, int units) {
        const int u = kmma_first_unit(g, G, units);
        nb = nb_;
        m = m_;
        S = S_;
        ts = std::min(KM_STAGE, KM_CT / S);
        left = kmma_first_unit(g + 1, G, units) - u;
        sr = u % S;
        kmma_run_of(u / S, nb, m, bi, run);
        unit();
    }
    RR_DEV int tile() const { return (bi + run * m) * KM_CT + sr * (KM_CT / S) + q * ts; }
    RR_DEV bool diag() const { return run == 0 && q < KM_CT / ts; }      // (S > 1: one stage a unit)
    RR_DEV int own(int wave) const { return wave - (tile() - bi * KM_CT); }   // the wave's own tile, in a diagonal block
    RR_DEV int rslot() const { return (bi + run) * S + sr; }
    RR_DEV int cslot() const { return diag() ? nb * S : bi * S; }
    RR_DEV bool unit_ends() const { return q + 1 == nq; }
    RR_DEV bool ends() const { return left == 1 && q + 1 == nq; }
    RR_DEV void next() {
        if (++q < nq) return;
        --left;
        if (++sr == S) {
            sr = 0;
            if (++run * m >= nb - bi) {
                run = 0;
                ++bi;
            }
        }
        unit();
    }
};

// Sum over the 32 lanes of a half-wave of v[0..15] (reduce-scatter butterfly in a
// fixed order): on return lanes 2e and 2e + 1 of the half hold the total of v[e].
template <typename T>
RR_DEV T kmma_rowsum16(const T (&v)[16], int l32) {
    T w8[8], w4[4], w2[2], w1[1];
#pragma unroll
    for (int e = 0; e < 8; ++e) w8[e] = swap16_sum(v[e], v[8 + e]);
    lane_halve<8, T, 4>(w8, w4, l32);
    lane_halve<4, T, 2>(w4, w2, l32);
    lane_halve<2, T, 1>(w2, w1, l32);
    // lanes 2e and 2e + 1 add the same two partials in opposite order: equal sums
    return w1[0] + lane_xor<1>(w1[0]);
}

// The packed row and column records (kmma.hpp) of every point, straight from the
// points: rows scaled by g, the squared norms added as k_sqnorms adds them.  Points
// past n up to the whole 256-row block are zeros (their entries multiply u = 0), and so
// is the chunk after the last tile.
template <int DM>
__global__ __launch_bounds__(256) void k_kmma_records(int64_t n, int64_t npad, int d, const float* __restrict__ pts,
                                                      float g, bf16x8_t* __restrict__ rrec,
                                                      bf16x8_t* __restrict__ crec) {
    constexpr int UC = kmma_chunks<DM>(), NC = kmma_ncoord<DM>();
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t tile = e >> 6;
    const int lane = (int)(e & 63), h = lane >> 5;
    const int64_t i = tile * 32 + (lane & 31);
    bf16x8_t z;
#pragma unroll
    for (int t = 0; t < 8; ++t) z[t] = (__bf16)0.0f;
    if (e == 0) {   // a zero after the last tile
        rrec[npad * 2 * UC] = z;
        crec[npad * 2 * UC] = z;
    }
    if (i >= npad) return;
    bf16x8_t* ro = rrec + tile * UC * 64 + lane;
    bf16x8_t* co = crec + tile * UC * 64 + lane;
    if (i >= n) {
        for (int c = 0; c < UC; ++c) { ro[c * 64] = z; co[c * 64] = z; }
        return;
    }
    float xr[NC];
    float sq = 0.0f;
#pragma unroll
    for (int k = 0; k < DM; ++k) {
        const float v = k < d ? pts[(int64_t)k * n + i] : 0.0f;
        sq = fmaf(v, v, sq);
        if constexpr (DM >= 16) {
            // coordinate 16 m + 8 h + t is the half's element 8 m + t
            if ((k >> 3 & 1) == h) xr[8 * (k >> 4) + (k & 7)] = v;
        } else {
            xr[k] = v;
        }
    }
    // a chunk is written by the first step that uses it
    kmma_record_x<DM, true>(xr, sq, g, h, [&](int s, const bf16x8_t& v) { ro[kmma_uc<DM, true>(s) * 64] = v; });
    kmma_record_x<DM, false>(xr, sq, g, h, [&](int s, const bf16x8_t& v) { co[kmma_uc<DM, false>(s) * 64] = v; });
}

size_t kernel_mma_record_bytes(int64_t n, int dm) {
    const int64_t npad = (n + KM_RB - 1) / KM_RB * KM_RB;
    const int uc = dm <= 4 ? kmma_chunks<4>() : dm <= 8 ? kmma_chunks<8>() : dm <= 16 ? kmma_chunks<16>() : kmma_chunks<32>();
    return ((size_t)npad * 2 * uc + 1) * sizeof(bf16x8_t);
}

void launch_kmma_records(const KernelOp& op, void* rrec, void* crec, hipStream_t st) {
    const int64_t npad = (op.n + KM_RB - 1) / KM_RB * KM_RB;
    const float g = op.kind == 1 ? kernel_c32(op.kind, op.kconst) : 1.0f;
    const unsigned grid = (unsigned)(2 * npad / 256);
#define KREC(DD) \
    k_kmma_records<DD><<<grid, 256, 0, st>>>(op.n, npad, op.d, op.pts, g, (bf16x8_t*)rrec, (bf16x8_t*)crec)
    switch (op.dm) {
        case 4: KREC(4); break;
        case 8: KREC(8); break;
        case 16: KREC(16); break;
        default: KREC(32); break;
    }
#undef KREC
}

// v[32 t .. 32 t + 32) (t wave-uniform, zeros from n on; ntf = n / 32) to the LDS doubles
// at off; zero: a zero double.
RR_DEV void lds_copy_32(const double* v, int t, int64_t n, int ntf, const double* zero, int lane, uint32_t off) {
    if (t < ntf) {
        lds_copy4(v + (int64_t)t * 32, 4 * lane, off);
    } else {
        const int64_t j = (int64_t)t * 32 + (lane >> 1);
        lds_copy4_lanes(reinterpret_cast<const uint32_t*>(j < n ? v + j : zero) + (lane & 1), off);
    }
}

// Before a copy over LDS that this wave alone reads and has read in the same stage: the
// compiler does not know of the copy, so nothing else keeps it behind those reads.
RR_DEV void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The lane number as a value that the compiler cannot see through: addresses formed from
// it are formed where they are used instead of being held (and spilled) across a stage.
RR_DEV int fresh_lane() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t & 63;
}

// One block: number item of items, for NR (1 or 2) columns q0, q0 + 1 of nrt.
// T: the type of the products and partial sums (double; float for the estimate grade
// of the power iterations, whose per-item partials are still stored as double).
// Shared by k_ksym_mma (item = block index) and the grouped serving kernel (items of
// many operators in one launch; a block may run items one after the other).  The sums of
// a unit do not depend on the blocks' sizes.
//
// While a stage is computed, the next stage's records and u travel to the other half of
// the LDS buffers, and the previous stage's column partials are added up: a stage costs
// one barrier.
template <int KIND, int DM, int NR, typename T>
RR_DEV void ksym_mma_item(int item, int64_t n, const bf16x8_t* __restrict__ rrec, const bf16x8_t* __restrict__ crec,
                          float c, const double* __restrict__ u, double* __restrict__ part, int nb, int m, int S,
                          int items, int units, int nrt, int q0) {
    constexpr int KB = KmmaShape<DM>::KB, UC = kmma_chunks<DM>(), ST = KM_STAGE;
    __shared__ __attribute__((aligned(16))) bf16x8_t bsb[2][ST * UC * 64];   // column records of a stage
    __shared__ __attribute__((aligned(16))) double usb[2][NR][32 * ST];      // u of its columns
    __shared__ __attribute__((aligned(16))) double urb[NR][KM_RB];           // u of the rows
    __shared__ T cwb[2][KM_WAVES][NR][32 * ST];                               // column partials per wave

    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    KmmaWalk wk;
    wk.start(item, items, nb, m, S, units);
    const int ts = wk.ts, tsh = 31 - __builtin_clz(ts);
    u += (int64_t)q0 * n;
    part += (int64_t)q0 * n;

    const uint32_t bs_off = (uint32_t)(size_t)(__attribute__((address_space(3))) bf16x8_t*)&bsb[0][0];
    const uint32_t us_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&usb[0][0][0];
    const int ntf = (int)(n / 32);   // whole tiles
    const double* zero = reinterpret_cast<const double*>(crec + (int64_t)nb * KM_CT * UC * 64);   // (past the records)
    const uint32_t ur_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&urb[0][0];
    // records and u of the ts tiles from tile on, into the buffers' half kp; row >= 0:
    // also u of that row block, each wave its own 32 rows (urb is read when a row block
    // begins; a block that starts with a row block's last stage reads it and fetches the
    // next one's in the same stage)
    auto fetch = [&](int tile, int kp, int row) {
        const int lane = fresh_lane();
        if (row >= 0) {
            lds_reads_done();
#pragma unroll
            for (int p = 0; p < NR; ++p)
                lds_copy_32(u + p * n, row * KM_CT + wave, n, ntf, zero, lane,
                            ur_off + (p * KM_RB + 32 * wave) * 8);
        }
        const bf16x8_t* src = crec + (int64_t)tile * UC * 64;
#pragma unroll
        for (int e0 = 0; e0 < ST * UC; e0 += KM_WAVES) {
            const int e = e0 + wave;
            if (e < ts * UC) lds_copy16(src + e * 64, lane, bs_off + (kp * ST * UC + e) * 1024);
        }
        if (wave < NR * ts) {   // 32 columns of u per wave
            const int uq = wave >> tsh, ut = wave & (ts - 1);
            lds_copy_32(u + uq * n, tile + ut, n, ntf, zero, lane, us_off + ((kp * NR + uq) * ST + ut) * 256);
        }
    };
    // column sums of a finished stage of columns j0 on from its partials, to dst: the
    // eight waves in a fixed order
    auto flush = [&](int j0, double* dst, int kp) {
        const int p = wave / (KM_STAGE / 2);
        if (p >= NR) return;
        const int jl = (wave & (KM_STAGE / 2 - 1)) * 64 + fresh_lane(), j = j0 + jl;
        if (jl < 32 * ts && j < n) {
            T v = T(0);
#pragma unroll
            for (int w = 0; w < KM_WAVES; ++w) v += cwb[kp][w][p][jl];
            dst[p * n + j] = (double)v;
        }
    };

    bf16x8_t areg[UC];
    T ui[16][NR], acc[16][NR];
    fetch(wk.tile(), 0, wk.bi);
    const int64_t slotd = (int64_t)nrt * n;   // doubles per slot
    int pj0 = 0;           // the previous stage's columns and slot
    double* pdst = part;
    int kp = 0;
#pragma unroll 1
    for (bool begin = true;; begin = false) {
        const int tile = wk.tile(), bi = wk.bi;
        const bool first = begin || (wk.run == 0 && wk.sr == 0 && wk.q == 0);   // of the block or the row block
        const int lane = fresh_lane(), h = lane >> 5, l32 = lane & 31;
        if (first) {   // the wave's rows: A operands
#pragma unroll
            for (int s = 0; s < UC; ++s) areg[s] = rrec[(((int64_t)bi * KM_CT + wave) * UC + s) * 64 + lane];
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of the stage has arrived
        __syncthreads();
        // the records count as arrived here: a later wait for them would also wait for the
        // next stage's copies
#pragma unroll
        for (int s = 0; s < UC; ++s) asm volatile("" : "+v"(areg[s]));
        if (first) {   // u at the 16 rows of this lane's outputs (0 past n)
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int p = 0; p < NR; ++p) {
                    ui[e][p] = T(urb[p][32 * wave + 8 * (e >> 2) + 4 * h + (e & 3)]);
                    acc[e][p] = T(0);
                }
        }
        const bool ends = wk.ends(), unit_ends = wk.unit_ends(), dg = wk.diag();
        const int own = wk.own(wave), rslot = wk.rslot(), cslot = wk.cslot();
        wk.next();   // (from here on the walk is at the next stage)
        if (!ends) fetch(wk.tile(), kp ^ 1, wk.bi != bi ? wk.bi : -1);
        if (!begin) flush(pj0, pdst, kp ^ 1);
        auto dots = [&](int ct) {
            f32x16_t d;
#pragma unroll
            for (int e = 0; e < 16; ++e) d[e] = 0.0f;
#pragma unroll
            for (int s = 0; s < KB; ++s)
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(areg[kmma_uc<DM, true>(s)],
                                                            bsb[kp][(ct * UC + kmma_uc<DM, false>(s)) * 64 + lane], d, 0, 0, 0);
            return d;
        };
        // DG: the wave's own tile of a diagonal block; only pairs with row <= column
        // count (row sums), and row < column (column sums)
        auto entries = [&](int ct, const f32x16_t& dot, auto dg) {
            constexpr bool DG = decltype(dg)::value;
            const int jl = 32 * ct + l32;   // the lane's column within the stage
            T uj[NR], cs[2][NR];
#pragma unroll
            for (int p = 0; p < NR; ++p) {
                uj[p] = T(usb[kp][p][jl]);
                cs[0][p] = T(0);
                cs[1][p] = T(0);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const T kv = T(kmma_entry<KIND>(dot[e], c));
                T kr = kv, kc = kv;
                if constexpr (DG) {
                    const int rr = 8 * (e >> 2) + 4 * h + (e & 3);   // the entry's row within the tile
                    kr = rr <= l32 ? kv : T(0);
                    kc = rr < l32 ? kv : T(0);
                }
#pragma unroll
                for (int p = 0; p < NR; ++p) {
                    acc[e][p] = fma(kr, uj[p], acc[e][p]);
                    cs[e & 1][p] = fma(kc, ui[e][p], cs[e & 1][p]);
                }
            }
            // the two half-waves hold the same column for different rows; both store
            // the same sum (addition is commutative)
#pragma unroll
            for (int p = 0; p < NR; ++p) cwb[kp][wave][p][jl] = xor_pair_sum<32>(cs[0][p] + cs[1][p]);
        };
        // in the diagonal block wave w forms only the column tiles >= w, so each pair
        // is evaluated once and the operator stays exactly symmetric
        int ct = 0;
        if (dg) {
            for (; ct < ts && ct < own; ++ct)
#pragma unroll
                for (int p = 0; p < NR; ++p) cwb[kp][wave][p][32 * ct + l32] = T(0);
            if (ct < ts && ct == own) {
                entries(ct, dots(ct), std::true_type{});
                ++ct;
            }
        }
        if constexpr (NR == 2 && sizeof(T) == 8) {
            // two waves per SIMD: the next tile's exponent MFMAs are issued beside this
            // tile's entries (the second accumulator fits this variant's registers)
            if (ct < ts) {
                f32x16_t dcur = dots(ct);
#pragma unroll 1
                for (; ct + 1 < ts; ++ct) {
                    const f32x16_t dnext = dots(ct + 1);
                    entries(ct, dcur, std::false_type{});
                    dcur = dnext;
                }
                entries(ct, dcur, std::false_type{});
            }
        } else {
#pragma unroll 1
            for (; ct < ts; ++ct) entries(ct, dots(ct), std::false_type{});
        }
        pj0 = tile * 32;
        pdst = part + cslot * slotd;
        if (unit_ends) {
            // row sums of the unit
            const int lane = fresh_lane(), h = lane >> 5, l32 = lane & 31;
            const int64_t r0 = (int64_t)bi * KM_RB + 32 * wave;
#pragma unroll
            for (int p = 0; p < NR; ++p) {
                T v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) { v[e] = acc[e][p]; acc[e][p] = T(0); }
                const T tot = kmma_rowsum16(v, l32);
                const int e = l32 >> 1;
                const int64_t i = r0 + 8 * (e >> 2) + 4 * h + (e & 3);
                if ((l32 & 1) == 0 && i < n) part[rslot * slotd + p * n + i] = (double)tot;
            }
        }
        if (ends) break;
        kp ^= 1;
    }
    __syncthreads();
    flush(pj0, pdst, kp);
}

template <int KIND, int DM, int NR, typename T>
__global__ __launch_bounds__(KM_THREADS) __attribute__((amdgpu_waves_per_eu(NR * sizeof(T) <= 8 ? 4 : 2))) void k_ksym_mma(
    int64_t n, const bf16x8_t* __restrict__ rrec, const bf16x8_t* __restrict__ crec, float c,
    const double* __restrict__ u, double* __restrict__ part, int nb, int m, int S, int units, int nrt,
    const int32_t* __restrict__ stop) {
    if (stop && *stop) return;
    ksym_mma_item<KIND, DM, NR, T>(blockIdx.x, n, rrec, crec, c, u, part, nb, m, S, gridDim.x, units, nrt,
                                   NR * blockIdx.y);
}

// y_q = scale * (sum of row i's slots) + mu u_q, with block partials of u_q^T y_q.
// Block: the 256 rows of one row block b (so the slot list is uniform over the
// block) and 1024 threads: four groups of 256 split the list
//   column slots p S (p < b), the run slots b S .. z1 - 1, the diagonal slot nb S
// into four contiguous quarters, each summed with four running sums, and group 0
// adds the quarters in a fixed order (bitwise reproducible, the same for one or
// two columns).
// Block bx of the nblk = ceil(n / 256) blocks of one finish, columns [q0, q1) (one a
// block in the launch of its own; shared with the grouped serving kernel).
constexpr int KF_GROUPS = 4;
RR_DEV void ksym_mma_finish_block(unsigned bx, unsigned nblk, int q0, int q1, int64_t n, int rb, int nb, int m, int S,
                                  int nr,
                                  const double* __restrict__ part, double scale, double mu,
                                  const double* __restrict__ u, double* __restrict__ y,
                                  double* __restrict__ dot_part) {
    __shared__ double quart[KF_GROUPS - 1][256];
    __shared__ double sc[4];
    const int t = threadIdx.x & 255, g = threadIdx.x >> 8;
    const int64_t i = (int64_t)bx * 256 + t;
    const int b = (int)(((int64_t)bx * 256) / rb);
    const int64_t z1 = (int64_t)(b + (nb - b + m - 1) / m) * S;
    const int64_t nrun = z1 - (int64_t)b * S;
    const int64_t T = b + nrun + 1;
    const int64_t k0 = T * g / KF_GROUPS, k1 = T * (g + 1) / KF_GROUPS;
    auto slot = [&](int64_t k) -> int64_t {
        return k < b ? k * S : (k < b + nrun ? (int64_t)b * S + (k - b) : (int64_t)nb * S);
    };
    for (int q = q0; q < q1; ++q) {
        double s = 0.0;
        if (i < n) {
            double s4[4] = {0.0, 0.0, 0.0, 0.0};
            int64_t k = k0;
            for (; k + 16 <= k1; k += 16) {   // sixteen loads in flight, added in the same order
                double v[16];
#pragma unroll
                for (int w = 0; w < 16; ++w) v[w] = part[(slot(k + w) * nr + q) * n + i];
#pragma unroll
                for (int w = 0; w < 16; ++w) s4[w & 3] += v[w];
            }
            for (; k + 4 <= k1; k += 4)
#pragma unroll
                for (int w = 0; w < 4; ++w) s4[w] += part[(slot(k + w) * nr + q) * n + i];
            for (; k < k1; ++k) s4[0] += part[(slot(k) * nr + q) * n + i];
            s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        }
        // quart and sc are reused for the next column only after the barrier below
        if (g > 0) quart[g - 1][t] = s;
        __syncthreads();
        double dot = 0.0;
        if (g == 0 && i < n) {
            const double tot = (s + quart[0][t]) + (quart[1][t] + quart[2][t]);
            const double ui = u[(int64_t)q * n + i];
            const double yi = fma(scale, tot, mu * ui);
            y[(int64_t)q * n + i] = yi;
            dot = ui * yi;
        }
        if (g == 0) {
            dot = wave_sum(dot);
            if ((t & 63) == 0) sc[t >> 6] = dot;
        }
        __syncthreads();
        if (threadIdx.x == 0)
            dot_part[(int64_t)q * nblk + bx] = (sc[0] + sc[1]) + (sc[2] + sc[3]);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256 * KF_GROUPS) void k_ksym_mma_finish(int64_t n, int rb, int nb, int m, int S,
                                                                     int nr,
                                                                     const double* __restrict__ part,
                                                                     double scale, double mu,
                                                                     const double* __restrict__ u,
                                                                     double* __restrict__ y,
                                                                     double* __restrict__ dot_part,
                                                                     const int32_t* __restrict__ stop) {
    if (stop && *stop) return;
    ksym_mma_finish_block(blockIdx.x, gridDim.x, blockIdx.y, blockIdx.y + 1, n, rb, nb, m, S, nr, part, scale, mu, u, y, dot_part);
}

// ------------------------------------------------------------------ float64
// The same work items, partial slots and finish as k_ksym_mma, with float64 entries
// (the restart residuals of the float64 refinement and the float64 working
// precision).  The Gram part of the exponent
//   t_ij = h_i + h_j + sum_k (g x_ik) x_jk = -g r_ij^2 / 2,   h_i = -g |x_i|^2 / 2,
// runs on v_mfma_f64_16x16x4_f64 with h_i as the accumulator's initial value; h_j,
// the table exp2 (kentry64) and the float64 row and column sums run on the vector
// ALU.  A wave's 32 x 32 tile is four 16 x 16 MFMA tiles (a, b): lane l supplies
// A[row 16 a + l%16][k 4 s + l/16] and B[k 4 s + l/16][column 16 b + l%16] of step s
// and holds element e of the product at row 16 a + 4 e + l/16, column 16 b + l%16, so
// a lane owns 8 rows and 2 columns of the tile.  Column sums: the lane's 8 rows, then
// the four lanes of a column (l/16 = 0..3), then the eight waves in a fixed order;
// row sums: the lane's columns over the item, then the 16 lanes of a row.  Each pair
// is evaluated once, also inside the diagonal blocks (wave w forms the column tiles
// >= w, and in its own tile only row <= column for the row sums and row < column for
// the column sums), so the operator is exactly symmetric.
typedef double f64x4_t __attribute__((ext_vector_type(4)));

template <int KIND, int DM, int NR>
__global__ __launch_bounds__(KM_THREADS) __attribute__((amdgpu_waves_per_eu(NR == 1 ? 4 : 2))) void k_ksym_mma64(
    int64_t n, const double* __restrict__ xp, const double* __restrict__ hd, double g, double kconst,
    const double* __restrict__ u, double* __restrict__ part, int nb, int m, int S, int units,
    const int32_t* __restrict__ stop) {
    constexpr int KS = DM / 4, ST = KM_STAGE;   // MFMA steps of 4 coordinates
    constexpr int TB = 2 * KS * 64;              // packed doubles of a 32-point tile
    __shared__ __attribute__((aligned(16))) double bsb[2][ST * TB];       // column records of a stage
    __shared__ __attribute__((aligned(16))) double hsb[2][32 * ST];       // h_j of its columns
    __shared__ __attribute__((aligned(16))) double usb[2][NR][32 * ST];   // u_j
    __shared__ __attribute__((aligned(16))) double hr[KM_RB];             // h_i of the rows
    __shared__ __attribute__((aligned(16))) double urb[NR][KM_RB];        // u_i
    __shared__ double cwb[2][KM_WAVES][NR][32 * ST];                       // column partials per wave
    __shared__ double tab[EXP2_TAB];
    if (stop && *stop) return;
    exp2_table_fill(tab);

    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    KmmaWalk wk;
    wk.start(blockIdx.x, gridDim.x, nb, m, S, units);
    const int ts = wk.ts, tsh = 31 - __builtin_clz(ts);

    const uint32_t bs_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&bsb[0][0];
    const uint32_t hs_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&hsb[0][0];
    const uint32_t us_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&usb[0][0][0];
    const uint32_t ur_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&urb[0][0];
    const uint32_t hr_off = (uint32_t)(size_t)(__attribute__((address_space(3))) double*)&hr[0];
    const int ntf = (int)(n / 32);   // whole tiles
    const double* zero = xp + (int64_t)nb * KM_CT * TB;   // (past the records)
    auto fetch = [&](int tile, int kp, int row) {
        const int lane = fresh_lane();
        if (row >= 0) {
            const int t = row * KM_CT + wave;
#pragma unroll
            for (int p = 0; p < NR; ++p) lds_copy_32(u + p * n, t, n, ntf, zero, lane, ur_off + (p * KM_RB + 32 * wave) * 8);
            lds_copy_32(hd, t, n, ntf, zero, lane, hr_off + 32 * wave * 8);
        }
        const double* src = xp + (int64_t)tile * TB;
#pragma unroll
        for (int e0 = 0; e0 < ST * TB / 128; e0 += KM_WAVES) {
            const int e = e0 + wave;
            if (e < ts * TB / 128) lds_copy16(src + e * 128, lane, bs_off + (kp * ST * TB / 128 + e) * 1024);
        }
        // u and h of 32 columns per wave and turn
        for (int e = wave; e < (NR + 1) * ts; e += KM_WAVES) {
            const int uq = e >> tsh, ut = e & (ts - 1);
            if (uq == NR) lds_copy_32(hd, tile + ut, n, ntf, zero, lane, hs_off + (kp * ST + ut) * 256);
            else lds_copy_32(u + uq * n, tile + ut, n, ntf, zero, lane, us_off + ((kp * NR + uq) * ST + ut) * 256);
        }
    };
    // column sums of a finished stage of columns j0 on from its partials, to dst: the
    // eight waves in a fixed order
    auto flush = [&](int j0, double* dst, int kp) {
        const int p = wave / (KM_STAGE / 2);
        if (p >= NR) return;
        const int jl = (wave & (KM_STAGE / 2 - 1)) * 64 + fresh_lane(), j = j0 + jl;
        if (jl < 32 * ts && j < n) {
            double v = double(0);
#pragma unroll
            for (int w = 0; w < KM_WAVES; ++w) v += cwb[kp][w][p][jl];
            dst[p * n + j] = (double)v;
        }
    };

    double areg[2][KS];
    double ui[8][NR], acc[8][NR];
    fetch(wk.tile(), 0, wk.bi);
    const int64_t slotd = (int64_t)NR * n;   // doubles per slot
    int pj0 = 0;           // the previous stage's columns and slot
    double* pdst = part;
    int kp = 0;
#pragma unroll 1
    for (bool begin = true;; begin = false) {
        const int tile = wk.tile(), bi = wk.bi;
        const int64_t r0 = (int64_t)bi * KM_RB + 32 * wave;   // the wave's 32 rows
        const bool first = begin || (wk.run == 0 && wk.sr == 0 && wk.q == 0);   // of the block or the row block
        const int lane = fresh_lane(), lr = lane >> 4, lc = lane & 15;
        if (first) {   // A operands: g x_i of rows 16 a + lc
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    areg[a][s] = g * xp[((int64_t)bi * KM_CT + wave) * TB + (a * KS + s) * 64 + lane];
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's part of the stage has arrived
        __syncthreads();
        // the records count as arrived here: a later wait for them would also wait for the
        // next stage's copies
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(areg[a][s]));
        if (first) {   // u_i at the lane's output rows (0 past n); h_i stays in LDS
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int p = 0; p < NR; ++p) {
                    ui[e][p] = urb[p][32 * wave + 16 * (e >> 2) + 4 * (e & 3) + lr];
                    acc[e][p] = 0.0;
                }
        }
        const bool ends = wk.ends(), unit_ends = wk.unit_ends(), dg = wk.diag();
        const int own = wk.own(wave), rslot = wk.rslot(), cslot = wk.cslot();
        wk.next();   // (from here on the walk is at the next stage)
        if (!ends) fetch(wk.tile(), kp ^ 1, -1);   // (the next row block's u and h: below)
        if (!begin) flush(pj0, pdst, kp ^ 1);
        auto tile_of = [&](int ct, auto dgc) {
            constexpr bool DG = decltype(dgc)::value;
            f64x4_t d[2][2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                f64x4_t hv;
#pragma unroll
                for (int e = 0; e < 4; ++e) hv[e] = hr[32 * wave + 16 * a + 4 * e + lr];
                d[a][0] = hv;
                d[a][1] = hv;
            }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const double b0 = bsb[kp][ct * TB + s * 64 + lane];
                const double b1 = bsb[kp][ct * TB + (KS + s) * 64 + lane];
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    d[a][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(areg[a][s], b0, d[a][0], 0, 0, 0);
                    d[a][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(areg[a][s], b1, d[a][1], 0, 0, 0);
                }
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int jl = 32 * ct + 16 * b + lc;
                const double hj = hsb[kp][jl];
                double uj[NR], cs[NR];
#pragma unroll
                for (int p = 0; p < NR; ++p) { uj[p] = usb[kp][p][jl]; cs[p] = 0.0; }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double kv = kentry64<KIND>(d[a][b][e] + hj, kconst, tab);
                        double kr = kv, kc = kv;
                        if constexpr (DG) {
                            const int rrow = 16 * a + 4 * e + lr, rcol = 16 * b + lc;
                            kr = rrow <= rcol ? kv : 0.0;
                            kc = rrow < rcol ? kv : 0.0;
                        }
#pragma unroll
                        for (int p = 0; p < NR; ++p) {
                            acc[4 * a + e][p] = fma(kr, uj[p], acc[4 * a + e][p]);
                            cs[p] = fma(kc, ui[4 * a + e][p], cs[p]);
                        }
                    }
                // the four lanes of the column add in a fixed pattern (equal results)
#pragma unroll
                for (int p = 0; p < NR; ++p) {
                    double v = cs[p];
                    v = xor_pair_sum<16>(v);
                    v = xor_pair_sum<32>(v);
                    if (lr == 0) cwb[kp][wave][p][jl] = v;
                }
            }
        };
        int ct = 0;
        if (dg) {
            for (; ct < ts && ct < own; ++ct)
                if (lr == 0)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int p = 0; p < NR; ++p) cwb[kp][wave][p][32 * ct + 16 * b + lc] = 0.0;
            if (ct < ts && ct == own) {
                tile_of(ct, std::true_type{});
                ++ct;
            }
        }
#pragma unroll 1
        for (; ct < ts; ++ct) tile_of(ct, std::false_type{});
        pj0 = tile * 32;
        pdst = part + cslot * slotd;
        if (unit_ends) {
            // row sums of the unit: the 16 lanes of a row add in a fixed butterfly
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int p = 0; p < NR; ++p) {
                    double v = acc[r][p];
                    acc[r][p] = 0.0;
                    v = v + lane_xor<1>(v);
                    v = v + lane_xor<2>(v);
                    v = v + lane_xor<4>(v);
                    v = v + lane_xor<8>(v);
                    const int64_t i = r0 + 16 * (r >> 2) + 4 * (r & 3) + lr;
                    if (lc == 0 && i < n) part[rslot * slotd + p * n + i] = v;
                }
        }
        if (ends) break;
        if (wk.bi != bi) {   // this wave has read the last of its rows' h_i, and u if it formed no tile
            lds_reads_done();
            const int t = wk.bi * KM_CT + wave, lane = fresh_lane();
#pragma unroll
            for (int p = 0; p < NR; ++p) lds_copy_32(u + p * n, t, n, ntf, zero, lane, ur_off + (p * KM_RB + 32 * wave) * 8);
            lds_copy_32(hd, t, n, ntf, zero, lane, hr_off + 32 * wave * 8);
        }
        kp ^= 1;
    }
    __syncthreads();
    flush(pj0, pdst, kp);
}

// Packed float64 records of launch_kernel_matvec_mma64: 32-point tiles of two 16-point
// halves, each KS = dm / 4 units of 64 doubles (lane l: coordinate 4 s + l / 16 of point
// l % 16, the MFMA operand of step s); zeros past d and past n, and one zero after the
// last tile.
__global__ __launch_bounds__(256) void k_kmma_records64(int64_t n, int64_t npad, int d, int dm, double g,
                                                        const float* __restrict__ pts, double* __restrict__ xp,
                                                        double* __restrict__ hd) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e > npad * dm) return;
    if (e < n) {   // h_e = -g |x_e|^2 / 2, added as k_point_records64 adds it
        double s = 0.0;
        for (int k = 0; k < d; ++k) {
            const double v = (double)pts[(int64_t)k * n + e];
            s = fma(v, v, s);
        }
        hd[e] = -0.5 * g * s;
    }
    const int ks = dm / 4, lane = (int)(e & 63);
    const int64_t unit = e >> 6;
    const int64_t i = unit / ks * 16 + (lane & 15);
    const int k = 4 * (int)(unit % ks) + (lane >> 4);
    xp[e] = i < n && k < d ? (double)pts[(int64_t)k * n + i] : 0.0;
}

size_t kernel_mma_record64_bytes(int64_t n, int dm) {
    const int64_t npad = (n + KM_RB - 1) / KM_RB * KM_RB;
    return ((size_t)npad * dm + 2) * sizeof(double);
}

void launch_kmma_records64(const KernelOp& op, double* xp, double* hd, hipStream_t st) {
    const int64_t npad = (op.n + KM_RB - 1) / KM_RB * KM_RB;
    k_kmma_records64<<<(unsigned)(npad * op.dm / 256 + 1), 256, 0, st>>>(op.n, npad, op.d, op.dm,
                                                                            kernel_g64(op.kind, op.kconst), op.pts, xp,
                                                                            hd);
}

void launch_slot_finish(int64_t n, int nb, int m, int S, int nr, const double* part, double scale, double mu,
                        const double* u, double* y, double* dot_part, const int32_t* stop, hipStream_t st) {
    k_ksym_mma_finish<<<dim3((unsigned)((n + 255) / 256), (unsigned)nr), 256 * KF_GROUPS, 0, st>>>(
        n, KM_RB, nb, m, S, nr, part, scale, mu, u, y, dot_part, stop);
}

void launch_kernel_matvec_mma64(const KernelOp& op, const double* u, int nr, double mu, double* y,
                                double* dot_part, double* ws, const int32_t* stop, hipStream_t st) {
    const KmmaPlan p = kmma_plan(op.n);
    const double g = kernel_g64(op.kind, op.kconst);
    const unsigned grid = (unsigned)kmma_blocks(p, op.kind, nr, nr > 1);
    {
        ProfScope prof(nr == 1 ? PROF_KERNEL_MATVEC64 : -1, st);
#define KM64(K, DD, Q) k_ksym_mma64<K, DD, Q><<<grid, KM_THREADS, 0, st>>>(op.n, op.xp, op.hd, g, op.kconst, u, ws, p.nb, p.m, p.S, (int)p.units, stop)
#define KM64D(K, Q)                      \
    switch (op.dm) {                     \
        case 4: KM64(K, 4, Q); break;    \
        case 8: KM64(K, 8, Q); break;    \
        case 16: KM64(K, 16, Q); break;  \
        default: KM64(K, 32, Q); break;  \
    }
        if (op.kind == 1) {
            if (nr == 1) { KM64D(1, 1) } else { KM64D(1, 2) }
        } else {
            if (nr == 1) { KM64D(2, 1) } else { KM64D(2, 2) }
        }
#undef KM64D
#undef KM64
    }
    launch_slot_finish(op.n, p.nb, p.m, p.S, nr, ws, op.scale, mu, u, y, dot_part, stop, st);
}

template <int KIND, int NR, typename T>
static void kmma_dispatch(const KernelOp& op, float c, const double* u, int nr, double* ws,
                          const KmmaPlan& p, const int32_t* stop, hipStream_t st) {
    const dim3 grid((unsigned)kmma_blocks(p, op.kind, nr, NR * sizeof(T) > 8), (unsigned)(nr / NR));
#define KML(DD)                                                                                           \
    k_ksym_mma<KIND, DD, NR, T><<<grid, KM_THREADS, 0, st>>>(op.n, (const bf16x8_t*)op.rrec,               \
                                                             (const bf16x8_t*)op.crec, c, u, ws, p.nb, p.m, \
                                                             p.S, (int)p.units, nr, stop)
    switch (op.dm) {
        case 4: KML(4); break;
        case 8: KML(8); break;
        case 16: KML(16); break;
        default: KML(32); break;
    }
#undef KML
}

int kernel_mma_max_cols(int dm) { return dm <= 16 ? 4 : 2; }

bool kernel_mma_ok(int64_t n, int d) {
    const KmmaPlan p = kmma_plan(n);
    return d <= 32 && (int64_t)p.nb * p.S + 1 <= KM_MAX_SLOTS;
}

KmmaPlanInfo kernel_mma_plan_info(int64_t n, int kind, int nr) {
    const KmmaPlan p = kmma_plan(n);
    return KmmaPlanInfo{p.nb, p.m, p.S, (int)p.units, kmma_blocks(p, kind, 1, nr > 1)};
}

size_t kernel_mma_ws_doubles(int64_t n, int nr) {
    const KmmaPlan p = kmma_plan(n);
    return ((size_t)p.nb * p.S + 1) * nr * (size_t)n;
}

// nr in {1, 2} (also 4 with float64 sums when kernel_mma_max_cols(dm) allows); u, y
// column-major with leading dimension n; ws holds kernel_mma_ws_doubles(n, nr) doubles.
// a32: float32 products and partial sums (estimate grade, nr <= 2).
void launch_kernel_matvec_mma(const KernelOp& op, const double* u, int nr, double mu, double* y,
                              double* dot_part, double* ws, const int32_t* stop, hipStream_t st,
                              bool a32) {
    const KmmaPlan p = kmma_plan(op.n);
    const float c = kernel_c32(op.kind, op.kconst);
    {
        ProfScope prof(nr == 1 && !a32 ? PROF_KERNEL_MATVEC : -1, st);
#define KMD(K)                                                                  \
    if (a32) {                                                                  \
        if (nr == 1) kmma_dispatch<K, 1, float>(op, c, u, nr, ws, p, stop, st); \
        else kmma_dispatch<K, 2, float>(op, c, u, nr, ws, p, stop, st);         \
    } else {                                                                    \
        if (nr == 1) kmma_dispatch<K, 1, double>(op, c, u, nr, ws, p, stop, st); \
        else kmma_dispatch<K, 2, double>(op, c, u, nr, ws, p, stop, st);        \
    }
        if (op.kind == 1) { KMD(1) } else { KMD(2) }
#undef KMD
    }
    launch_slot_finish(op.n, p.nb, p.m, p.S, nr, ws, op.scale, mu, u, y, dot_part, stop, st);
}

// ------------------------------------------------------------------ grouped
// The product and finish of many column blocks (of many requests) in one persistent
// launch each: work item w of the list belongs to the block whose first item is the
// largest <= w, and runs that block's item w - w_mat (the same block of threads
// k_ksym_mma would run for it).  Column blocks whose columns have all stopped are
// skipped.
RR_DEV bool group_pair_runs(const GPair& g) {
    const BState* st = gu(g.st);
    const int32_t nc = gu(g.ncols);
    for (int32_t q = 0; q < nc; ++q)
        if (gu(st[q].run)) return true;
    return false;
}

template <int KIND, int DM, int NR>
__global__ __launch_bounds__(KM_THREADS) __attribute__((amdgpu_waves_per_eu(NR == 1 ? 4 : 2))) void k_group_mat(
    const GTable* __restrict__ tab, int list, const GPair* __restrict__ units, int32_t* ctr) {
    __shared__ int32_t wsh;
    const int32_t off = gu(tab->list[list].off), cnt = gu(tab->list[list].count);
    const int32_t total = gu(tab->list[list].total);
    GroupCursor cur(ctr, &wsh);
    while (true) {
        const int32_t w = cur.next();
        if (w >= total) return;
        const int32_t ui = group_find(units, off, off + cnt, w, [](const GPair& g) { return g.w_mat; });
        const GPair& g = units[ui];
        if (!group_pair_runs(g)) continue;
        constexpr int NC = NR < 2 ? 1 : 2;   // four columns run as two pairs
        for (int q0 = 0; q0 < NR; q0 += NC) {
            if (q0 > 0) __syncthreads();
            ksym_mma_item<KIND, DM, NC, double>((unsigned)(w - gu(g.w_mat)), gu(g.n), gu(g.rrec), gu(g.crec),
                                                gu(g.c), gu(g.u), gu(g.part), gu(g.nb), gu(g.m), gu(g.S), gu(g.items),
                                                gu(g.units), NR, q0);
        }
    }
}

__global__ __launch_bounds__(256 * KF_GROUPS) void k_group_fin(const GTable* __restrict__ tab,
                                                               const GPair* __restrict__ units, int32_t* ctr) {
    __shared__ int32_t wsh;
    const int32_t off = gu(tab->list[GL_FIN].off), cnt = gu(tab->list[GL_FIN].count);
    const int32_t total = gu(tab->list[GL_FIN].total);
    GroupCursor cur(ctr, &wsh);
    while (true) {
        const int32_t w = cur.next();
        if (w >= total) return;
        const int32_t ui = group_find(units, off, off + cnt, w, [](const GPair& g) { return g.w_fin; });
        const GPair& g = units[ui];
        if (!group_pair_runs(g)) continue;
        ksym_mma_finish_block((unsigned)(w - gu(g.w_fin)), (unsigned)gu(g.nfb), 0, gu(g.nr), gu(g.n), KM_RB, gu(g.nb),
                              gu(g.m), gu(g.S), gu(g.nr), gu(g.part), gu(g.scale), gu(g.mu), gu(g.u), gu(g.y),
                              gu(g.dot));
    }
}

int group_mat_list(int kind, int dm, int nr) {
    return GL_MAT + 12 * (kind - 1) + 3 * group_rec_class(dm) + (nr >= 4 ? 2 : nr >= 2 ? 1 : 0);
}

template <int KIND, int DM>
static void group_mat_width(int wc, int list, int blocks, const GTable* tab, const GPair* pairs, int32_t* ctr,
                            hipStream_t st) {
    if (wc == 0) k_group_mat<KIND, DM, 1><<<blocks, KM_THREADS, 0, st>>>(tab, list, pairs, ctr);
    else if (wc == 1) k_group_mat<KIND, DM, 2><<<blocks, KM_THREADS, 0, st>>>(tab, list, pairs, ctr);
    else if constexpr (DM <= 16) k_group_mat<KIND, DM, 4><<<blocks, KM_THREADS, 0, st>>>(tab, list, pairs, ctr);
}

void launch_group_mat(int list, int blocks, const GTable* tab, const GPair* pairs, int32_t* ctr, hipStream_t st) {
    const int kind = (list - GL_MAT) / 12 + 1, rc = ((list - GL_MAT) % 12) / 3, wc = (list - GL_MAT) % 3;
#define KGMD(K)                                                              \
    switch (rc) {                                                            \
        case 0: group_mat_width<K, 4>(wc, list, blocks, tab, pairs, ctr, st); break;   \
        case 1: group_mat_width<K, 8>(wc, list, blocks, tab, pairs, ctr, st); break;   \
        case 2: group_mat_width<K, 16>(wc, list, blocks, tab, pairs, ctr, st); break;  \
        default: group_mat_width<K, 32>(wc, list, blocks, tab, pairs, ctr, st); break; \
    }
    if (kind == 1) { KGMD(1) } else { KGMD(2) }
#undef KGMD
}

void launch_group_fin(int blocks, const GTable* tab, const GPair* pairs, int32_t* ctr, hipStream_t st) {
    k_group_fin<<<blocks, 256 * KF_GROUPS, 0, st>>>(tab, pairs, ctr);
}

}  // namespace rr
