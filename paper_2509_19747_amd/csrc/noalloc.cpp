// rr_apply_operator_noalloc: the operator product y = (A + mu I) u of
// rr_apply_operator (the matvec of every Krylov iteration, Section 6) for callers
// that cannot allocate device memory (code under graph capture, tight serving
// loops).  Every buffer the product needs beyond u and y -- the point records of
// a kernel operator, the float32 copy of a dense A, the partial-sum slots and the
// dot partials -- is carved from one file-scope device array, `scratch`.
//
// The array's host-side name is not a device address: its address on each device
// is taken once per device with hipGetSymbolAddress (first call on that device,
// with the device current) and only that pointer is handed to kernels.  Calls on
// one device share the array and it keeps the last call's contents; calls that
// overlap on one device race.  Nothing here allocates, frees or synchronises.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "ctx.hpp"

namespace {

// What a call may count against (accepted_bytes), and the array, which also holds what
// the packed records take beyond that count (at most 6.3 MiB for any accepted operator, with
// 32 coordinates).
constexpr size_t kScratchBytes = (size_t)64 << 20;
constexpr size_t kArrayBytes = (size_t)72 << 20;
constexpr int kMaxDevices = 64;

__device__ __align__(256) unsigned char scratch[kArrayBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device.
void* scratch_on_device() {
    int dev = 0;
    RR_HIP(hipGetDevice(&dev));
    RR_REQUIRE(dev >= 0 && dev < kMaxDevices, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            throw rr::RrError{RR_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)};
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

// Bump layout inside the scratch array (256-byte aligned pieces).
struct Carve {
    size_t off = 0;
    size_t take(size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) / 256 * 256;
        return o;
    }
};

struct Layout {
    size_t rrec = 0, crec = 0, xp = 0, hd = 0, a32 = 0, part = 0, ws = 0, total = 0;
};

Layout layout_for(const rr_operator& A, int32_t prec) {
    Layout L;
    Carve c;
    const int64_t n = A.n;
    if (rr::is_kernel(A)) {
        const int dm = rr::kernel_record_len(A.d);
        if (prec == RR_PREC_FP64) {
            L.xp = c.take(rr::kernel_mma_record64_bytes(n, dm));
            L.hd = c.take((size_t)n * sizeof(double));
        } else {
            L.rrec = c.take(rr::kernel_mma_record_bytes(n, dm));
            L.crec = c.take(rr::kernel_mma_record_bytes(n, dm));
        }
        L.part = c.take((size_t)rr::kernel_matvec_blocks(n) * sizeof(double));
        L.ws = c.take((rr::kernel_mma_ws_doubles(n, 1) + 1) * sizeof(double));
    } else {
        if (prec != RR_PREC_FP64) L.a32 = c.take((size_t)n * n * sizeof(float));
        L.part = c.take((size_t)rr::dense_matvec_blocks(n) * sizeof(double));
    }
    L.total = c.off;
    return L;
}

// The bytes that a call counts against kScratchBytes: float32 and float64 point records,
// norms and the slot partials for a kernel operator, the float32 copy for a dense one.
size_t accepted_bytes(const rr_operator& A, int32_t prec) {
    Carve c;
    const int64_t n = A.n;
    if (rr::is_kernel(A)) {
        const int dm = rr::kernel_record_len(A.d);
        c.take((size_t)n * sizeof(float));
        c.take((size_t)n * dm * sizeof(float));
        c.take((size_t)n * dm * sizeof(double));
        c.take((size_t)n * sizeof(double));
        c.take((size_t)rr::kernel_matvec_blocks(n) * sizeof(double));
        c.take((rr::kernel_mma_ws_doubles(n, 1) + 1) * sizeof(double));
    } else {
        if (prec != RR_PREC_FP64) c.take((size_t)n * n * sizeof(float));
        c.take((size_t)rr::dense_matvec_blocks(n) * sizeof(double));
    }
    return c.off;
}

}  // namespace

using namespace rr;

extern "C" rr_status rr_apply_operator_noalloc(const rr_operator* A, double mu, int32_t prec, const double* u,
                                               double* y, void* hip_stream) {
    return guarded([&]() -> rr_status {
        validate_operator(A);
        RR_REQUIRE(u != nullptr && y != nullptr, "u or y is null");
        RR_REQUIRE(std::isfinite(mu), "mu must be finite");
        RR_REQUIRE(prec >= 0 && prec <= 2, "unknown precision");
        const size_t need = accepted_bytes(*A, prec);
        const Layout L = layout_for(*A, prec);
        if (need > kScratchBytes || L.total > kArrayBytes || (is_kernel(*A) && !kernel_mma_ok(A->n, A->d)))
            throw RrError{RR_EINVAL, "operator too large for the no-allocation scratch: needs " +
                                         std::to_string(need) + " bytes, the scratch holds " +
                                         std::to_string(kScratchBytes)};
        require_device();
        unsigned char* base = (unsigned char*)scratch_on_device();
        hipStream_t st = (hipStream_t)hip_stream;
        const int64_t n = A->n;
        double* part = (double*)(base + L.part);
        if (is_kernel(*A)) {
            KernelOp k;
            k.kind = A->kind;
            k.n = n;
            k.d = A->d;
            k.pts = A->pts;
            k.dm = kernel_record_len(A->d);
            k.kconst = A->kconst;
            k.scale = A->scale;
            k.sqn = nullptr;
            k.xa = nullptr;
            if (prec == RR_PREC_FP64) {
                k.xp = (const double*)(base + L.xp);
                k.hd = (const double*)(base + L.hd);
                launch_kmma_records64(k, (double*)(base + L.xp), (double*)(base + L.hd), st);
            } else {
                k.rrec = base + L.rrec;
                k.crec = base + L.crec;
                launch_kmma_records(k, base + L.rrec, base + L.crec, st);
            }
            launch_kernel_matvec(k, prec == RR_PREC_FP64, u, mu, y, part, (double*)(base + L.ws), nullptr, st);
        } else if (prec != RR_PREC_FP64) {
            float* a32 = (float*)(base + L.a32);
            launch_copy_mat(DT_F64, A->A, A->lda, DT_F32, a32, n, n, n, st);
            launch_dense_matvec(DT_F32, n, a32, n, u, mu, y, part, nullptr, st);
        } else {
            launch_dense_matvec(DT_F64, n, A->A, A->lda, u, mu, y, part, nullptr, st);
        }
        RR_HIP(hipGetLastError());
        return RR_OK;
    });
}

extern "C" size_t rr_noalloc_scratch_bytes(void) { return kScratchBytes; }
