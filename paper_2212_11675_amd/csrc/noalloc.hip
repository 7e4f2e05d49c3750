// aprod 2 without a handle and without any allocation, for callers that cannot allocate
// device memory (code under HIP graph capture, tight serving loops, harnesses that forbid
// it): x += A^T y straight on the caller's arrays in the paper's row layout.
//
// The star-ordered kernel keeps each block's instrumental and global sums in LDS and writes
// them to a partial-sum buffer, reduced by a second kernel; that buffer is `scratch`, a file-scope device array of fixed size that every call on a GPU shares
// (each GPU holds its own copy until the process ends).  Without the attitude-ordered copy a
// setup would build, the attitude columns take one atomic add per coefficient.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "gsr.h"
#include "gsr_internal.hpp"
#include "kernels.hpp"
#include "products.hpp"

using namespace gsr;

namespace {

constexpr int64_t kScratchDoubles = 4 << 20;  // 32 MiB of block partial sums
static __device__ __align__(256) double scratch[kScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch_ptr[kMaxDevices] = {};

// The device address of this device's `scratch` (looked up once per device, with it current).
gsr_status scratch_of(int dev, double** out) {
    if (dev < 0 || dev >= kMaxDevices) return fail(GSR_E_UNSUPPORTED, "device %d", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *out = g_scratch_ptr[dev];
    return GSR_OK;
}

// The star-ordered columns over the caller's row layout, four lanes per row (lane q: slots
// 4k + q).  Astrometric: a star's rows are contiguous; a run is written once by the wave that
// ends it, with a plain read-modify-write when the whole star lies inside the wave's chunk and
// an atomic add when the star continues into a neighbouring chunk.  Instrumental and global:
// accumulated in LDS, the block's n_instr + 1 sums go to part[blockIdx].
static __global__ __launch_bounds__(512) void k_aprod2_star_rows(
    Geo g, const double* __restrict__ vals, const int32_t* __restrict__ star,
    const int32_t* __restrict__ instr, const double* __restrict__ y, double* __restrict__ x,
    double* __restrict__ part, int chunk_rows) {
    extern __shared__ double lds[];  // [n_instr] instrumental, [1] global
    const int nI = g.I;
    double* lglob = lds + nI;
    for (int k = threadIdx.x; k <= nI; k += blockDim.x) lds[k] = 0.0;
    __syncthreads();

    const int lane = threadIdx.x % kWave, rg = lane / kQuad, q = lane % kQuad;
    const int wpb = blockDim.x / kWave;
    const int64_t nchunks = (g.m + chunk_rows - 1) / chunk_rows;
    double gacc = 0.0;
    for (int64_t ch = (int64_t)blockIdx.x * wpb + threadIdx.x / kWave; ch < nchunks;
         ch += (int64_t)gridDim.x * wpb) {
        const int64_t r_beg = ch * (int64_t)chunk_rows;
        const int64_t r_end = min(r_beg + chunk_rows, g.m);
        // stars shared with the neighbouring chunks are written with atomics
        const int32_t shared_first =
            (r_beg > 0 && star[r_beg - 1] == star[r_beg]) ? star[r_beg] : -1;
        const int32_t shared_last =
            (r_end < g.m && star[r_end] == star[r_end - 1]) ? star[r_end - 1] : -1;
        // finished star: row group 0 writes it (astro q; astro 4 from q = 0)
        auto flush = [&](int32_t key, const double (&t)[2]) {
            if (rg != 0) return;
            double* xa = x + (int64_t)kAstro * key;
            if (key == shared_first || key == shared_last) {
                atomic_add_f64(xa + q, t[0]);
                if (q == 0) atomic_add_f64(xa + 4, t[1]);
            } else {
                xa[q] += t[0];
                if (q == 0) xa[4] += t[1];
            }
        };
        double acc[2] = {0.0, 0.0};  // this lane's share of the open run
        int32_t ckey = -1;
        for (int64_t r0 = r_beg; r0 < r_end; r0 += kStepRows) {
            const int64_t r = r0 + rg;
            const bool valid = r < r_end;
            int32_t key = -1;
            double v[2] = {0.0, 0.0};
            if (valid) {
                const double* __restrict__ row = vals + r * kPar + q;
                const double a0 = ld_val(row);
                const double a1 = (q == 0) ? ld_val(row + 4) : 0.0;
                const double a4 = (q != 0) ? ld_val(row + 16) : 0.0;
                const double a5 = ld_val(row + 20);
                key = star[r];
                const double yy = y[r];
                v[0] = a0 * yy;
                v[1] = a1 * yy;
                const double p4 = a4 * yy, p5 = a5 * yy;
                if (q != 0) {
                    const int32_t ia = instr[r * kInstr + q - 1];
                    atomicAdd(lds + ia, p4);
                }
                if (q != 3) {
                    const int32_t ib = instr[r * kInstr + 3 + q];
                    atomicAdd(lds + ib, p5);
                } else {
                    gacc += p5;
                }
            }
            run_step<2, kQuad>(key, v, acc, ckey, flush);
        }
        run_close<2, kQuad>(acc, ckey, flush);
    }
    const double gs = wave_sum(gacc);
    if (lane == 0) atomicAdd(lglob, gs);
    __syncthreads();
    double* dst = part + (int64_t)blockIdx.x * (nI + 1);
    for (int k = threadIdx.x; k <= nI; k += blockDim.x) dst[k] = lds[k];
}

// x[attitude columns of row r] += A[r, 5 + 4a + j] y[r]; four lanes per row, lane j takes
// column t + j of the three axes.
static __global__ __launch_bounds__(256) void k_aprod2_att_rows(Geo g,
                                                                const double* __restrict__ vals,
                                                                const int32_t* __restrict__ att,
                                                                const double* __restrict__ y,
                                                                double* __restrict__ x) {
    const int q = threadIdx.x % kQuad;
    const int64_t step = (int64_t)gridDim.x * blockDim.x / kQuad;
    for (int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kQuad; r < g.m;
         r += step) {
        const double yy = y[r];
        const int64_t c = g.att0 + att[r] + q;
        const double* __restrict__ a = vals + r * kPar + kAstro + q;
#pragma unroll
        for (int ax = 0; ax < kAxes; ++ax)
            atomic_add_f64(x + c + (int64_t)ax * g.T, a[kParAxis * ax] * yy);
    }
}

}  // namespace

extern "C" gsr_status gsr_aprod2_noalloc(const gsr_dims* dims, const double* vals,
                                         const int32_t* star, const int32_t* att,
                                         const int32_t* instr, const double* y, double* x,
                                         void* stream) {
    g_last_error.clear();
    gsr_status st = check_dims(dims);
    if (st != GSR_OK) return st;
    if (dims->n_instr > kInstrLdsMax)
        return fail(GSR_E_UNSUPPORTED,
                    "n_instr %d beyond the maximum of this entry point (%d): its instrumental "
                    "sums must fit one block's LDS and the partial-sum scratch",
                    dims->n_instr, kInstrLdsMax);
    if (dims->n_rows == 0) return GSR_OK;
    if (!vals || !star || !att || !instr || !y || !x) return fail(GSR_E_INVAL, "null argument");
    int dev = 0, n_cu = 0;
    if ((st = check_device(&dev, &n_cu)) != GSR_OK) return st;
    double* part = nullptr;
    if ((st = scratch_of(dev, &part)) != GSR_OK) return st;
    const Geo g = make_geo(dims);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // one partial row (n_instr + 1 sums) per block: as many blocks as the scratch holds, at
    // most two per compute unit
    const int64_t ncols = (int64_t)g.I + 1;
    const int blocks = (int)std::max<int64_t>(
        1, std::min<int64_t>(2 * (int64_t)n_cu, kScratchDoubles / ncols));
    constexpr int kThreads = 512;
    const int64_t waves = (int64_t)blocks * kThreads / kWave;
    int64_t chunk = std::max<int64_t>(kStepRows, std::min<int64_t>(1024, g.m / (4 * waves)));
    chunk = (chunk + kStepRows - 1) / kStepRows * kStepRows;
    const size_t lds_bytes = sizeof(double) * ncols;
    hipLaunchKernelGGL(k_aprod2_star_rows, dim3(blocks), dim3(kThreads), lds_bytes, s, g, vals,
                       star, instr, y, x, part, (int)chunk);
    const int slices = std::max(1, std::min(32, blocks / 8));
    hipLaunchKernelGGL(k_reduce_partials, dim3((unsigned)((ncols + 255) / 256), slices),
                       dim3(256), 0, s, (int)ncols, blocks, part, x + g.ins0, nullptr, 0);
    const int64_t att_blocks = std::min<int64_t>((g.m * kQuad + 255) / 256, 8 * (int64_t)n_cu);
    hipLaunchKernelGGL(k_aprod2_att_rows, dim3((unsigned)att_blocks), dim3(256), 0, s, g, vals,
                       att, y, x);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "gsr_aprod2_noalloc launch");
    return GSR_OK;
}
