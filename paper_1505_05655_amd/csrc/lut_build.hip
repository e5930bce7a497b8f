// LUT build kernel (LUT generation, a task named in §I): every entry of
// lut[b][d][v] from the binary64 calibration polynomial of (b, d).
//
// One thread computes 8 consecutive levels of one LUT row and writes them
// with a single 16-byte store when the row pitch allows it. For rows of 512
// levels or more, a wave evaluates whole rows, 512 consecutive levels per
// pass, so the row index and the row's coefficients are wave-uniform (scalar
// loads, no per-lane index arithmetic) and each wave store writes 1 KiB
// contiguously.
// The arithmetic is the fixed, uncontracted binary64 sequence of
// rc::lut_round, so every entry is bit-identical to the CPU definition.
#include <algorithm>

#include "device_ops.h"
#include "kernels.h"

namespace rc {

__global__ __launch_bounds__(256) void k_lut_build(const double* __restrict__ coeffs, int64_t rows,
                                                   int32_t levels, int32_t chunks,
                                                   int32_t log_chunks, int32_t vec,
                                                   uint16_t* __restrict__ lut) {
    const int64_t total = rows * (int64_t)chunks;
    const uint32_t top2 = (uint32_t)(levels - 1) * 0x10001u;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        // Row and 8-level chunk of this thread (a shift when chunks is 2^k).
        const int64_t row = log_chunks >= 0 ? (t >> log_chunks) : t / chunks;
        const int v0 = (int)(t - row * chunks) * 8;
        const double* a = coeffs + row * 4;
        double x[8];
        levels8(v0, x);
        store_lut8(lut + row * (int64_t)levels + v0,
                   lut_eight(a[0], a[1], a[2], a[3], x, top2), levels - v0, vec != 0, false);
    }
}

// Coefficients of R consecutive rows from row0 (rows past the last: the last).
template <int R>
__device__ __forceinline__ void load_coeffs(const double* __restrict__ coeffs, int64_t row0,
                                            int64_t rows, double (&a)[R][4]) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const double* c = coeffs + (row0 + i < rows ? row0 + i : rows - 1) * 4;
#pragma unroll
        for (int k = 0; k < 4; ++k) a[i][k] = c[k];
    }
}

// Wave w of the grid evaluates rows R w .. R w + R - 1 (then R times the
// number of waves further on), 512 levels per pass; the doubles of a pass's
// levels are converted once for the R rows. Bound by instruction issue (10
// operations per entry at 4 cycles a wave, the cheapest first: 6 of the
// polynomial, 1 level, 1 rounding, 1 conversion, half a packed conversion and
// half a packed minimum) and, from there, by its stores. nt: non-temporal
// 16-byte stores, for LUTs larger than the L2 caches, which the correction
// after the build does not find there anyway (on the 3 x 50000 x 6000 scene
// the correction after a build took 0.77 ms instead of 0.83 ms on one GPU, and
// the same 0.82-0.84 ms either way on two others; the build itself is not
// slower).
template <int R>
__global__ __launch_bounds__(256) void k_lut_build_rows(const double* __restrict__ coeffs,
                                                        int64_t rows, int32_t levels, int32_t vec,
                                                        int32_t nt, uint16_t* __restrict__ lut) {
    const int lane = threadIdx.x & 63;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const uint32_t top2 = (uint32_t)(levels - 1) * 0x10001u;
    for (int64_t g = (int64_t)blockIdx.x * (blockDim.x >> 6) +
                     __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
         g * R < rows; g += nwaves) {
        double a[R][4];
        load_coeffs<R>(coeffs, g * R, rows, a);
        for (int v0 = lane * 8; v0 < levels; v0 += 512) {
            double x[8];
            levels8(v0, x);
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if (g * R + i < rows)
                    store_lut8(lut + (g * R + i) * (int64_t)levels + v0,
                               lut_eight(a[i][0], a[i][1], a[i][2], a[i][3], x, top2),
                               levels - v0, vec != 0, nt != 0);
            }
        }
    }
}

// rc_lut_build_ws: R consecutive LUT rows per wave, evaluated and stored as
// k_lut_build_rows does, and encoded from the registers they are stored from;
// the encoding goes to the [band][block][detector] layout rc_correct_ws uses,
// so its tiles can stage it without an encoding pass. A plane line of 16
// detectors holds the words of several waves: workgroups are renumbered so
// that each XCD takes one range of rows and its L2 merges them.
template <int R>
__global__ __launch_bounds__(256) void k_lut_build_ws(const double* __restrict__ coeffs,
                                                      int64_t rows, int32_t detectors,
                                                      int32_t levels, uint16_t* __restrict__ lut,
                                                      int32_t lut_vec, int32_t xcds,
                                                      uint64_t* __restrict__ planes,
                                                      int16_t* __restrict__ heads) {
    const int NB = (levels + 63) >> 6;
    const uint32_t top2 = (uint32_t)(levels - 1) * 0x10001u;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t g = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x, xcds) *
                         (blockDim.x >> 6) +
                     __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
         g * R < rows; g += nwaves) {
        double a[R][4];
        load_coeffs<R>(coeffs, g * R, rows, a);
        size_t o[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t b = (g * R + i) / detectors;
            o[i] = (size_t)b * (size_t)NB * (size_t)detectors + (size_t)(g * R + i - b * detectors);
        }
        encode_rows<R, false>(
            levels,
            [&](int v0, bool, u32x4 (&w)[R]) {
                double x[8];
                levels8(v0, x);
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    w[i] = lut_eight(a[i][0], a[i][1], a[i][2], a[i][3], x, top2);
                    if (g * R + i < rows && v0 < levels)
                        store_lut8(lut + (g * R + i) * (int64_t)levels + v0, w[i], levels - v0,
                                   lut_vec != 0, true);
                }
            },
            [&](int i, int blk, uint64_t z, int16_t h) {
                if (g * R + i >= rows) return;
                planes[o[i] + (size_t)blk * (size_t)detectors] = z;
                heads[o[i] + (size_t)blk * (size_t)detectors] = h;
            });
    }
}

// The dense encoding of a LUT in memory ([bands][blocks][detectors] planes and
// headers): R consecutive rows per wave, their loads of a pass in flight
// together, workgroups renumbered as in k_lut_build_ws.
template <int R>
__global__ __launch_bounds__(256) void k_dense_encode(const uint16_t* __restrict__ lut,
                                                      int64_t rows, int32_t detectors,
                                                      int32_t levels, int32_t lut_vec,
                                                      int32_t xcds, uint64_t* __restrict__ planes,
                                                      int16_t* __restrict__ heads) {
    const int NB = (levels + 63) >> 6;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t g = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x, xcds) *
                         (blockDim.x >> 6) +
                     __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
         g * R < rows; g += nwaves) {
        size_t o[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t b = (g * R + i) / detectors;
            o[i] = (size_t)b * (size_t)NB * (size_t)detectors + (size_t)(g * R + i - b * detectors);
        }
        encode_rows<R, true>(
            levels,
            [&](int v0, bool whole, u32x4 (&w)[R]) {
#pragma unroll
                for (int i = 0; i < R; ++i)
                    w[i] = load_lut8(lut + (g * R + i < rows ? g * R + i : rows - 1) *
                                               (int64_t)levels,
                                     v0, levels, whole, lut_vec != 0);
            },
            [&](int i, int blk, uint64_t z, int16_t h) {
                if (g * R + i >= rows) return;
                planes[o[i] + (size_t)blk * (size_t)detectors] = z;
                heads[o[i] + (size_t)blk * (size_t)detectors] = h;
            });
    }
}

namespace {

// Workgroups of 4 waves for `rows` rows, `per` per wave (grid-stride beyond
// 2^20 workgroups).
dim3 row_grid(int64_t rows, int per) {
    return dim3((unsigned)std::min<int64_t>((rows + 4 * per - 1) / (4 * per), (int64_t)1 << 20));
}

bool rows_vec(const uint16_t* lut, int32_t levels) {
    return levels % 8 == 0 && ((uintptr_t)lut & 15u) == 0;
}

}  // namespace

hipError_t launch_lut_build_ws(const double* coeffs, int64_t rows, int32_t detectors,
                               int32_t levels, uint16_t* lut, uint64_t* planes, int16_t* heads,
                               int xcds, hipStream_t stream) {
    const int vec = rows_vec(lut, levels) ? 1 : 0;
    hipLaunchKernelGGL(k_lut_build_ws<2>, row_grid(rows, 2), dim3(256), 0, stream, coeffs, rows,
                       detectors, levels, lut, vec, xcds, planes, heads);
    return hipGetLastError();
}

hipError_t launch_dense_encode(const uint16_t* lut, int32_t bands, int32_t detectors,
                               int32_t levels, uint64_t* planes, int16_t* heads, int xcds,
                               hipStream_t stream) {
    const int64_t rows = (int64_t)bands * detectors;
    if (rows <= 0) return hipSuccess;
    const int vec = rows_vec(lut, levels) ? 1 : 0;
    hipLaunchKernelGGL(k_dense_encode<1>, row_grid(rows, 1), dim3(256), 0, stream, lut, rows,
                       detectors, levels, vec, xcds, planes, heads);
    return hipGetLastError();
}

hipError_t launch_lut_build(const double* coeffs, int64_t rows, int32_t levels, uint16_t* lut,
                            hipStream_t stream) {
    const bool vec = rows_vec(lut, levels);
    if (levels >= 512) {
        // Non-temporal above the GPU's aggregate L2 (8 XCDs x 4 MiB).
        const int nt = (double)rows * (double)levels * 2.0 > (double)(32u << 20) ? 1 : 0;
        // Rows per wave: 4 while that leaves every SIMD 4 waves, else 1.
        if (rows >= 16384)
            hipLaunchKernelGGL(k_lut_build_rows<4>, row_grid(rows, 4), dim3(256), 0, stream,
                               coeffs, rows, levels, vec ? 1 : 0, nt, lut);
        else
            hipLaunchKernelGGL(k_lut_build_rows<1>, row_grid(rows, 1), dim3(256), 0, stream,
                               coeffs, rows, levels, vec ? 1 : 0, nt, lut);
        return hipGetLastError();
    }
    const int32_t chunks = (levels + 7) / 8;
    int32_t log_chunks = -1;
    if ((chunks & (chunks - 1)) == 0) {
        log_chunks = 0;
        while ((1 << log_chunks) < chunks) ++log_chunks;
    }
    const int64_t total = rows * (int64_t)chunks;
    const int threads = 256;
    int64_t blocks = (total + threads - 1) / threads;
    if (blocks > (int64_t)1 << 20) blocks = (int64_t)1 << 20;  // grid-stride beyond this
    hipLaunchKernelGGL(k_lut_build, dim3((unsigned)blocks), dim3(threads), 0, stream, coeffs, rows,
                       levels, chunks, log_chunks, vec ? 1 : 0, lut);
    return hipGetLastError();
}

}  // namespace rc
