// ebic_layout.hip -- upload kernels: the resident matrix layout.
//
// The matrix is kept column-major (one column of 64 consecutive rows is one
// coalesced 256-byte segment for a wave) with a leading dimension padded to
// a multiple of 64 rows; padding rows hold 0. Missing cells are stored as
// NaN: the paper lets the user mark missing values with a predefined value
// (Methods, "Handling missing values"), so cells equal to that sentinel are
// converted here. An optional second copy holds the fill value in place of
// every missing cell, for the mode in which missing values take part in the
// comparison.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ebic_internal.h"

namespace ebic {

namespace {

// ---------------------------------------------------------------------------
// Layout: 64x64 tiles through LDS. Row-major source -> column-major
// destination with coalesced reads (along a source row) and coalesced writes
// (along a destination column). Sentinel cells become NaN.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_layout(const float *__restrict__ src, int64_t ld_src, int32_t src_col_major, int64_t nr,
         int32_t cols, int64_t r0, float *__restrict__ dst, int64_t ld, float sentinel,
         float *__restrict__ dst_fill, float fill)
{
    __shared__ float t[64][65];
    const int64_t rb = (int64_t)blockIdx.x * 64;  // first source row of the tile
    const int32_t cb = blockIdx.y * 64;            // first column of the tile
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 x 4
    if (!src_col_major) {
        for (int y = ty; y < 64; y += 4) {
            const int64_t r = rb + y;
            const int32_t c = cb + tx;
            t[y][tx] = (r < nr && c < cols) ? src[r * ld_src + c] : 0.f;
        }
    } else {
        for (int y = ty; y < 64; y += 4) {
            const int64_t r = rb + tx;
            const int32_t c = cb + y;
            t[tx][y] = (r < nr && c < cols) ? src[(int64_t)c * ld_src + r] : 0.f;
        }
    }
    __syncthreads();
    for (int y = ty; y < 64; y += 4) {
        const int32_t c = cb + y;
        const int64_t r = rb + tx;
        if (c < cols && r < nr) {
            float v = t[tx][y];
            const bool missing = v != v || v == sentinel;
            if (missing) v = __builtin_nanf("");
            dst[(int64_t)c * ld + r0 + r] = v;
            if (dst_fill) dst_fill[(int64_t)c * ld + r0 + r] = missing ? fill : v;
        }
    }
}

// ---------------------------------------------------------------------------
// Rank codes: for every cell, the number of cells of its row that are
// smaller (IEEE <, so NaN is never smaller and -0 is not smaller than +0).
// A block stages 32 rows of all columns in LDS; the half-waves (lane & 31 =
// row) each count for an even run of the columns. Bound by the comparisons,
// cols x cols a row: a compare and an add of its carry each, so a half-wave
// counts for 16 columns per value read (then eight, then four), and equal
// values are found without a comparison of their own: the counts of a row
// of distinct values add up to cols x (cols - 1) / 2, and each pair of equal
// values takes one off. Blocks of 32 rows rather than 64 even out the last
// wave of blocks. 10-bit codes at 54,675 x 178: 330 us with a column at a
// time and equality counted beside it, 128 us so (the comparisons alone take
// 88); 436,444 x 310 6.8 and 2.4 ms.
// ---------------------------------------------------------------------------
constexpr int kCodeRows = 32;

template <int R>
__device__ __forceinline__ void count_smaller(const float *t, int32_t cols, int32_t c0, int row, uint32_t (&n)[R])
{
    float v[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        v[k] = t[min(c0 + k, cols - 1) * kCodeRows + row];
        n[k] = 0;
    }
#pragma unroll 4
    for (int32_t j = 0; j < cols; ++j) {
        const float u = t[j * kCodeRows + row];
#pragma unroll
        for (int k = 0; k < R; ++k) n[k] += u < v[k] ? 1u : 0u;
    }
}

// put(column, count) for every column of this half-wave.
template <class Put>
__device__ __forceinline__ void rank_columns(const float *t, int32_t cols, Put &&put)
{
    const int halves = blockDim.x / kCodeRows, row = threadIdx.x & (kCodeRows - 1);
    const int32_t per = (cols + halves - 1) / halves, first = (int32_t)(threadIdx.x / kCodeRows) * per;
    const int32_t mine = min(per, cols - first);
    auto run = [&](auto size, int32_t o) {
        constexpr int R = decltype(size)::value;
        uint32_t n[R];
        count_smaller<R>(t, cols, first + o, row, n);
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (o + k < mine) put(first + o + k, n[k]);
    };
    int32_t o = 0;  // (the same in every half-wave)
    for (; o + 12 < per; o += 16) run(std::integral_constant<int, 16>(), o);
    for (; o + 4 < per; o += 8) run(std::integral_constant<int, 8>(), o);
    for (; o < per; o += 4) run(std::integral_constant<int, 4>(), o);
}

// The codes as FP16 integers; a missing cell gets NaN. Padding rows get 0.
__global__ void __launch_bounds__(1024)
k_codes(const float *__restrict__ X, int64_t rows, int64_t ld, int32_t cols, uint16_t *__restrict__ C)
{
    extern __shared__ float t[];  // [cols][kCodeRows]
    const int row = threadIdx.x & (kCodeRows - 1);
    const int64_t r = (int64_t)blockIdx.x * kCodeRows + row;
    for (int32_t c = threadIdx.x / kCodeRows; c < cols; c += blockDim.x / kCodeRows)
        t[c * kCodeRows + row] = X[(int64_t)c * ld + r];
    __syncthreads();
    const bool live = r < rows;
    rank_columns(t, cols, [&](int32_t c, uint32_t n) {
        const float v = t[c * kCodeRows + row];
        uint16_t code = __half_as_ushort(__int2half_rn((int32_t)n));  // exact: n < 2048
        if (v != v) code = kCodeNaN;
        C[(int64_t)c * ld + r] = live ? code : (uint16_t)0;
    });
}

// The fill-substituted values of row r into t, a missing cell noted; then
// put(column, count) for every column, and *tie = 1 if the row is below
// `rows` and holds two equal values.
template <class Put>
__device__ __forceinline__ void rank_filled(const float *__restrict__ X, int64_t rows, int64_t ld, int32_t cols,
                                            int64_t r, float fill, float *t, int32_t *__restrict__ has_nan,
                                            int32_t *__restrict__ tie, Put &&put)
{
    __shared__ uint32_t sum[kCodeRows];
    const int row = threadIdx.x & (kCodeRows - 1);
    const bool live = r < rows;
    bool missing = false;
    if (threadIdx.x < kCodeRows) sum[row] = 0;
    for (int32_t c = threadIdx.x / kCodeRows; c < cols; c += blockDim.x / kCodeRows) {
        float v = live ? X[(int64_t)c * ld + r] : 0.f;
        if (v != v) {
            missing = true;
            v = fill;
        }
        t[c * kCodeRows + row] = v;
    }
    if (missing) *has_nan = 1;
    __syncthreads();
    uint32_t total = 0;
    rank_columns(t, cols, [&](int32_t c, uint32_t n) {
        total += n;
        put(c, live ? n : 0u);
    });
    atomicAdd(&sum[row], total);
    __syncthreads();
    // (cols at most 512: the sum of a row's counts stays below 2^17)
    if (threadIdx.x < kCodeRows && live && sum[row] != (uint32_t)cols * (uint32_t)(cols - 1) / 2) *tie = 1;
}

// ---------------------------------------------------------------------------
// Byte or 16-bit rank codes: of the fill-substituted values, in the
// interleaved order of the SWAR evaluation. Bytes: within each 256-row
// group the word of lane l holds rows l, 64 + l, 128 + l, 192 + l; 16 bits:
// within each 128-row group it holds rows l and 64 + l. Rows past the
// matrix get 0. Also flags any missing cell, and each 512-row group with a
// row that holds two equal values.
// ---------------------------------------------------------------------------
template <typename C>
__global__ void __launch_bounds__(1024)
k_swar_codes(const float *__restrict__ X, int64_t rows, int64_t ld, int32_t cols, float fill,
             C *__restrict__ out, int64_t ld_out, int32_t *__restrict__ has_nan, int32_t *__restrict__ ties, int64_t r0)
{
    extern __shared__ float t[];  // [cols][kCodeRows]
    const int64_t r = r0 + (int64_t)blockIdx.x * kCodeRows + (threadIdx.x & (kCodeRows - 1));
    // Position of row r (in elements of C) inside its interleaved group.
    const int64_t pos = sizeof(C) == 1 ? (r & ~(int64_t)255) + 4 * (r & 63) + ((r >> 6) & 3)
                                       : (r & ~(int64_t)127) + 2 * (r & 63) + ((r >> 6) & 1);
    rank_filled(X, rows, ld, cols, r, fill, t, has_nan, ties + (r >> 9),
                [&](int32_t c, uint32_t n) { out[(int64_t)c * ld_out + pos] = (C)n; });
}

// 10-bit rank codes: the same counts, three rows per 32-bit word. Rows
// [64 b, 64 b + 64) are field b mod 3 of 192-row group b / 3: each code is
// OR-ed into its word (the blocks of a group write disjoint fields of the
// same words). Flags a missing cell, and each 192-row group with a row that
// holds two equal values.
__global__ void __launch_bounds__(1024)
k_t10_codes(const float *__restrict__ X, int64_t rows, int64_t ld, int32_t cols, float fill,
            uint32_t *__restrict__ out, int64_t ld_words, int32_t *__restrict__ has_nan,
            int32_t *__restrict__ ties, int64_t r0)
{
    extern __shared__ float t[];  // [cols][kCodeRows]
    const int64_t first = r0 + (int64_t)blockIdx.x * kCodeRows, r = first + (threadIdx.x & (kCodeRows - 1));
    const int32_t b = (int32_t)(first / 64), group = b / 3, shift = 10 * (b % 3);
    uint32_t *words = out + (int64_t)group * 64 + (r & 63);
    rank_filled(X, rows, ld, cols, r, fill, t, has_nan, ties + group, [&](int32_t c, uint32_t n) {
        if (n) atomicOr(words + (int64_t)c * ld_words, n << shift);
    });
}

__global__ void k_zero_pad(float *__restrict__ dst, int64_t rows, int64_t ld, int32_t cols)
{
    const int64_t pad = ld - rows;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= pad * cols) return;
    const int64_t c = idx / pad, r = rows + idx % pad;
    dst[c * ld + r] = 0.f;
}

}  // namespace

// Threads of a code block: with its LDS (128 bytes per column) they leave
// room for 28 waves per CU or more, and a half-wave counts for 16 columns or
// so: 20,000 x 500 takes 569, 393 and 374 us with four, eight and 16 waves,
// 54,675 x 178 takes 134, 128 and 164, 436,444 x 64 (bytes) 133, 137 and 267.
static unsigned code_threads(int32_t cols)
{
    return 64u * (cols <= 128 ? 4 : cols <= 320 ? 8 : 16);
}

hipError_t launch_codes(const float *X, int64_t rows, int64_t ld, int32_t cols, uint16_t *C,
                        hipStream_t s)
{
    if (cols > kMaxCodeCols) return hipErrorInvalidValue;
    const size_t lds = (size_t)cols * kCodeRows * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_codes),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    clear_last_error();
    hipLaunchKernelGGL(k_codes, dim3((unsigned)(ld / kCodeRows)), dim3(code_threads(cols)), lds, s, X, rows, ld, cols, C);
    return hipGetLastError();
}

hipError_t launch_byte_codes(const float *X, int64_t rows, int64_t ld, int32_t cols, float fill,
                             uint8_t *B, int64_t ldb, int32_t *has_nan, int32_t *ties, int64_t r0, int64_t r1,
                             hipStream_t s)
{
    if (cols > kMaxByteCols || ldb % 512 != 0 || ldb < rows || r0 % kUploadUnit != 0 || r0 >= r1 || r1 % kCodeRows != 0 ||
        r1 > ldb)
        return hipErrorInvalidValue;
    const size_t lds = (size_t)cols * kCodeRows * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_swar_codes<uint8_t>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    clear_last_error();
    hipLaunchKernelGGL(k_swar_codes<uint8_t>, dim3((unsigned)((r1 - r0) / kCodeRows)), dim3(code_threads(cols)), lds, s, X,
                       rows, ld, cols, fill, B, ldb, has_nan, ties, r0);
    return hipGetLastError();
}

hipError_t launch_half_codes(const float *X, int64_t rows, int64_t ld, int32_t cols, float fill,
                             uint8_t *Hc, int64_t ldh, int32_t *has_nan, int32_t *ties, hipStream_t s)
{
    if (cols > kMaxCodeCols || ldh % 512 != 0 || ldh / 2 < rows) return hipErrorInvalidValue;
    const size_t lds = (size_t)cols * kCodeRows * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_swar_codes<uint16_t>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    clear_last_error();
    hipLaunchKernelGGL(k_swar_codes<uint16_t>, dim3((unsigned)(ldh / 2 / kCodeRows)), dim3(code_threads(cols)), lds, s, X, rows,
                       ld, cols, fill, reinterpret_cast<uint16_t *>(Hc), ldh / 2, has_nan, ties, (int64_t)0);
    return hipGetLastError();
}

hipError_t launch_t10_codes(const float *X, int64_t rows, int64_t ld, int32_t cols, float fill,
                            uint8_t *T10, int64_t ld10, int32_t *has_nan, int32_t *ties, int64_t r0, int64_t r1,
                            hipStream_t s)
{
    const int64_t groups = (rows + kT10Rows - 1) / kT10Rows;
    if (cols > kMaxT10Cols || ld10 < groups * 256 || ld10 % 256 != 0 || ld / 64 < (rows + 63) / 64 ||
        r0 % kUploadUnit != 0 || r0 >= r1 || r1 % 64 != 0 || r1 > groups * kT10Rows)
        return hipErrorInvalidValue;
    const size_t lds = (size_t)cols * kCodeRows * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_t10_codes),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // (X is read only for rows below `rows`)
    clear_last_error();
    hipLaunchKernelGGL(k_t10_codes, dim3((unsigned)((r1 - r0) / kCodeRows)), dim3(code_threads(cols)), lds, s, X, rows, ld,
                       cols, fill, reinterpret_cast<uint32_t *>(T10), ld10 / 4, has_nan, ties, r0);
    return hipGetLastError();
}

hipError_t launch_layout(const float *src, int64_t ld_src, bool src_col_major, int64_t nr,
                         int32_t cols, int64_t r0, float *dst, int64_t ld, float sentinel,
                         float *dst_fill, float fill, hipStream_t s)
{
    if (nr <= 0) return hipSuccess;
    dim3 grid((unsigned)((nr + 63) / 64), (unsigned)((cols + 63) / 64));
    clear_last_error();
    hipLaunchKernelGGL(k_layout, grid, dim3(256), 0, s, src, ld_src, (int32_t)src_col_major, nr,
                       cols, r0, dst, ld, sentinel, dst_fill, fill);
    return hipGetLastError();
}

hipError_t launch_zero_pad(float *dst, int64_t rows, int64_t ld, int32_t cols, hipStream_t s)
{
    const int64_t total = (ld - rows) * cols;
    if (total <= 0) return hipSuccess;
    const int threads = 256;
    clear_last_error();
    hipLaunchKernelGGL(k_zero_pad, dim3((unsigned)((total + threads - 1) / threads)), dim3(threads),
                       0, s, dst, rows, ld, cols);
    return hipGetLastError();
}

}  // namespace ebic
