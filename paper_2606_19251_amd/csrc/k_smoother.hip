// Sparse pseudo-inverse smoother assembly (paper Sec. 3.1, Eq. 5):
//   q_ii = f_d(a_ii/s) / a_ii,   q_ij = f_o(a_ij/s) / (a_ii + a_jj),   s = max |offdiag(A)|,
//   f_d(x) = d0 + x(d1 + x(d2 + ...)),   f_o(x) = x(o1 + x(o2 + ...)).
// Evaluated in FP64 with Horner's rule, each operation rounded on its own (this file is
// built with -ffp-contract=off and the pragma below) and IEEE division, so the values
// are reproducible bit for bit by any implementation that follows the same order.
// The entries are streamed per block of rows with the row data (coefficients, scale, a_ii) in
// LDS; the diagonal of the neighbour j is a gather from the level's diagonal array.
#include "kernels.hpp"

namespace amgg {

namespace {

__device__ __forceinline__ double horner_diag(double x, const double* c, int deg) {
#pragma clang fp contract(off)
    double t = c[deg];
    for (int k = deg - 1; k >= 0; --k) t = c[k] + x * t;
    return t;
}

__device__ __forceinline__ double horner_off(double x, const double* o, int deg) {
#pragma clang fp contract(off)
    // o[0] = o1 ... o[deg-1] = o_deg
    double t = o[deg - 1];
    for (int k = deg - 2; k >= 0; --k) t = o[k] + x * t;
    return x * t;
}

// Row i of Q and of its diagonal with coefficients c[0..2deg] and scale s.
__device__ __forceinline__ void assemble_row(int32_t i, const int32_t* __restrict__ ptr,
                                             const int32_t* __restrict__ col, const double* __restrict__ val,
                                             const double* __restrict__ diag, const double* c, int deg, double s,
                                             double* __restrict__ q64, float* __restrict__ q32,
                                             double* __restrict__ qd64, float* __restrict__ qd32) {
#pragma clang fp contract(off)
    const double aii = diag[i];
    const int32_t pb = ptr[i], pe = ptr[i + 1];
    // eight entries at a time: their columns and values, then the neighbours' diagonals, are
    // loaded together (a past-the-end slot re-reads the row's last entry and is not stored)
    constexpr int kE = 8;
    for (int32_t base = pb; base < pe; base += kE) {
        int32_t j[kE];
        double a[kE], dj[kE];
#pragma unroll
        for (int q = 0; q < kE; ++q) {
            const int32_t p = min(base + q, pe - 1);
            j[q] = col[p];
            a[q] = val[p];
        }
#pragma unroll
        for (int q = 0; q < kE; ++q) dj[q] = diag[j[q]];
#pragma unroll
        for (int q = 0; q < kE; ++q) {
            const int32_t p = base + q;
            if (p < pe) {
                const double x = a[q] / s;
                double v;
                if (j[q] == i) {
                    v = horner_diag(x, c, deg) / a[q];
                    qd64[i] = v;
                    qd32[i] = static_cast<float>(v);
                } else {
                    v = horner_off(x, c + deg + 1, deg) / (aii + dj[q]);
                }
                q64[p] = v;
                q32[p] = static_cast<float>(v);
            }
        }
    }
}

constexpr int kAsmCap = 4096;  // entries of a workgroup's rows staged through LDS
constexpr int kAsmChunk = 4;   // entries per thread per round

// Rows per workgroup: the most whose mean entries fill at most three rounds of kAsmChunk entries per
// thread, and never so many that the level gives fewer than 512 workgroups (two per CU). A chain of
// FP64 divisions and a gather per entry makes a workgroup latency-bound, so long rows (25-60
// entries on the coarse levels of 3D hierarchies) and small levels want few rows each; with 256 rows
// everywhere such blocks also overflowed the LDS map and ran one thread per row. Measured on the
// hierarchy of 998k tetrahedral cells, us per level with 256 rows and with this rule: 998k rows of
// 5 entries 45 / 46, 499k of 11 42 / 43, 122k of 25 73 / 29, 20k of 42 42 / 13, 3k of 50 49 / 7, 464
// of 46 47 / 6; the whole smoother setup of that hierarchy 2.30 -> 2.13 ms.
inline int asm_rows(int32_t n, int32_t nnz) {
    const int64_t mean = (static_cast<int64_t>(nnz) + n - 1) / n;
    int r = kBlock;
    while (r > 16 && (r * mean > 3 * kAsmChunk * kBlock || static_cast<int64_t>(n) < 512 * r)) r /= 2;
    return r;
}

// A workgroup owns ROWS consecutive rows. ROWS threads first form the rows' coefficients, scale and
// diagonal (the per-row data of Eq. 5) in LDS and the rows' entries are marked with their local
// row index (kBlock / ROWS threads per row); the block's entries are then streamed with unit stride
// (coalesced column, value and output streams), each entry taking its row's data from LDS. The
// arithmetic per entry is the per-row form's (assemble_row), so the values are the same bit for
// bit; a block whose entries overflow the LDS map falls back to one thread per row.
// BLOCKS: block-diagonal level (coefficient row and scale of the row's block, a coefficient
// row < 0 gives zero coefficients); else one coefficient set and scale[0].
template <bool BLOCKS, int ROWS>
__global__ __launch_bounds__(kBlock) void assemble_stream_kernel(
    int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col, const double* __restrict__ val,
    const double* __restrict__ diag, int32_t nblk, const int32_t* __restrict__ off, const double* __restrict__ scale,
    const int32_t* __restrict__ crow, PolyCoeffs pc, const float* __restrict__ coeffs_dev, int32_t stride,
    double* __restrict__ q64, float* __restrict__ q32, double* __restrict__ qd64, float* __restrict__ qd32) {
#pragma clang fp contract(off)
    static_assert(ROWS <= 256 && kBlock % ROWS == 0, "local row indices are stored in 8 bits");
    constexpr int kMark = kBlock / ROWS;  // threads that mark a row's entries
    __shared__ uint8_t rowof[kAsmCap];
    __shared__ double cs[ROWS][2 * 4 + 1];
    __shared__ double srow[ROWS], arow[ROWS];
    const int deg = pc.degree;
    const int t = static_cast<int>(threadIdx.x);
    const int32_t r0 = static_cast<int32_t>(blockIdx.x) * ROWS;
    const int32_t r1 = min(r0 + ROWS, n);
    const int32_t e0 = ptr[r0];
    const int32_t ne = ptr[r1] - e0;
    const bool fits = ne <= kAsmCap;
    const int32_t i = r0 + t;
    const bool own = t < ROWS && i < r1;
    if (fits && r0 + t / kMark < r1) {
        const int32_t m = r0 + t / kMark;
        for (int32_t k = ptr[m] - e0 + t % kMark; k < ptr[m + 1] - e0; k += kMark)
            rowof[k] = static_cast<uint8_t>(t / kMark);
    }
    if (own) {
        int32_t b = 0, r = 0;
        if constexpr (BLOCKS) {
            int32_t lo = 0, hi = nblk - 1;  // block of row i
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) / 2;
                if (off[mid] <= i)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            b = lo;
            r = crow[b];
        }
        for (int k = 0; k < 2 * deg + 1; ++k) {
            if (pc.diag_only && k > deg) {
                cs[t][k] = 0.0;
                continue;
            }
            if constexpr (BLOCKS)
                cs[t][k] = r < 0 ? 0.0
                           : coeffs_dev ? static_cast<double>(coeffs_dev[static_cast<int64_t>(r) * stride + k])
                                        : pc.c[k];
            else
                cs[t][k] = coeffs_dev ? static_cast<double>(coeffs_dev[k]) : pc.c[k];
        }
        srow[t] = scale[b];
        arow[t] = diag[i];
    }
    __syncthreads();
    if (!fits) {
        if (own) assemble_row(i, ptr, col, val, diag, cs[t], deg, srow[t], q64, q32, qd64, qd32);
        return;
    }
    for (int32_t base = 0; base < ne; base += kAsmChunk * kBlock) {
        int32_t j[kAsmChunk];
        double a[kAsmChunk], dj[kAsmChunk];
#pragma unroll
        for (int q = 0; q < kAsmChunk; ++q) {
            const int32_t k = min(base + t + q * kBlock, ne - 1);
            j[q] = col[e0 + k];
            a[q] = val[e0 + k];
        }
#pragma unroll
        for (int q = 0; q < kAsmChunk; ++q) dj[q] = diag[j[q]];
#pragma unroll
        for (int q = 0; q < kAsmChunk; ++q) {
            const int32_t k = base + t + q * kBlock;
            if (k < ne) {
                const int lr = rowof[k];
                const int32_t row = r0 + lr;
                const double x = a[q] / srow[lr];
                double v;
                if (j[q] == row) {
                    v = horner_diag(x, cs[lr], deg) / a[q];
                    qd64[row] = v;
                    qd32[row] = static_cast<float>(v);
                } else {
                    v = horner_off(x, cs[lr] + deg + 1, deg) / (arow[lr] + dj[q]);
                }
                q64[e0 + k] = v;
                q32[e0 + k] = static_cast<float>(v);
            }
        }
    }
}

template <bool BLOCKS, typename... Args>
hipError_t launch_assemble(int32_t n, int32_t nnz, hipStream_t stream, Args... args) {
    const int rows = asm_rows(n, nnz);
    const dim3 grid(static_cast<unsigned>((n + rows - 1) / rows));
    switch (rows) {
#define AMGG_CASE(R)                                                              \
    case R:                                                                       \
        assemble_stream_kernel<BLOCKS, R><<<grid, kBlock, 0, stream>>>(n, args...); \
        break;
        AMGG_CASE(256)
        AMGG_CASE(128)
        AMGG_CASE(64)
        AMGG_CASE(32)
        AMGG_CASE(16)
#undef AMGG_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t assemble_smoother(int32_t n, int32_t nnz, const int32_t* ptr, const int32_t* col, const double* val,
                             const double* diag, const double* scale, const PolyCoeffs& pc,
                             const float* coeffs_dev, double* q64, float* q32, double* qd64, float* qd32,
                             hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    if (pc.degree < 1 || pc.degree > 4) return hipErrorInvalidValue;
    return launch_assemble<false>(n, nnz, stream, ptr, col, val, diag, 1, static_cast<const int32_t*>(nullptr), scale,
                                  static_cast<const int32_t*>(nullptr), pc, coeffs_dev, 0, q64, q32, qd64, qd32);
}

hipError_t assemble_smoother_blocks(int32_t n, int32_t nnz, const int32_t* ptr, const int32_t* col, const double* val,
                                    const double* diag, int32_t nblk, const int32_t* off, const double* scale,
                                    const int32_t* crow, const PolyCoeffs& pc, const float* coeffs_dev,
                                    int32_t stride, double* q64, float* q32, double* qd64, float* qd32,
                                    hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    if (pc.degree < 1 || pc.degree > 4 || nblk < 1) return hipErrorInvalidValue;
    return launch_assemble<true>(n, nnz, stream, ptr, col, val, diag, nblk, off, scale, crow, pc, coeffs_dev, stride,
                                 q64, q32, qd64, qd32);
}

}  // namespace amgg
