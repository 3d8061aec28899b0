// Two passes of a V-cycle level in one kernel, for levels so small that a pass is the latency of its
// dependent loads and of its launch rather than the bytes it moves:
//   down:  f_c = R (f - A u)            (residual and restriction)
//   up:    z = u + P e,  y = z + d (f - A z)   (prolongation, correction and a diagonal smoothing step)
// What the first pass would hand to the second is formed again by every thread that needs it (a
// residual by the 1.9 coarse rows that restrict it, a corrected unknown by its 5-13 neighbours): on
// these levels the cache serves the extra reads, and a kernel has three dependent loads where two
// passes have six and a launch between them. The matrices are read from rows padded to a common
// width, so that a row's place needs no row pointer.
// This file is built with -ffp-contract=off and every row is summed from left to right, so the results
// are bitwise those of the separate passes.
#include <type_traits>

#include "kernels.hpp"

namespace amgg {

namespace {

// Padded copy of a CSR matrix: row i's entries at [i w, i w + w), the rest with column -1.
__global__ __launch_bounds__(kBlock) void pad_rows_kernel(int32_t n, int w, const int32_t* __restrict__ ptr,
                                                         const int32_t* __restrict__ col,
                                                         const double* __restrict__ val, int32_t* __restrict__ pcol,
                                                         double* __restrict__ p64, float* __restrict__ p32) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (t >= static_cast<int64_t>(n) * w) return;
    const int32_t i = static_cast<int32_t>(t / w), k = static_cast<int32_t>(t % w);
    const int32_t b = ptr[i], len = ptr[i + 1] - b;
    const bool in = k < len;
    const double v = in ? val[b + k] : 0.0;
    pcol[t] = in ? col[b + k] : -1;
    p64[t] = v;
    p32[t] = static_cast<float>(v);
}

// Four neighbouring values of a padded row (16-byte loads: w is a multiple of 4, arrays are aligned)
template <typename T>
__device__ __forceinline__ void load4(const T* __restrict__ p, T (&v)[4]) {
    if constexpr (sizeof(T) == 4) {
        const int4 a = *reinterpret_cast<const int4*>(p);
        v[0] = __builtin_bit_cast(T, a.x);
        v[1] = __builtin_bit_cast(T, a.y);
        v[2] = __builtin_bit_cast(T, a.z);
        v[3] = __builtin_bit_cast(T, a.w);
    } else {
        const double2 a = reinterpret_cast<const double2*>(p)[0], b = reinterpret_cast<const double2*>(p)[1];
        v[0] = a.x;
        v[1] = a.y;
        v[2] = b.x;
        v[3] = b.y;
    }
}

// Lane Q's value of every four lanes.
template <int Q, typename T>
__device__ __forceinline__ T quad_bcast(T v) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), Q * 0x55, 0xf, 0xf, true));
    } else {
        const int2 w = __builtin_bit_cast(int2, v);
        return __builtin_bit_cast(T, make_int2(__builtin_amdgcn_update_dpp(0, w.x, Q * 0x55, 0xf, 0xf, true),
                                               __builtin_amdgcn_update_dpp(0, w.y, Q * 0x55, 0xf, 0xf, true)));
    }
}

// 32 threads per coarse row: four threads per entry of its row of R, which form the entry's residual
// together (thread q holds entries 4 q .. 4 q + 3 of every 16 of the row of A; the running sum passes
// from thread to thread, so that it is the row's sum from left to right). Rows of R of up to 8 ER
// entries, of A of up to 16 RA. All loads of a stage are issued together.
constexpr int kDownRows = kBlock / 32;
template <typename T, int ER, int RA>
__global__ __launch_bounds__(kBlock) void resid_restrict_kernel(int32_t nc, PadView<T> R, PadView<T> A,
                                                               const T* __restrict__ u, const T* __restrict__ f,
                                                               T* __restrict__ fc, const T* __restrict__ dc,
                                                               T* __restrict__ uc) {
    __shared__ T prod[kDownRows][8 * ER];
    const int lr = threadIdx.x / 32, k = threadIdx.x % 32 / 4, q = threadIdx.x % 4;
    const int32_t row = blockIdx.x * kDownRows + lr;
    int32_t i[ER];
    T rv[ER];
    T dr = T(0);
#pragma unroll
    for (int m = 0; m < ER; ++m) {
        i[m] = -1;
        rv[m] = T(0);
        const int e = k + 8 * m;
        if (row < nc && e < R.w) {
            i[m] = R.col[row * R.w + e];
            rv[m] = R.val[row * R.w + e];
        }
    }
    if (dc && row < nc) dr = dc[row];
    int32_t c[ER][RA][4];
    T v[ER][RA][4], g[ER][RA][4], fi[ER];
#pragma unroll
    for (int m = 0; m < ER; ++m) {
        const int32_t r = max(i[m], 0);
        fi[m] = f[r];
#pragma unroll
        for (int a = 0; a < RA; ++a) {
            const int at = r * A.w + min(16 * a + 4 * q, A.w - 4);
            load4<int32_t>(A.col + at, c[m][a]);
            load4<T>(A.val + at, v[m][a]);
        }
    }
#pragma unroll
    for (int m = 0; m < ER; ++m)
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e) g[m][a][e] = u[max(c[m][a][e], 0)];
#pragma unroll
    for (int m = 0; m < ER; ++m) {
        T s = T(0);
#pragma unroll
        for (int a = 0; a < RA; ++a) {
            auto step = [&](auto from) {
                T t = s;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (16 * a + 4 * q < A.w && c[m][a][e] >= 0) t += v[m][a][e] * g[m][a][e];
                s = quad_bcast<decltype(from)::value>(t);
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        }
        if (q == 0) prod[lr][k + 8 * m] = rv[m] * (fi[m] - s);
    }
    int len = 0;  // entries of the coarse row (they come first in it)
#pragma unroll
    for (int m = 0; m < ER; ++m)
        len += __popc(static_cast<unsigned int>(__builtin_amdgcn_ballot_w64(i[m] >= 0) >> (threadIdx.x & 32))) / 4;
    __syncthreads();
    if (threadIdx.x % 32 == 0 && row < nc) {
        T s = T(0);
        for (int e = 0; e < len; ++e) s += prod[lr][e];
        fc[row] = s;
        if (dc) uc[row] = dr * s;
    }
}

// TA threads per fine row, EA entries of its row of A each (entry k + TA m): each forms the corrected
// unknown at its entries' columns.
template <typename T, int TA, int EA>
__global__ __launch_bounds__(kBlock) void prolong_jacobi_kernel(int32_t n, PadView<T> A, PadView<T> P,
                                                               const T* __restrict__ e, const T* __restrict__ u,
                                                               const T* __restrict__ f, const T* __restrict__ d,
                                                               T* __restrict__ y) {
    constexpr int kRows = kBlock / TA;
    __shared__ T prod[kRows][TA * EA];
    __shared__ T own[kRows];
    const int lr = threadIdx.x / TA, k = threadIdx.x % TA;
    const int32_t row = blockIdx.x * kRows + lr;
    int32_t j[EA];
    T a[EA], z[EA];
    T fr = T(0), dr = T(0);
#pragma unroll
    for (int m = 0; m < EA; ++m) {
        j[m] = -1;
        a[m] = T(0);
        if (row < n && k + TA * m < A.w) {
            j[m] = A.col[row * A.w + k + TA * m];
            a[m] = A.val[row * A.w + k + TA * m];
        }
    }
    if (k == 0 && row < n) {
        fr = f[row];
        dr = d[row];
    }
#pragma unroll
    for (int m = 0; m < EA; ++m) z[m] = u[max(j[m], 0)];
    {
        T s[EA];
#pragma unroll
        for (int m = 0; m < EA; ++m) s[m] = T(0);
        for (int p = 0; p < P.w; p += 4) {
            int32_t c[EA][4];
            T v[EA][4], g[EA][4];
#pragma unroll
            for (int m = 0; m < EA; ++m) {
                load4<int32_t>(P.col + max(j[m], 0) * P.w + p, c[m]);
                load4<T>(P.val + max(j[m], 0) * P.w + p, v[m]);
            }
#pragma unroll
            for (int m = 0; m < EA; ++m)
#pragma unroll
                for (int q = 0; q < 4; ++q) g[m][q] = e[max(c[m][q], 0)];
#pragma unroll
            for (int m = 0; m < EA; ++m)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (c[m][q] >= 0) s[m] += v[m][q] * g[m][q];
        }
#pragma unroll
        for (int m = 0; m < EA; ++m) z[m] = z[m] + s[m];
    }
    int len = 0;  // entries of the row (they come first in it)
#pragma unroll
    for (int m = 0; m < EA; ++m) {
        if (j[m] >= 0) prod[lr][k + TA * m] = a[m] * z[m];
        if (j[m] >= 0 && j[m] == row) own[lr] = z[m];
        len += __popcll((__builtin_amdgcn_ballot_w64(j[m] >= 0) >> (threadIdx.x & 63 & ~(TA - 1))) & ((1ull << TA) - 1));
    }
    __syncthreads();
    if (k == 0 && row < n) {
        T s = T(0);
        for (int q = 0; q < len; ++q) s += prod[lr][q];
        y[row] = own[lr] + dr * (fr - s);
    }
}

inline dim3 rows_grid(int32_t n, int per) { return dim3(static_cast<unsigned>((n + per - 1) / per)); }

}  // namespace

hipError_t pad_rows(int32_t n, int w, const int32_t* ptr, const int32_t* col, const double* val, int32_t* pcol,
                    double* p64, float* p32, hipStream_t stream) {
    const int64_t t = static_cast<int64_t>(n) * w;
    if (t <= 0) return hipSuccess;
    pad_rows_kernel<<<static_cast<unsigned>((t + kBlock - 1) / kBlock), kBlock, 0, stream>>>(n, w, ptr, col, val, pcol,
                                                                                            p64, p32);
    return hipGetLastError();
}

template <typename T>
hipError_t resid_restrict(int32_t nc, const PadView<T>& R, const PadView<T>& A, const T* u, const T* f, T* fc,
                          const T* dc, T* uc, hipStream_t stream) {
    if (R.w < 4 || R.w > kPairMaxWidthR || A.w < 4 || A.w > kPairMaxWidthA || (dc == nullptr) != (uc == nullptr))
        return hipErrorInvalidValue;
#define AMGG_CASE(ER, RA)                                                                                        \
    if (R.w <= 8 * ER && A.w <= 16 * RA)                                                                         \
        return launch_kernel(resid_restrict_kernel<T, ER, RA>, rows_grid(nc, kDownRows), dim3(kBlock), stream, nc, R, \
                             A, u, f, fc, dc, uc);
    AMGG_CASE(1, 1)
    AMGG_CASE(2, 1)
    AMGG_CASE(4, 1)
    AMGG_CASE(1, 2)
    AMGG_CASE(2, 2)
    AMGG_CASE(4, 2)
    AMGG_CASE(1, 4)
    AMGG_CASE(2, 4)
    AMGG_CASE(4, 4)
#undef AMGG_CASE
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t prolong_jacobi(int32_t n, const PadView<T>& A, const PadView<T>& P, const T* e, const T* u, const T* f,
                          const T* d, T* y, hipStream_t stream) {
    if (A.w < 4 || A.w > kPairMaxWidthA || P.w < 4) return hipErrorInvalidValue;
#define AMGG_CASE(TA, EA)                                                                                         \
    if (A.w <= TA * EA)                                                                                           \
        return launch_kernel(prolong_jacobi_kernel<T, TA, EA>, rows_grid(n, kBlock / TA), dim3(kBlock), stream, n, A, \
                             P, e, u, f, d, y);
    AMGG_CASE(8, 1)
    AMGG_CASE(16, 1)
    AMGG_CASE(16, 2)
    AMGG_CASE(16, 4)
#undef AMGG_CASE
    return hipErrorInvalidValue;
}

#define AMGG_INST(T)                                                                                               \
    template hipError_t resid_restrict<T>(int32_t, const PadView<T>&, const PadView<T>&, const T*, const T*, T*,   \
                                          const T*, T*, hipStream_t);                                              \
    template hipError_t prolong_jacobi<T>(int32_t, const PadView<T>&, const PadView<T>&, const T*, const T*,       \
                                          const T*, const T*, T*, hipStream_t);
AMGG_INST(float)
AMGG_INST(double)
#undef AMGG_INST

}  // namespace amgg
