// Setup-side kernels: diagonal and off-diagonal scale of each level, the exact transpose
// R = P^T, and the dense coarsest-level factorisation, inverse and per-cycle product.
#include <algorithm>
#include <cmath>
#include <utility>

#include "kernels.hpp"

namespace amgg {

namespace {

inline dim3 grid_for(int64_t n) {
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g < 1) g = 1;
    return dim3(static_cast<unsigned>(g));
}

// Diagonal of every row (bad[0] set where it is missing or not positive) and, per workgroup, the largest
// |off-diagonal| entry (-1: none), in one pass over the rows.
__global__ __launch_bounds__(kBlock) void diag_absmax_kernel(int32_t n, const int32_t* __restrict__ ptr,
                                                            const int32_t* __restrict__ col,
                                                            const double* __restrict__ val, double* __restrict__ diag,
                                                            int32_t* __restrict__ bad, double* __restrict__ partial) {
    __shared__ double red[kBlock];
    double m = -1.0;
    for (int32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        double d = 0.0;
        bool found = false;
        for (int32_t p = ptr[i]; p < ptr[i + 1]; ++p) {
            const double v = val[p];
            if (col[p] == i) {
                d = v;
                found = true;
            } else {
                m = fmax(m, fabs(v));
            }
        }
        diag[i] = d;
        if (!found || !(d > 0.0)) atomicOr(bad, 1);
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kBlock) void absmax_final_kernel(const double* __restrict__ partial, int count,
                                                             double* __restrict__ scale) {
    __shared__ double red[kBlock];
    double m = -1.0;
    for (int k = threadIdx.x; k < count; k += kBlock) m = fmax(m, partial[k]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) scale[0] = red[0] <= 0.0 ? 1.0 : red[0];  // no nonzero off-diagonal: s = 1
}

// --- transpose -----------------------------------------------------------------------
__global__ void count_cols_kernel(int32_t nnz, const int32_t* __restrict__ col, int32_t* __restrict__ cnt) {
    const int32_t p = blockIdx.x * kBlock + threadIdx.x;
    if (p < nnz) atomicAdd(&cnt[col[p] + 1], 1);
}

// In-place inclusive scan of a[1..m] (setup only): the range is cut into at most
// kScanParts contiguous pieces; pass 1 sums each piece, pass 2 scans the piece sums, pass 3
// scans each piece from its offset. Integer sums: the result does not depend on the order.
constexpr int kScanBlock = 1024;  // 16 wavefronts
constexpr int64_t kScanParts = 1024;  // at most ceil(m / kScanBlock) <= m pieces
static_assert(kScanParts <= kScanPartsMax, "pack_columns scratch holds the piece sums");

__device__ int32_t block_inclusive_scan(int32_t v, int32_t* lds, int32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    if (lane == 63) lds[wave] = v;
    __syncthreads();
    if (wave == 0) {
        int32_t w = lane < kScanBlock / 64 ? lds[lane] : 0;
        for (int o = 1; o < kScanBlock / 64; o <<= 1) {
            const int32_t t = __shfl_up(w, o, 64);
            if (lane >= o) w += t;
        }
        if (lane < kScanBlock / 64) lds[lane] = w;
    }
    __syncthreads();
    if (wave > 0) v += lds[wave - 1];
    *total = lds[kScanBlock / 64 - 1];
    __syncthreads();
    return v;
}

__global__ __launch_bounds__(kScanBlock) void scan_reduce_kernel(int32_t m, int32_t piece,
                                                                 const int32_t* __restrict__ a,
                                                                 int32_t* __restrict__ parts) {
    __shared__ int32_t lds[kScanBlock / 64];
    const int64_t lo = 1 + static_cast<int64_t>(blockIdx.x) * piece;
    const int64_t hi = min(lo + piece, static_cast<int64_t>(m) + 1);
    int32_t s = 0;
    for (int64_t k = lo + threadIdx.x; k < hi; k += kScanBlock) s += a[k];
    int32_t total;
    block_inclusive_scan(s, lds, &total);
    if (threadIdx.x == 0) parts[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanBlock) void scan_parts_kernel(int32_t nparts, int32_t* __restrict__ parts) {
    __shared__ int32_t lds[kScanBlock / 64];
    const int32_t v = threadIdx.x < nparts ? parts[threadIdx.x] : 0;
    int32_t total;
    const int32_t incl = block_inclusive_scan(v, lds, &total);
    if (threadIdx.x < nparts) parts[threadIdx.x] = incl - v;  // exclusive
}

__global__ __launch_bounds__(kScanBlock) void scan_apply_kernel(int32_t m, int32_t piece, int32_t* __restrict__ a,
                                                                const int32_t* __restrict__ parts) {
    __shared__ int32_t lds[kScanBlock / 64];
    const int64_t lo = 1 + static_cast<int64_t>(blockIdx.x) * piece;
    const int64_t hi = min(lo + piece, static_cast<int64_t>(m) + 1);
    int32_t carry = parts ? parts[blockIdx.x] : 0;
    for (int64_t base = lo; base < hi; base += kScanBlock) {
        const int64_t k = base + threadIdx.x;
        const int32_t v = k < hi ? a[k] : 0;
        int32_t total;
        const int32_t incl = block_inclusive_scan(v, lds, &total);
        if (k < hi) a[k] = carry + incl;
        carry += total;
    }
}

__global__ void scatter_transpose_kernel(int32_t nf, const int32_t* __restrict__ p_ptr,
                                         const int32_t* __restrict__ p_col, const double* __restrict__ p_val,
                                         int32_t* __restrict__ cursor, int32_t* __restrict__ r_col,
                                         double* __restrict__ r_val) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= nf) return;
    for (int32_t p = p_ptr[i]; p < p_ptr[i + 1]; ++p) {
        const int32_t dst = atomicAdd(&cursor[p_col[p]], 1);
        r_col[dst] = i;
        r_val[dst] = p_val[p];
    }
}

// The scatter order within a row depends on atomics; sorting by column restores the one
// exact transpose. kSortLanes lanes hold a row of up to 4 entries each and put every entry at its rank (the
// row's entries passed by shuffles); a longer row is sorted in place by one lane. With one thread per row
// throughout, the chain of dependent moves took 20 us a level however small; 4 to 7 us here.
constexpr int kSortLanes = 16;

// A row of at most Q kSortLanes entries [lo, hi).
template <int Q>
__device__ __forceinline__ void rank_row(int32_t lo, int32_t hi, int lane, int32_t* __restrict__ r_col,
                                         double* __restrict__ r_val) {
    int32_t key[Q], rank[Q];
    double v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int32_t k = lo + q * kSortLanes + lane;
        key[q] = k < hi ? r_col[k] : INT32_MAX;
        v[q] = k < hi ? r_val[k] : 0.0;
        rank[q] = 0;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int here = min(kSortLanes, hi - lo - q * kSortLanes);
        for (int l = 0; l < here; ++l) {
            const int32_t other = __shfl(key[q], l, kSortLanes);
#pragma unroll
            for (int t = 0; t < Q; ++t)  // equal columns keep their order
                rank[t] += other < key[t] || (other == key[t] && q * kSortLanes + l < t * kSortLanes + lane) ? 1 : 0;
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (lo + q * kSortLanes + lane < hi) {
            r_col[lo + rank[q]] = key[q];
            r_val[lo + rank[q]] = v[q];
        }
}

__global__ __launch_bounds__(kBlock) void sort_rows_kernel(int32_t nc, const int32_t* __restrict__ r_ptr,
                                                          int32_t* __restrict__ r_col, double* __restrict__ r_val) {
    const int32_t c = blockIdx.x * (kBlock / kSortLanes) + threadIdx.x / kSortLanes;
    if (c >= nc) return;
    const int lane = threadIdx.x % kSortLanes;
    const int32_t lo = r_ptr[c], hi = r_ptr[c + 1];
    if (hi - lo <= kSortLanes) return rank_row<1>(lo, hi, lane, r_col, r_val);
    if (hi - lo <= 4 * kSortLanes) return rank_row<4>(lo, hi, lane, r_col, r_val);
    if (lane != 0) return;
    for (int32_t a = lo + 1; a < hi; ++a) {
        const int32_t key = r_col[a];
        const double v = r_val[a];
        int32_t b = a - 1;
        while (b >= lo && r_col[b] > key) {
            r_col[b + 1] = r_col[b];
            r_val[b + 1] = r_val[b];
            --b;
        }
        r_col[b + 1] = key;
        r_val[b + 1] = v;
    }
}

// --- dense coarsest level --------------------------------------------------------------
__global__ void dense_zero_kernel(int64_t total, double* __restrict__ M) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (k < total) M[k] = 0.0;
}

// Matrices of at most kLuRows rows are factorised in panels from column-major storage, larger ones by one
// workgroup from row-major storage.
constexpr int32_t kLuRows = 1024;

// Rows [0, n) of ptr (columns shifted by -col0) into the dense n x n matrix M: entry (i, j) at i si + j sj.
__global__ void dense_scatter_kernel(int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                     const double* __restrict__ val, int32_t col0, int64_t si, int64_t sj,
                                     double* __restrict__ M) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    for (int32_t p = ptr[i]; p < ptr[i + 1]; ++p) M[i * si + (col[p] - col0) * sj] = val[p];
}

// A_L + alpha 1 1^T with alpha = mean(diag)/n (constant null space of all-Neumann problems).
__global__ __launch_bounds__(1024) void dense_rank_one_kernel(int32_t n, double* __restrict__ M) {
    __shared__ double red[1024];
    double s = 0.0;
    for (int32_t i = threadIdx.x; i < n; i += 1024) s += M[static_cast<int64_t>(i) * n + i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double alpha = red[0] / n / n;
    const int64_t total = static_cast<int64_t>(n) * n;
    for (int64_t k = threadIdx.x; k < total; k += 1024) M[k] += alpha;
}

// LU with partial pivoting (largest |pivot|, smallest row index on ties) by one workgroup, for more than
// kLuRows rows; lu_panel_kernel and lu_update_kernel form the same factors.
__global__ __launch_bounds__(1024) void dense_lu_kernel(int32_t n, double* __restrict__ M, int32_t* __restrict__ piv,
                                                        int32_t* __restrict__ bad) {
    __shared__ double sval[1024];
    __shared__ int32_t sidx[1024];
    const int tid = threadIdx.x;
    for (int32_t k = tid; k < n; k += 1024) piv[k] = k;
    __syncthreads();
    for (int32_t k = 0; k < n; ++k) {
        double best = -1.0;
        int32_t bi = n;
        for (int32_t i = k + tid; i < n; i += 1024) {
            const double v = fabs(M[static_cast<int64_t>(i) * n + k]);
            if (v > best) {
                best = v;
                bi = i;
            }
        }
        sval[tid] = best;
        sidx[tid] = bi;
        __syncthreads();
        for (int w = 512; w > 0; w >>= 1) {
            if (tid < w) {
                const double ov = sval[tid + w];
                const int32_t oi = sidx[tid + w];
                if (ov > sval[tid] || (ov == sval[tid] && oi < sidx[tid])) {
                    sval[tid] = ov;
                    sidx[tid] = oi;
                }
            }
            __syncthreads();
        }
        const int32_t p = sidx[0];
        const double pv = sval[0];
        __syncthreads();
        if (!(pv > 0.0)) {
            if (tid == 0) bad[0] = 1;
            return;
        }
        if (p != k)
            for (int32_t j = tid; j < n; j += 1024) {
                const double t = M[static_cast<int64_t>(k) * n + j];
                M[static_cast<int64_t>(k) * n + j] = M[static_cast<int64_t>(p) * n + j];
                M[static_cast<int64_t>(p) * n + j] = t;
            }
        if (tid == 0) piv[k] = p;
        __syncthreads();
        const double pivot = M[static_cast<int64_t>(k) * n + k];
        for (int32_t i = k + 1 + tid; i < n; i += 1024) M[static_cast<int64_t>(i) * n + k] /= pivot;
        __syncthreads();
        const int32_t m = n - k - 1;
        const int64_t cnt = static_cast<int64_t>(m) * m;
        for (int64_t e = tid; e < cnt; e += 1024) {
            const int32_t i = k + 1 + static_cast<int32_t>(e / m);
            const int32_t j = k + 1 + static_cast<int32_t>(e % m);
            M[static_cast<int64_t>(i) * n + j] -= M[static_cast<int64_t>(i) * n + k] * M[static_cast<int64_t>(k) * n + j];
        }
        __syncthreads();
    }
}

// The same factorisation in panels of kLuPanel columns: this kernel factorises one panel, lu_update_kernel
// the rows and columns right of it. A thread owns a row of the matrix and keeps its panel entries in
// registers; rows stay where they are and only their place in the order changes: pos[row] is the row's
// place after the exchanges so far, perm[place] its inverse for the places with a pivot. Every entry
// receives its updates in the order of the unblocked form, so pivots and factors are the same. What bounds
// a column's step is the chain search - pivot row through LDS - division - update behind two
// barriers (1.4 us), where the unblocked form passed the whole trailing matrix through one workgroup's memory
// port. Finalizing one dense matrix of 124 / 250 / 500 / 1000 rows: 0.76 / 3.4 / 21 / 155 ms unblocked with a
// workgroup per column of the inverse, 0.36 / 0.76 / 2.0 / 6.0 ms in panels with a wavefront per
// column.
constexpr int kLuPanel = 32;

// f(0), ..., f(N - 1) with constant arguments (a loop of this length is not unrolled by itself, and the
// row's entries would leave the registers)
template <int... K, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, K...>, F f) {
    (f(std::integral_constant<int, K>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// The wavefront's largest value, in every lane; DPP and lane swaps where shuffles would go through the LDS unit.
template <int CTRL>
__device__ __forceinline__ double dpp_max(double v) {
    const int2 b = __builtin_bit_cast(int2, v);
    const double o = __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, b.x, CTRL, 0xf, 0xf, true),
                                                          __builtin_amdgcn_update_dpp(0, b.y, CTRL, 0xf, 0xf, true)));
    return o > v ? o : v;
}
__device__ __forceinline__ double wave_max(double v) {
    v = dpp_max<0xb1>(v);   // lane ^ 1
    v = dpp_max<0x4e>(v);   // lane ^ 2
    v = dpp_max<0x141>(v);  // mirrored within 8
    v = dpp_max<0x140>(v);  // mirrored within 16
    auto greater = [](auto lo, auto hi) {
        const double x = __builtin_bit_cast(double, make_uint2(lo[0], hi[0]));
        const double y = __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
        return x > y ? x : y;
    };
    uint2 b = __builtin_bit_cast(uint2, v);
    v = greater(__builtin_amdgcn_permlane16_swap(b.x, b.x, false, false),
                __builtin_amdgcn_permlane16_swap(b.y, b.y, false, false));
    b = __builtin_bit_cast(uint2, v);
    return greater(__builtin_amdgcn_permlane32_swap(b.x, b.x, false, false),
                   __builtin_amdgcn_permlane32_swap(b.y, b.y, false, false));
}

__global__ __launch_bounds__(kLuRows) void lu_panel_kernel(int32_t n, int32_t k0, double* __restrict__ M,
                                                          int32_t* __restrict__ pos, int32_t* __restrict__ perm,
                                                          int32_t* __restrict__ bad) {
    struct Cand {
        double v;
        int32_t place, row;
    };
    __shared__ Cand cand[kLuRows / 64];
    __shared__ double prow[kLuPanel];
    if (bad[0]) return;  // an earlier panel met a zero pivot
    const int row = threadIdx.x, waves = blockDim.x / 64;
    const bool live = row < n;
    int32_t place = !live ? -1 : k0 == 0 ? row : pos[row];
    const bool open = place >= k0;  // no pivot row before this panel
    double a[kLuPanel];
#pragma unroll
    for (int c = 0; c < kLuPanel; ++c)
        a[c] = open && k0 + c < n ? M[static_cast<int64_t>(k0 + c) * n + row] : 0.0;
    bool singular = false;
    static_for<kLuPanel>([&](auto kc) {
        constexpr int k = kc;
        const int32_t at = k0 + k;
        if (at >= n || singular) return;
        const double v = place >= at && fabs(a[k]) >= 0.0 ? fabs(a[k]) : -1.0;  // a NaN is no pivot
        const double top = wave_max(v);
        uint64_t tied = top > 0.0 ? __builtin_amdgcn_ballot_w64(v == top) : 0;
        Cand best{top, INT32_MAX, 0};
        for (; tied; tied &= tied - 1) {  // all but always one lane
            const int l = __builtin_ctzll(tied);
            const int32_t pl = __builtin_amdgcn_readlane(place, l);
            if (pl < best.place) best = {top, pl, (row & ~63) + l};
        }
        if ((row & 63) == 0) cand[row / 64] = best;
        __syncthreads();
        best = cand[0];
        for (int w = 1; w < waves; ++w)
            if (cand[w].v > best.v || (cand[w].v == best.v && cand[w].place < best.place)) best = cand[w];
        singular = !(best.v > 0.0);  // the same in every thread
        if (singular) return;
        if (place == at) place = best.place;
        if (row == best.row) {
            place = at;
            perm[at] = row;
#pragma unroll
            for (int c = k; c < kLuPanel; ++c) prow[c] = a[c];
        }
        __syncthreads();
        if (place > at) {
            const double l = a[k] / prow[k];
            a[k] = l;
#pragma unroll
            for (int c = k + 1; c < kLuPanel; ++c) a[c] -= l * prow[c];
        }
    });
    if (singular) {
        if (row == 0) bad[0] = 1;
        return;
    }
    if (!live) return;
    pos[row] = place;
    if (!open) return;
#pragma unroll
    for (int c = 0; c < kLuPanel; ++c)
        if (k0 + c < n) M[static_cast<int64_t>(k0 + c) * n + row] = a[c];
}

// Right of the panel at k0: one workgroup per kLuStrip columns solves them for the panel's pivot rows and updates
// the rows below, every entry's terms in column order.
constexpr int kLuStrip = kBlock / kLuPanel;

__global__ __launch_bounds__(kBlock) void lu_update_kernel(int32_t n, int32_t k0, double* __restrict__ M,
                                                          const int32_t* __restrict__ pos,
                                                          const int32_t* __restrict__ perm,
                                                          const int32_t* __restrict__ bad) {
    __shared__ double Ls[kLuPanel][kLuPanel + 1], Us[kLuPanel][kLuStrip];
    if (bad[0]) return;
    const int tid = threadIdx.x, i = tid / kLuStrip, cc = tid % kLuStrip;
    const int32_t j0 = k0 + kLuPanel + static_cast<int32_t>(blockIdx.x) * kLuStrip;  // a full panel is left of it
    const int32_t wide = min(kLuStrip, n - j0), mine = perm[k0 + i];
    for (int c = cc; c < kLuPanel; c += kLuStrip) Ls[i][c] = M[static_cast<int64_t>(k0 + c) * n + mine];
    double u = cc < wide ? M[static_cast<int64_t>(j0 + cc) * n + mine] : 0.0;
    for (int c = 0; c < kLuPanel; ++c) {
        if (i == c) Us[c][cc] = u;
        __syncthreads();
        if (i > c) u -= Ls[i][c] * Us[c][cc];
    }
    if (cc < wide) M[static_cast<int64_t>(j0 + cc) * n + mine] = u;
    __syncthreads();
    for (int32_t row = tid; row < n; row += kBlock) {
        if (pos[row] < k0 + kLuPanel) continue;
        double m[kLuStrip];
#pragma unroll
        for (int q = 0; q < kLuStrip; ++q) m[q] = q < wide ? M[static_cast<int64_t>(j0 + q) * n + row] : 0.0;
#pragma unroll 8
        for (int c = 0; c < kLuPanel; ++c) {
            const double l = M[static_cast<int64_t>(k0 + c) * n + row];
#pragma unroll
            for (int q = 0; q < kLuStrip; ++q) m[q] -= l * Us[c][q];
        }
#pragma unroll
        for (int q = 0; q < kLuStrip; ++q)
            if (q < wide) M[static_cast<int64_t>(j0 + q) * n + row] = m[q];
    }
}

// Column j of the inverse from the panels' factors: one wavefront per column, the places of x over the lanes'
// registers (lane l holds l, l + 64, ...), so that a step is a lane broadcast and its products, without
// barriers. Q: registers per lane, n <= 64 Q.
template <int Q>
__global__ __launch_bounds__(64) void lu_inverse_kernel(int32_t n, const double* __restrict__ M,
                                                       const int32_t* __restrict__ perm,
                                                       const int32_t* __restrict__ bad, double* __restrict__ inv) {
    if (bad[0]) return;  // factorisation failed: leave the inverse untouched
    const int32_t j = blockIdx.x, lane = threadIdx.x;
    int32_t pr[Q];
    double x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int32_t i = 64 * q + lane;
        pr[q] = i < n ? perm[i] : 0;
        x[q] = i < n && pr[q] == j ? 1.0 : 0.0;
    }
    auto bcast = [](double v, int l) {
        const int2 b = __builtin_bit_cast(int2, v);
        return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(b.x, l), __builtin_amdgcn_readlane(b.y, l)));
    };
#pragma unroll
    for (int q0 = 0; q0 < Q; ++q0) {
        const int kn = min(64, n - 64 * q0);
#pragma unroll 4
        for (int kk = 0; kk < kn; ++kk) {
            const double* Lk = M + static_cast<int64_t>(64 * q0 + kk) * n;
            const double b = bcast(x[q0], kk);
#pragma unroll
            for (int q = q0; q < Q; ++q) {
                const double t = x[q] - Lk[pr[q]] * b;
                if (q > q0 || lane > kk) x[q] = t;
            }
        }
    }
#pragma unroll
    for (int q0 = Q - 1; q0 >= 0; --q0) {
        const int kn = min(64, n - 64 * q0);
#pragma unroll 4
        for (int kk = kn - 1; kk >= 0; --kk) {
            const double* Uk = M + static_cast<int64_t>(64 * q0 + kk) * n;
            const double b = bcast(x[q0] / Uk[pr[q0]], kk);
#pragma unroll
            for (int q = 0; q <= q0; ++q) {
                const double t = x[q] - Uk[pr[q]] * b;
                if (q < q0 || lane < kk) x[q] = t;
            }
            if (lane == kk) x[q0] = b;
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (64 * q + lane < n) inv[static_cast<int64_t>(64 * q + lane) * n + j] = x[q];
}

// Column j of the inverse: solve L U x = Perm e_j, one workgroup per column, x in LDS.
__global__ __launch_bounds__(kBlock) void dense_inverse_cols_kernel(int32_t n, const double* __restrict__ LU,
                                                                   const int32_t* __restrict__ piv,
                                                                   const int32_t* __restrict__ bad,
                                                                   double* __restrict__ inv) {
    extern __shared__ double b[];
    if (bad[0]) return;  // factorisation failed: leave the inverse untouched
    const int32_t j = blockIdx.x;
    const int tid = threadIdx.x;
    for (int32_t i = tid; i < n; i += kBlock) b[i] = (i == j) ? 1.0 : 0.0;
    __syncthreads();
    if (tid == 0)
        for (int32_t k = 0; k < n; ++k) {
            const int32_t p = piv[k];
            if (p != k && p >= 0 && p < n) {
                const double t = b[k];
                b[k] = b[p];
                b[p] = t;
            }
        }
    __syncthreads();
    for (int32_t k = 0; k < n; ++k) {
        const double bk = b[k];
        for (int32_t i = k + 1 + tid; i < n; i += kBlock) b[i] -= LU[static_cast<int64_t>(i) * n + k] * bk;
        __syncthreads();
    }
    for (int32_t k = n - 1; k >= 0; --k) {
        if (tid == 0) b[k] /= LU[static_cast<int64_t>(k) * n + k];
        __syncthreads();
        const double bk = b[k];
        for (int32_t i = tid; i < k; i += kBlock) b[i] -= LU[static_cast<int64_t>(i) * n + k] * bk;
        __syncthreads();
    }
    for (int32_t i = tid; i < n; i += kBlock) inv[static_cast<int64_t>(i) * n + j] = b[i];
}

// y = inv x in FP64, one wavefront per row (coalesced row reads of the inverse).
template <typename T>
__global__ __launch_bounds__(kBlock) void dense_gemv_kernel(int32_t n, const double* __restrict__ inv,
                                                           const T* __restrict__ x, T* __restrict__ y) {
    const int32_t row = blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    if (row < n) {
        const double* a = inv + static_cast<int64_t>(row) * n;
        for (int32_t j = lane; j < n; j += 64) s += a[j] * static_cast<double>(x[j]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (row < n && lane == 0) y[row] = static_cast<T>(s);
}


// --- block-diagonal levels ---------------------------------------------------------------
__device__ __forceinline__ int32_t block_of(int32_t i, int32_t nblk, const int32_t* __restrict__ off) {
    int32_t lo = 0, hi = nblk - 1;  // largest b with off[b] <= i
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) / 2;
        if (off[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// scale[b] = max |a_ij| over the off-diagonal entries of block b's rows (1 if none), one
// workgroup per block; a maximum does not depend on the order.
__global__ __launch_bounds__(kBlock) void block_absmax_kernel(const int32_t* __restrict__ off,
                                                             const int32_t* __restrict__ ptr,
                                                             const int32_t* __restrict__ col,
                                                             const double* __restrict__ val,
                                                             double* __restrict__ scale) {
    __shared__ double red[kBlock];
    const int32_t b = blockIdx.x;
    double m = -1.0;
    for (int32_t i = off[b] + threadIdx.x; i < off[b + 1]; i += kBlock)
        for (int32_t p = ptr[i]; p < ptr[i + 1]; ++p)
            if (col[p] != i) m = fmax(m, fabs(val[p]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) scale[b] = red[0] <= 0.0 ? 1.0 : red[0];
}

// bad = 1 if an entry of P couples fine block b with another coarse block.
__global__ void prolong_blocks_kernel(int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                      int32_t nblk, const int32_t* __restrict__ foff,
                                      const int32_t* __restrict__ coff, int32_t* __restrict__ bad) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int32_t b = block_of(i, nblk, foff);
    for (int32_t p = ptr[i]; p < ptr[i + 1]; ++p)
        if (col[p] < coff[b] || col[p] >= coff[b + 1]) bad[0] = 1;
}

// y = blockdiag(inv_b) x: row i of block b is a dot product with row (i - off[b]) of inv_b,
// summed exactly as dense_gemv_kernel sums a row of a single inverse.
template <typename T>
__global__ __launch_bounds__(kBlock) void block_dense_gemv_kernel(int32_t n, int32_t nblk,
                                                                 const int32_t* __restrict__ off,
                                                                 const int64_t* __restrict__ doff,
                                                                 const double* __restrict__ inv,
                                                                 const T* __restrict__ x, T* __restrict__ y) {
    const int32_t row = blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    if (row < n) {
        const int32_t b = block_of(row, nblk, off);
        const int32_t o = off[b], nb = off[b + 1] - o;
        const double* a = inv + doff[b] + static_cast<int64_t>(row - o) * nb;
        for (int32_t j = lane; j < nb; j += 64) s += a[j] * static_cast<double>(x[o + j]);
    }
#pragma unroll
    for (int off2 = 32; off2 > 0; off2 >>= 1) s += __shfl_xor(s, off2, 64);
    if (row < n && lane == 0) y[row] = static_cast<T>(s);
}

// a[1..m] becomes its inclusive scan; parts: scratch of at least min(m, kScanParts) ints. A few thousand
// values are one workgroup's work: three launches cost more than its few rounds.
void inclusive_scan(int32_t m, int32_t* a, int32_t* parts, hipStream_t stream) {
    if (m <= 4 * kScanBlock) {
        scan_apply_kernel<<<1, kScanBlock, 0, stream>>>(m, m, a, nullptr);
        return;
    }
    const int32_t nparts = static_cast<int32_t>(
        std::min<int64_t>(kScanParts, (static_cast<int64_t>(m) + kScanBlock - 1) / kScanBlock));
    const int32_t piece = static_cast<int32_t>((static_cast<int64_t>(m) + nparts - 1) / nparts);
    scan_reduce_kernel<<<nparts, kScanBlock, 0, stream>>>(m, piece, a, parts);
    scan_parts_kernel<<<1, kScanBlock, 0, stream>>>(nparts, parts);
    scan_apply_kernel<<<nparts, kScanBlock, 0, stream>>>(m, piece, a, parts);
}

// --- halo lists of the fused smoothing kernels -------------------------------------------
// One workgroup per block of `rows` rows. Its distinct outside columns go through a hash table in LDS and
// are sorted there; then every entry finds its slot by bisection and groups of 8 lanes copy the halo
// rows' entries. Without FILL: the block's halo rows and halo entries into hoff[b + 1] and heoff[b + 1], and
// out[0] is set if it has more than kHaloCap rows or kHaloEntCap entries; with FILL the lists
// themselves at the scanned offsets. Forming the list twice is cheaper than keeping it: both passes of
// a level read its pattern from cache. (101k-row triangulation, its levels of 37k rows and less:
// 6.15 ms with copies to the host, sorting there and copies back, 0.15 ms here.)
constexpr int kHaloSlots = 2 * kHaloCap;  // at most kHaloCap + kBlock columns enter the table
static_assert(kHaloCap + kBlock <= kHaloSlots, "an insertion always finds a free slot");

template <bool FILL>
__global__ __launch_bounds__(kBlock) void halo_kernel(int32_t n, int32_t nnz, int rows, const int32_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ col, const double* __restrict__ val,
                                                     const float* __restrict__ val32, HaloOut h,
                                                     int32_t* __restrict__ out) {
    __shared__ int32_t table[kHaloSlots], list[kHaloCap], end[kHaloCap], wsum[kBlock / 64], count, bad;
    const int32_t b = blockIdx.x, tid = threadIdx.x;
    const int32_t r0 = b * rows, r1 = min(r0 + rows, n);
    const int32_t e0 = ptr[r0], e1 = ptr[r1];
    if (FILL && (out[0] != 0 || out[1] > nnz)) return;  // the level has no lists
    for (int i = tid; i < kHaloSlots; i += kBlock) table[i] = -1;
    for (int i = tid; i < kHaloCap; i += kBlock) list[i] = INT32_MAX;
    if (tid == 0) count = bad = 0;
    __syncthreads();
    for (int32_t k = e0 + tid; k < e1; k += kBlock) {
        const int32_t j = col[k];
        if (j >= r0 && j < r1) continue;
        if (j < 0 || j >= n) {
            bad = 1;
            continue;
        }
        if (__hip_atomic_load(&count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kHaloCap) break;
        for (uint32_t s = static_cast<uint32_t>(j) * 2654435761u >> 8;; ++s) {
            const int32_t was = atomicCAS(&table[s % kHaloSlots], -1, j);
            if (was == j) break;
            if (was == -1) {
                const int32_t at = atomicAdd(&count, 1);
                if (at < kHaloCap) list[at] = j;
                break;
            }
        }
    }
    __syncthreads();
    const int32_t m = count;
    if (m > kHaloCap || bad) {
        if (tid == 0) {
            out[0] = 1;
            if (!FILL) h.hoff[b + 1] = h.heoff[b + 1] = 0;
        }
        return;
    }
    int32_t span = 2;
    while (span < m) span *= 2;
    for (int32_t size = 2; size <= span; size *= 2)  // bitonic
        for (int32_t step = size / 2; step > 0; step /= 2) {
            for (int32_t i = tid; i < span / 2; i += kBlock) {
                const int32_t lo = 2 * i - (i & (step - 1)), hi = lo + step;
                const int32_t x = list[lo], y = list[hi];
                if ((x > y) == ((lo & size) == 0)) {
                    list[lo] = y;
                    list[hi] = x;
                }
            }
            __syncthreads();
        }
    // ends of the halo rows' entries: every thread its four rows, the threads by a scan
    constexpr int kPer = kHaloCap / kBlock;
    int32_t len[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int32_t i = tid * kPer + q;
        len[q] = i < m ? ptr[list[i] + 1] - ptr[list[i]] : 0;
        sum += len[q];
    }
    int32_t incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, 64);
        if ((tid & 63) >= o) incl += t;
    }
    if ((tid & 63) == 63) wsum[tid / 64] = incl;
    __syncthreads();
    for (int w = 0; w < tid / 64; ++w) incl += wsum[w];
    int32_t at = incl - sum;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        at += len[q];
        end[tid * kPer + q] = at;
    }
    __syncthreads();
    const int32_t ents = end[kHaloCap - 1];
    if constexpr (!FILL) {
        if (tid == 0) {
            if (ents > kHaloEntCap) out[0] = 1;
            h.hoff[b + 1] = m;
            h.heoff[b + 1] = ents > kHaloEntCap ? 0 : ents;
            if (b == 0) h.hoff[0] = h.heoff[0] = 0;
        }
    } else {
        const int32_t o = h.hoff[b], eo = h.heoff[b];
        for (int32_t i = tid; i < m; i += kBlock) {
            h.halo[o + i] = list[i];
            h.hend[o + i] = static_cast<uint16_t>(end[i]);
        }
        for (int32_t k = e0 + tid; k < e1; k += kBlock) {
            const int32_t j = col[k];
            int32_t slot = j - r0;
            if (j < r0 || j >= r1) {
                int32_t lo = 0, hi = m;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) / 2;
                    if (list[mid] < j)
                        lo = mid + 1;
                    else
                        hi = mid;
                }
                slot = rows + lo;
            }
            h.hloc[k] = static_cast<uint16_t>(slot);
        }
        for (int32_t i = tid / 8; i < m; i += kBlock / 8) {
            const int32_t first = ptr[list[i]], dst = eo + (i > 0 ? end[i - 1] : 0), cnt = ptr[list[i] + 1] - first;
            for (int32_t q = tid % 8; q < cnt; q += 8) {
                h.hent[dst + q] = first + q;
                h.hcol[dst + q] = col[first + q];
                h.ha64[dst + q] = val[first + q];
                h.ha32[dst + q] = val32[first + q];
            }
        }
    }
}

// Inclusive scans of hoff[1..nb] and heoff[1..nb]; *total receives the latter's last value. (65536 rows
// of at most kHaloEntCap entries each stay below 2^31.)
static_assert(static_cast<int64_t>(kFuseMaxRows) * kHaloEntCap < INT32_MAX, "the totals fit");
__global__ __launch_bounds__(kScanBlock) void halo_scan_kernel(int32_t nb, int32_t* __restrict__ hoff,
                                                              int32_t* __restrict__ heoff,
                                                              int32_t* __restrict__ total) {
    __shared__ int32_t lds[kScanBlock / 64];
    int32_t c0 = 0, c1 = 0;
    for (int32_t base = 1; base <= nb; base += kScanBlock) {
        const int32_t k = base + threadIdx.x;
        int32_t t0, t1;
        const int32_t s0 = block_inclusive_scan(k <= nb ? hoff[k] : 0, lds, &t0);
        const int32_t s1 = block_inclusive_scan(k <= nb ? heoff[k] : 0, lds, &t1);
        if (k <= nb) {
            hoff[k] = c0 + s0;
            heoff[k] = c1 + s1;
        }
        c0 += t0;
        c1 += t1;
    }
    if (threadIdx.x == 0) *total = c1;
}

}  // namespace

hipError_t diag_and_scale(int32_t n, const int32_t* ptr, const int32_t* col, const double* val, double* diag,
                          int32_t* bad, double* partial, double* scale, hipStream_t stream) {
    const int blocks = n <= 0 ? 0 : std::min<int>(kReduceBlocks, (n + kBlock - 1) / kBlock);
    if (blocks > 0) diag_absmax_kernel<<<blocks, kBlock, 0, stream>>>(n, ptr, col, val, diag, bad, partial);
    absmax_final_kernel<<<1, kBlock, 0, stream>>>(partial, blocks, scale);
    return hipGetLastError();
}

// --- packed columns --------------------------------------------------------------------
// One workgroup per row block: the base column (the middle entry of the block's middle row,
// less 32767, at least 0: with sorted columns that entry sits among the row's near neighbours,
// the diagonal for a level matrix, so the 16-bit window is centred on the block's own
// neighbourhood), every entry's offset from it, and the count of far entries into cnt[b + 1]
// (none for a block beyond the product buffer, whose rows read the plain columns).
__global__ __launch_bounds__(kBlock) void pack_count_kernel(int32_t nrows, int rows, const int32_t* __restrict__ ptr,
                                                           const int32_t* __restrict__ col, uint16_t* __restrict__ off,
                                                           int32_t* __restrict__ base, int32_t* __restrict__ cnt) {
    __shared__ int32_t nfar;
    const int32_t b = blockIdx.x;
    const int32_t r0 = b * rows, r1 = min(r0 + rows, nrows);
    const int32_t e0 = ptr[r0], ne = ptr[r1] - e0;
    const int32_t rm = r0 + (r1 - r0) / 2;
    const int32_t mb = ptr[rm], me = ptr[rm + 1];
    const int32_t anchor = me > mb ? col[mb + (me - mb) / 2] : (ne > 0 ? col[e0 + ne / 2] : 0);
    const int32_t bs = max(0, anchor - 32767);
    if (threadIdx.x == 0) nfar = 0;
    __syncthreads();
    int32_t mine = 0;
    for (int32_t k = threadIdx.x; k < ne; k += kBlock) {
        const int64_t o = static_cast<int64_t>(col[e0 + k]) - bs;
        const bool near = o >= 0 && o < kFarCol;
        off[e0 + k] = near ? static_cast<uint16_t>(o) : kFarCol;
        mine += near ? 0 : 1;
    }
    if (mine) atomicAdd(&nfar, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        base[b] = bs;
        cnt[b + 1] = ne <= kStreamCap ? nfar : 0;
        if (b == 0) cnt[0] = 0;
    }
}

// Far entries of each block at foff[b]..: entry index within the block and full column, unless there are
// more than cap of them (total receives their number). Their order within a block is immaterial (each
// one is written to its own product slot).
__global__ __launch_bounds__(kBlock) void pack_far_kernel(int32_t nrows, int rows, const int32_t* __restrict__ ptr,
                                                         const int32_t* __restrict__ col,
                                                         const uint16_t* __restrict__ off,
                                                         const int32_t* __restrict__ foff,
                                                         uint16_t* __restrict__ fslot, int32_t* __restrict__ fcol,
                                                         int64_t cap, int32_t* __restrict__ total) {
    __shared__ int32_t pos;
    const int32_t b = blockIdx.x;
    if (b == 0 && threadIdx.x == 0) *total = foff[gridDim.x];
    if (foff[gridDim.x] > cap) return;
    const int32_t r0 = b * rows, r1 = min(r0 + rows, nrows);
    const int32_t e0 = ptr[r0], ne = ptr[r1] - e0;
    if (ne > kStreamCap || foff[b + 1] == foff[b]) return;  // uniform over the workgroup
    const int32_t f0 = foff[b];
    if (threadIdx.x == 0) pos = 0;
    __syncthreads();
    for (int32_t k = threadIdx.x; k < ne; k += kBlock)
        if (off[e0 + k] == kFarCol) {
            const int32_t j = f0 + atomicAdd(&pos, 1);
            fslot[j] = static_cast<uint16_t>(k);
            fcol[j] = col[e0 + k];
        }
}

hipError_t pack_columns(int32_t nrows, int32_t nnz, const int32_t* ptr, const int32_t* col, int rows, uint16_t* off,
                        int32_t* base, int32_t* foff, uint16_t* fslot, int32_t* fcol, int64_t cap, int32_t* parts,
                        int32_t* nfar, hipStream_t stream) {
    if (nrows <= 0 || nnz <= 0 || rows <= 0) return hipSuccess;
    const int32_t nb = (nrows + rows - 1) / rows;
    pack_count_kernel<<<nb, kBlock, 0, stream>>>(nrows, rows, ptr, col, off, base, foff);
    inclusive_scan(nb, foff, parts, stream);  // foff[b] = far entries before block b
    pack_far_kernel<<<nb, kBlock, 0, stream>>>(nrows, rows, ptr, col, off, foff, fslot, fcol, cap, nfar);
    return hipGetLastError();
}

hipError_t halo_lists(int32_t n, int32_t nnz, const int32_t* ptr, const int32_t* col, const double* val,
                      const float* val32, int rows, const HaloOut& h, int32_t* out, hipStream_t stream) {
    if (n <= 0 || rows <= 0) return hipErrorInvalidValue;
    const int32_t nb = (n + rows - 1) / rows;
    halo_kernel<false><<<nb, kBlock, 0, stream>>>(n, nnz, rows, ptr, col, val, val32, h, out);
    halo_scan_kernel<<<1, kScanBlock, 0, stream>>>(nb, h.hoff, h.heoff, out + 1);
    halo_kernel<true><<<nb, kBlock, 0, stream>>>(n, nnz, rows, ptr, col, val, val32, h, out);
    return hipGetLastError();
}

hipError_t transpose_csr(int32_t nf, int32_t nc, int32_t nnz, const int32_t* p_ptr, const int32_t* p_col,
                         const double* p_val, int32_t* r_ptr, int32_t* r_col, double* r_val, int32_t* cursor,
                         hipStream_t stream) {
    hipError_t e = vec_zero_bytes(r_ptr, sizeof(int32_t) * (nc + 1), stream);
    if (e != hipSuccess) return e;
    if (nnz > 0) count_cols_kernel<<<grid_for(nnz), kBlock, 0, stream>>>(nnz, p_col, r_ptr);
    inclusive_scan(nc, r_ptr, cursor, stream);  // piece sums live in `cursor`, which is free until the scatter below
    if ((e = vec_copy<int32_t>(nc, r_ptr, cursor, stream)) != hipSuccess) return e;
    scatter_transpose_kernel<<<grid_for(nf), kBlock, 0, stream>>>(nf, p_ptr, p_col, p_val, cursor, r_col, r_val);
    const int rows = kBlock / kSortLanes;
    if (nc > 0) sort_rows_kernel<<<(nc + rows - 1) / rows, kBlock, 0, stream>>>(nc, r_ptr, r_col, r_val);
    return hipGetLastError();
}

hipError_t dense_from_csr(int32_t n, const int32_t* ptr, const int32_t* col, const double* val, double* M,
                          int singular, hipStream_t stream, int32_t col0) {
    const int64_t total = static_cast<int64_t>(n) * n;
    dense_zero_kernel<<<grid_for(total), kBlock, 0, stream>>>(total, M);
    const bool by_column = n <= kLuRows;
    dense_scatter_kernel<<<grid_for(n), kBlock, 0, stream>>>(n, ptr, col, val, col0, by_column ? 1 : n,
                                                            by_column ? n : 1, M);
    if (singular) dense_rank_one_kernel<<<1, 1024, 0, stream>>>(n, M);
    return hipGetLastError();
}

hipError_t dense_lu_inverse(int32_t n, double* M, int32_t* piv, double* inv, int32_t* bad, hipStream_t stream) {
    if (n > kLuRows) {
        dense_lu_kernel<<<1, 1024, 0, stream>>>(n, M, piv, bad);
        dense_inverse_cols_kernel<<<n, kBlock, sizeof(double) * n, stream>>>(n, M, piv, bad, inv);
        return hipGetLastError();
    }
    int32_t *perm = piv, *pos = piv + n;
    for (int32_t k0 = 0; k0 < n; k0 += kLuPanel) {
        lu_panel_kernel<<<1, (n + 63) / 64 * 64, 0, stream>>>(n, k0, M, pos, perm, bad);
        const int32_t right = n - k0 - kLuPanel;
        if (right > 0)
            lu_update_kernel<<<(right + kLuStrip - 1) / kLuStrip, kBlock, 0, stream>>>(n, k0, M, pos, perm, bad);
    }
    auto inverse = n <= 64 ? lu_inverse_kernel<1> : n <= 128 ? lu_inverse_kernel<2> : n <= 256 ? lu_inverse_kernel<4>
                 : n <= 512 ? lu_inverse_kernel<8> : lu_inverse_kernel<16>;
    inverse<<<n, 64, 0, stream>>>(n, M, perm, bad, inv);
    return hipGetLastError();
}

template <typename T>
hipError_t dense_gemv(int32_t n, const double* inv, const T* x, T* y, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>((n + kBlock / 64 - 1) / (kBlock / 64)));
    return launch_kernel(dense_gemv_kernel<T>, grid, dim3(kBlock), stream, n, inv, x, y);
}
template hipError_t dense_gemv<float>(int32_t, const double*, const float*, float*, hipStream_t);
template hipError_t dense_gemv<double>(int32_t, const double*, const double*, double*, hipStream_t);

hipError_t block_absmax(int32_t nblk, const int32_t* off, const int32_t* ptr, const int32_t* col, const double* val,
                        double* scale, hipStream_t stream) {
    if (nblk <= 0) return hipSuccess;
    block_absmax_kernel<<<nblk, kBlock, 0, stream>>>(off, ptr, col, val, scale);
    return hipGetLastError();
}

hipError_t prolong_blocks_check(int32_t n, const int32_t* ptr, const int32_t* col, int32_t nblk, const int32_t* foff,
                                const int32_t* coff, int32_t* bad, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    prolong_blocks_kernel<<<grid_for(n), kBlock, 0, stream>>>(n, ptr, col, nblk, foff, coff, bad);
    return hipGetLastError();
}

template <typename T>
hipError_t block_dense_gemv(int32_t n, int32_t nblk, const int32_t* off, const int64_t* doff, const double* inv,
                            const T* x, T* y, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>((n + kBlock / 64 - 1) / (kBlock / 64)));
    return launch_kernel(block_dense_gemv_kernel<T>, grid, dim3(kBlock), stream, n, nblk, off, doff, inv, x, y);
}
template hipError_t block_dense_gemv<float>(int32_t, int32_t, const int32_t*, const int64_t*, const double*,
                                            const float*, float*, hipStream_t);
template hipError_t block_dense_gemv<double>(int32_t, int32_t, const int32_t*, const int64_t*, const double*,
                                             const double*, double*, hipStream_t);

}  // namespace amgg
