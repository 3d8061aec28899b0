// Device setup of one level (paper Sec. 2.2; Sec. 4: classical Ruge-Stueben, strength threshold
// theta; Alg. 1, step 2), bitwise equal to the host RS setup: strength of connection, direct
// interpolation from a given C/F split (the split itself, a sequential greedy, stays on the
// host) and the Galerkin product A_c = R (A P) with R = P^T.
//
// A sparse product C = L * M is formed row by row in LDS (one kernel counts the entries of each row, a second
// fills them). A group of 8 to 64 threads holds row i of C in a hash table, takes the entries L_ij in
// ascending column order and adds L_ij M_jk for all k of row j at once, every entry starting
// from 0.0, with product and sum rounded separately; the columns are then ranked. A row of more than 1024
// products is a workgroup's, which sorts the products by column and adds each column's in the same
// order. That is the row-by-row accumulation of the host product, so the values are the host's bit for
// bit. Rows are served by the size their product count needs, each class by a launch of its own.
// Rows of more than kRowMax products (a hub row), more than 2^31 - 1 products in all, or a bound on the
// expansion asked for by the caller take the expanding form:
//   symbolic  every product L_ij M_jk is expanded to a key (row i, column k); one radix sort
//             of the keys and a unique pass give C's pattern (rows in order, columns
//             ascending) without any floating point;
//   numeric   one thread per entry c_ik walks row i of L in ascending column order and adds
//             L_ij M_jk for every j whose row of M holds column k (binary search).
// Its numeric order is the same, so the result does not depend on the form, nor on how the symbolic
// phase orders or batches its work (row chunks that bound the temporary memory).
// Finest product of 623k tetrahedral cells (A 3.1M entries, P 1.5M): 2.05 ms expanding, 0.61 row-wise.
// This file is compiled with -ffp-contract=off: no product may be fused into its sum.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "amggnn.h"
#include "errors.hpp"
#include "kernels.hpp"

namespace amgg {
int hip_fail(hipError_t e, const char* where);
}

using namespace amgg;

namespace {

constexpr int kThreads = 256;

inline unsigned blocks_for(int64_t n) { return static_cast<unsigned>((n + kThreads - 1) / kThreads); }

// One thread per item; nothing is launched for zero items.
template <typename... KArgs, typename... Args>
void launch(void (*kernel)(KArgs...), int64_t items, hipStream_t st, Args... args) {
    if (items > 0)
        hipLaunchKernelGGL(kernel, dim3(blocks_for(items)), dim3(kThreads), 0, st, static_cast<KArgs>(args)...);
}

inline int bit_width(uint64_t v) {
    int b = 0;
    while (v) {
        ++b;
        v >>= 1;
    }
    return b;
}

// bad = 1 unless rows [0, n) form a CSR pattern with nnz entries and strictly ascending
// columns in [0, ncols); `bad` must be 0 on entry.
__global__ void validate_csr_kernel(int32_t n, int32_t ncols, int32_t nnz, const int32_t* __restrict__ ptr,
                                    const int32_t* __restrict__ col, int32_t* __restrict__ bad) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int32_t lo = ptr[i], hi = ptr[i + 1];
    bool ok = lo >= 0 && hi >= lo && hi <= nnz && (i > 0 || lo == 0) && (i < n - 1 || hi == nnz);
    for (int32_t p = lo; ok && p < hi; ++p) {
        const int32_t c = col[p];
        ok = c >= 0 && c < ncols && (p == lo || c > col[p - 1]);
    }
    if (!ok) *bad = 1;
}

// row[p] = i for every entry p of row i.
__global__ void row_index_kernel(int32_t n, const int32_t* __restrict__ ptr, int32_t* __restrict__ row) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    for (int32_t p = ptr[i]; p < ptr[i + 1]; ++p) row[p] = i;
}

// cnt[p] = length of the row of M that L's entry p selects; cnt[nnz_l] = 0 (scan sentinel).
__global__ void product_count_kernel(int32_t nnz_l, const int32_t* __restrict__ lcol,
                                     const int32_t* __restrict__ mptr, int64_t* __restrict__ cnt) {
    const int32_t p = blockIdx.x * kThreads + threadIdx.x;
    if (p > nnz_l) return;
    int64_t c = 0;
    if (p < nnz_l) {
        const int32_t j = lcol[p];
        c = mptr[j + 1] - mptr[j];
    }
    cnt[p] = c;
}

// Row chunk boundaries: bounds[m] = the last row r with (products before r) <= m * budget;
// bounds[0] = 0, bounds[m_count] = n. boff[m] = products before bounds[m].
__global__ void chunk_bounds_kernel(int32_t n, const int32_t* __restrict__ lptr, const int64_t* __restrict__ loff,
                                    int64_t budget, int32_t m_count, int32_t* __restrict__ bounds,
                                    int64_t* __restrict__ boff) {
    const int32_t m = blockIdx.x * kThreads + threadIdx.x;
    if (m > m_count) return;
    int32_t r;
    if (m == 0) {
        r = 0;
    } else if (m == m_count) {
        r = n;
    } else {
        const int64_t target = budget * m;
        int32_t lo = 0, hi = n;  // invariant: poff(lo) <= target; answer in [lo, hi]
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo + 1) / 2;
            if (loff[lptr[mid]] <= target)
                lo = mid;
            else
                hi = mid - 1;
        }
        r = lo;
    }
    bounds[m] = r;
    boff[m] = loff[lptr[r]];
}

// Keys of the products of L's entries [p0, p1): (row - r0) << kb | column of M.
__global__ void expand_kernel(int32_t p0, int32_t p1, const int32_t* __restrict__ lrow,
                              const int32_t* __restrict__ lcol, const int64_t* __restrict__ loff, int64_t base,
                              int32_t r0, int kb, const int32_t* __restrict__ mptr, const int32_t* __restrict__ mcol,
                              uint64_t* __restrict__ keys) {
    const int32_t p = p0 + blockIdx.x * kThreads + threadIdx.x;
    if (p >= p1) return;
    const int32_t j = lcol[p];
    const uint64_t hi = static_cast<uint64_t>(lrow[p] - r0) << kb;
    uint64_t* out = keys + (loff[p] - base);
    for (int32_t q = mptr[j]; q < mptr[j + 1]; ++q) *out++ = hi | static_cast<uint32_t>(mcol[q]);
}

__global__ void decode_cols_kernel(int32_t u, const uint64_t* __restrict__ uniq, uint64_t mask,
                                   int32_t* __restrict__ col) {
    const int32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e < u) col[e] = static_cast<int32_t>(uniq[e] & mask);
}

// rowptr[r] = base + (number of unique keys of rows before r), for the chunk's rows.
__global__ void decode_rowptr_kernel(int32_t rows, const uint64_t* __restrict__ uniq, int32_t u, int kb,
                                     int32_t base, int32_t* __restrict__ rowptr) {
    const int32_t r = blockIdx.x * kThreads + threadIdx.x;
    if (r >= rows) return;
    const uint64_t key = static_cast<uint64_t>(r) << kb;
    int32_t lo = 0, hi = u;
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (uniq[mid] < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    rowptr[r] = base + lo;
}

__global__ void set_int_kernel(int32_t* __restrict__ dst, int32_t v) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *dst = v;
}

// c_ik = sum over L's row i, ascending j, of L_ij * M_jk where M_jk is stored.
__global__ void numeric_kernel(int32_t u, const int32_t* __restrict__ crow, const int32_t* __restrict__ ccol,
                               const int32_t* __restrict__ lptr, const int32_t* __restrict__ lcol,
                               const double* __restrict__ lval, const int32_t* __restrict__ mptr,
                               const int32_t* __restrict__ mcol, const double* __restrict__ mval,
                               double* __restrict__ cval) {
    const int32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e >= u) return;
    const int32_t i = crow[e], k = ccol[e];
    double s = 0.0;
    for (int32_t p = lptr[i]; p < lptr[i + 1]; ++p) {
        const int32_t j = lcol[p];
        const int32_t end = mptr[j + 1];
        int32_t lo = mptr[j], hi = end;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (mcol[mid] < k)
                lo = mid + 1;
            else
                hi = mid;
        }
        if (lo < end && mcol[lo] == k) s = s + lval[p] * mval[lo];
    }
    cval[e] = s;
}

// flag[e] = 1 for entries kept in A_c (nonzero or diagonal); flag[u] = 0 (scan sentinel).
__global__ void keep_flag_kernel(int32_t u, const int32_t* __restrict__ crow, const int32_t* __restrict__ ccol,
                                 const double* __restrict__ cval, int32_t* __restrict__ flag) {
    const int32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e > u) return;
    flag[e] = e < u && (cval[e] != 0.0 || ccol[e] == crow[e]) ? 1 : 0;
}

__global__ void compact_kernel(int32_t u, const int32_t* __restrict__ flag, const int32_t* __restrict__ pos,
                               const int32_t* __restrict__ ccol, const double* __restrict__ cval,
                               int32_t* __restrict__ col2, double* __restrict__ val2) {
    const int32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e >= u || !flag[e]) return;
    col2[pos[e]] = ccol[e];
    val2[pos[e]] = cval[e];
}

__global__ void remap_rowptr_kernel(int32_t n, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ pos,
                                    int32_t* __restrict__ rowptr2) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i <= n) rowptr2[i] = pos[rowptr[i]];
}

// ---------------------------------------------------------------------------------------
// Host orchestration
// ---------------------------------------------------------------------------------------
struct Failure {
    int code;
    std::string msg;
};

void check(hipError_t e, const char* where) {
    if (e != hipSuccess) throw Failure{AMGG_EHIP, std::string(where) + ": " + hipGetErrorString(e)};
}

struct DevCsr {
    int32_t nrows = 0, ncols = 0, nnz = 0;
    int32_t* ptr = nullptr;
    int32_t* col = nullptr;
    double* val = nullptr;
};

// Device memory from the caller's allocator; what is not taken as a result is released
// when the pool goes out of scope.
class Pool {
  public:
    Pool(amgg_alloc_fn a, amgg_release_fn r, void* u, hipStream_t st) : alloc_(a), release_(r), user_(u), st_(st) {}
    ~Pool() {
        if (!live_.empty()) (void)hipStreamSynchronize(st_);  // queued work may still use them
        for (void* p : live_) release_(p, user_);
    }
    template <class T>
    T* get(int64_t count) {
        const size_t bytes = static_cast<size_t>(std::max<int64_t>(count, 1)) * sizeof(T);
        void* p = alloc_(bytes, user_);
        if (!p) throw Failure{AMGG_EWORKSPACE, "amgg_galerkin_device: allocation of " + std::to_string(bytes) +
                                                   " bytes failed"};
        live_.push_back(p);
        return static_cast<T*>(p);
    }
    void put(const void* p) {
        auto it = std::find(live_.begin(), live_.end(), p);
        if (it == live_.end()) return;
        check(hipStreamSynchronize(st_), "hipStreamSynchronize");
        release_(*it, user_);
        live_.erase(it);
    }
    size_t mark() const { return live_.size(); }
    // Releases what was taken since mark() and is still held, except the arrays of `kept` (null: of none).
    void put_since(size_t from, const DevCsr* kept);
    void keep(const void* p) {  // hand to the caller
        auto it = std::find(live_.begin(), live_.end(), p);
        if (it != live_.end()) live_.erase(it);
    }

  private:
    amgg_alloc_fn alloc_;
    amgg_release_fn release_;
    void* user_;
    hipStream_t st_;
    std::vector<void*> live_;
};

void Pool::put_since(size_t from, const DevCsr* kept) {
    const std::vector<void*> taken(live_.begin() + from, live_.end());
    for (void* p : taken)
        if (!kept || (p != kept->ptr && p != kept->col && p != kept->val)) put(p);
}

struct ConstCsr {
    int32_t nrows, ncols, nnz;
    const int32_t* ptr;
    const int32_t* col;
    const double* val;
};

template <class T>
T read_back(const T* dev, hipStream_t st) {
    T v{};
    check(hipMemcpyAsync(&v, dev, sizeof(T), hipMemcpyDeviceToHost, st), "hipMemcpyAsync");
    check(hipStreamSynchronize(st), "hipStreamSynchronize");
    return v;
}

// C = L * M with the pattern of every structurally generated entry (zeros kept).
DevCsr spgemm(Pool& pool, const ConstCsr& L, const ConstCsr& M, int64_t budget, hipStream_t st) {
    const int32_t n = L.nrows;
    DevCsr C;
    C.nrows = n;
    C.ncols = M.ncols;
    C.ptr = pool.get<int32_t>(static_cast<int64_t>(n) + 1);
    // products per entry of L and their offsets (row i's products start at loff[lptr[i]])
    int32_t* lrow = pool.get<int32_t>(L.nnz);
    int64_t* cnt = pool.get<int64_t>(static_cast<int64_t>(L.nnz) + 1);
    int64_t* loff = pool.get<int64_t>(static_cast<int64_t>(L.nnz) + 1);
    launch(row_index_kernel, n, st, n, L.ptr, lrow);
    launch(product_count_kernel, static_cast<int64_t>(L.nnz) + 1, st,
                       L.nnz, L.col, M.ptr, cnt);
    check(hipGetLastError(), "product count");
    size_t tb = 0;
    check(rocprim::exclusive_scan(nullptr, tb, cnt, loff, int64_t{0}, static_cast<size_t>(L.nnz) + 1,
                                  rocprim::plus<int64_t>(), st),
          "scan size");
    void* tmp = pool.get<unsigned char>(static_cast<int64_t>(tb));
    check(rocprim::exclusive_scan(tmp, tb, cnt, loff, int64_t{0}, static_cast<size_t>(L.nnz) + 1,
                                  rocprim::plus<int64_t>(), st),
          "product offsets");
    pool.put(tmp);
    pool.put(cnt);
    const int64_t total = read_back(loff + L.nnz, st);

    // row chunks of at most about `budget` products
    const int32_t m_count = static_cast<int32_t>(std::max<int64_t>(1, (total + budget - 1) / budget));
    int32_t* dbounds = pool.get<int32_t>(m_count + 1);
    int64_t* dboff = pool.get<int64_t>(m_count + 1);
    launch(chunk_bounds_kernel, m_count + 1, st, n, L.ptr, loff,
                       budget, m_count, dbounds, dboff);
    check(hipGetLastError(), "chunk bounds");
    std::vector<int32_t> bounds(m_count + 1);
    std::vector<int64_t> boff(m_count + 1);
    check(hipMemcpyAsync(bounds.data(), dbounds, sizeof(int32_t) * (m_count + 1), hipMemcpyDeviceToHost, st), "copy");
    check(hipMemcpyAsync(boff.data(), dboff, sizeof(int64_t) * (m_count + 1), hipMemcpyDeviceToHost, st), "copy");
    check(hipStreamSynchronize(st), "hipStreamSynchronize");
    pool.put(dbounds);
    pool.put(dboff);

    const int kb = std::max(1, bit_width(static_cast<uint64_t>(std::max(M.ncols, 1) - 1)));
    const uint64_t mask = (uint64_t{1} << kb) - 1;
    std::vector<int32_t*> part_col;
    std::vector<int32_t> part_u;
    int64_t u_total = 0;
    int32_t* dnum = pool.get<int32_t>(1);
    for (int32_t m = 0; m < m_count; ++m) {
        const int32_t r0 = bounds[m], r1 = bounds[m + 1];
        if (r1 <= r0) continue;
        const int64_t tc = boff[m + 1] - boff[m];
        if (tc > INT32_MAX) throw Failure{AMGG_EINVAL, "amgg_galerkin_device: a row holds more than 2^31 - 1 products"};
        int32_t u = 0;
        int32_t* col = pool.get<int32_t>(std::max<int64_t>(tc, 1));
        if (tc > 0) {
            const int rb = std::max(1, bit_width(static_cast<uint64_t>(r1 - r0 - 1)));
            uint64_t* ka = pool.get<uint64_t>(tc);
            uint64_t* kbuf = pool.get<uint64_t>(tc);
            int32_t p0 = 0, p1 = 0;
            check(hipMemcpyAsync(&p0, L.ptr + r0, sizeof(int32_t), hipMemcpyDeviceToHost, st), "copy");
            check(hipMemcpyAsync(&p1, L.ptr + r1, sizeof(int32_t), hipMemcpyDeviceToHost, st), "copy");
            check(hipStreamSynchronize(st), "hipStreamSynchronize");
            launch(expand_kernel, p1 - p0, st, p0, p1, lrow, L.col,
                               loff, boff[m], r0, kb, M.ptr, M.col, ka);
            check(hipGetLastError(), "expand");
            rocprim::double_buffer<uint64_t> db(ka, kbuf);
            size_t sb = 0, ub = 0;
            const unsigned int end_bit = static_cast<unsigned int>(kb + rb);
            check(rocprim::radix_sort_keys(nullptr, sb, db, static_cast<size_t>(tc), 0u, end_bit, st), "sort size");
            check(rocprim::unique(nullptr, ub, db.current(), db.alternate(), dnum, static_cast<size_t>(tc),
                                  rocprim::equal_to<uint64_t>(), st),
                  "unique size");
            void* t2 = pool.get<unsigned char>(static_cast<int64_t>(std::max(sb, ub)));
            check(rocprim::radix_sort_keys(t2, sb, db, static_cast<size_t>(tc), 0u, end_bit, st), "sort");
            uint64_t* sorted = db.current();
            uint64_t* uniq = db.alternate();
            check(rocprim::unique(t2, ub, sorted, uniq, dnum, static_cast<size_t>(tc), rocprim::equal_to<uint64_t>(),
                                  st),
                  "unique");
            pool.put(t2);
            u = read_back(dnum, st);
            if (u_total + u > INT32_MAX)
                throw Failure{AMGG_EINVAL, "amgg_galerkin_device: product has more than 2^31 - 1 entries"};
            launch(decode_cols_kernel, u, st, u, uniq, mask, col);
            launch(decode_rowptr_kernel, r1 - r0, st, r1 - r0, uniq,
                               u, kb, static_cast<int32_t>(u_total), C.ptr + r0);
            check(hipGetLastError(), "decode");
            check(hipStreamSynchronize(st), "hipStreamSynchronize");
            pool.put(ka);
            pool.put(kbuf);
        } else {
            launch(decode_rowptr_kernel, r1 - r0, st, r1 - r0,
                               static_cast<const uint64_t*>(nullptr), 0, kb, static_cast<int32_t>(u_total), C.ptr + r0);
            check(hipGetLastError(), "decode");
        }
        part_col.push_back(col);
        part_u.push_back(u);
        u_total += u;
    }
    pool.put(dnum);
    pool.put(lrow);
    pool.put(loff);
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, C.ptr + n, static_cast<int32_t>(u_total));
    check(hipGetLastError(), "row pointer");
    C.nnz = static_cast<int32_t>(u_total);
    if (part_col.size() == 1) {
        C.col = part_col[0];
    } else {
        C.col = pool.get<int32_t>(u_total);
        int64_t at = 0;
        for (size_t c = 0; c < part_col.size(); ++c) {
            if (part_u[c] > 0)
                check(hipMemcpyAsync(C.col + at, part_col[c], sizeof(int32_t) * part_u[c], hipMemcpyDeviceToDevice,
                                     st),
                      "copy");
            at += part_u[c];
        }
        check(hipStreamSynchronize(st), "hipStreamSynchronize");
        for (int32_t* p : part_col) pool.put(p);
    }
    // numeric phase
    int32_t* crow = pool.get<int32_t>(C.nnz);
    C.val = pool.get<double>(C.nnz);
    launch(row_index_kernel, n, st, n, C.ptr, crow);
    launch(numeric_kernel, C.nnz, st, C.nnz, crow, C.col, L.ptr,
                       L.col, L.val, M.ptr, M.col, M.val, C.val);
    check(hipGetLastError(), "numeric");
    check(hipStreamSynchronize(st), "hipStreamSynchronize");
    pool.put(crow);
    return C;
}

template <typename T>
void exclusive_scan_i32(Pool& pool, const T* in, int32_t* out, int64_t count, hipStream_t st) {
    size_t tb = 0;
    check(rocprim::exclusive_scan(nullptr, tb, in, out, int32_t{0}, static_cast<size_t>(count),
                                  rocprim::plus<int32_t>(), st),
          "scan size");
    void* tmp = pool.get<unsigned char>(static_cast<int64_t>(tb));
    check(rocprim::exclusive_scan(tmp, tb, in, out, int32_t{0}, static_cast<size_t>(count), rocprim::plus<int32_t>(),
                                  st),
          "scan");
}

// ---------------------------------------------------------------------------------------
// Row-wise product in LDS
// ---------------------------------------------------------------------------------------
// Classes of rows by their products: threads per row and most products. The first kHashClasses hold the row in
// a hash table with a slot for every product (so that it never overflows), the others sort the products.
constexpr int kClasses = 5, kHashClasses = 3;
constexpr int kClassThreads[kClasses] = {8, 16, 64, 256, 1024};
constexpr int kClassSlots[kClasses] = {32, 128, 1024, 2048, 8192};
constexpr int kRowMax = kClassSlots[kClasses - 1];

// nprod[i] = products of row i (some number above kRowMax where there are more); per class the number of its
// rows; [kClasses]: rows beyond the classes, [kClasses + 1]: all products. A thread per row; rows of more than
// kAlone entries are counted by the wavefront and only until they exceed kRowMax (a hub row of 20,000
// entries took its thread 2.7 ms).
constexpr int kAlone = 64;
__global__ __launch_bounds__(kThreads) void row_products_kernel(int32_t n, const int32_t* __restrict__ lptr,
                                                               const int32_t* __restrict__ lcol,
                                                               const int32_t* __restrict__ mptr,
                                                               int32_t* __restrict__ nprod,
                                                               unsigned long long* __restrict__ stats) {
    __shared__ unsigned long long sums[kClasses + 2];
    if (threadIdx.x < kClasses + 2) sums[threadIdx.x] = 0;
    __syncthreads();
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int32_t pb = i < n ? lptr[i] : 0, ne = i < n ? lptr[i + 1] - pb : 0;
    int64_t c = 0;
    if (ne <= kAlone)
        for (int32_t e = 0; e < ne; ++e) {
            const int32_t j = lcol[pb + e];
            c += mptr[j + 1] - mptr[j];
        }
    for (uint64_t rows = __builtin_amdgcn_ballot_w64(ne > kAlone); rows; rows &= rows - 1) {
        const int l = __builtin_ctzll(rows);
        const int32_t b = __builtin_amdgcn_readlane(pb, l), m = __builtin_amdgcn_readlane(ne, l);
        constexpr int kAhead = 4;
        int64_t sum = 0;
        for (int32_t e0 = 0; e0 < m && sum <= kRowMax; e0 += kAhead * 64) {
            int64_t v = 0;
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int32_t e = e0 + q * 64 + lane, j = lcol[b + min(e, m - 1)];
                v += e < m ? mptr[j + 1] - mptr[j] : 0;
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            sum += v;
        }
        if (lane == l) c = sum;
    }
    if (i < n) nprod[i] = static_cast<int32_t>(c < INT32_MAX ? c : INT32_MAX);
    int cls = 0;
    while (cls < kClasses && c > kClassSlots[cls]) ++cls;
    // one LDS update per wavefront and value (64 lanes on one address take turns)
#pragma unroll
    for (int k = 0; k <= kClasses; ++k) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(c > 0 && cls == k);
        if (lane == 0 && m) atomicAdd(&sums[k], static_cast<unsigned long long>(__popcll(m)));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0 && c) atomicAdd(&sums[kClasses + 1], static_cast<unsigned long long>(c));
    __syncthreads();
    if (threadIdx.x < kClasses + 2 && sums[threadIdx.x]) atomicAdd(stats + threadIdx.x, sums[threadIdx.x]);
}

// The rows of each class (their order within it decides nothing); a row without products has no entries.
struct ClassLists {
    int32_t* rows[kClasses];
};
__global__ __launch_bounds__(kThreads) void classify_rows_kernel(int32_t n, const int32_t* __restrict__ nprod,
                                                                ClassLists lists, int32_t* __restrict__ used,
                                                                int32_t* __restrict__ cnt) {
    __shared__ int32_t have[kClasses], at[kClasses];
    if (threadIdx.x < kClasses) have[threadIdx.x] = 0;
    __syncthreads();
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    int cls = kClasses, pos = 0;
    if (i < n) {
        const int32_t c = nprod[i];
        if (c == 0) cnt[i] = 0;
        cls = c == 0 ? kClasses : 0;
        while (cls < kClasses && c > kClassSlots[cls]) ++cls;
        if (cls < kClasses) pos = atomicAdd(&have[cls], 1);
    }
    __syncthreads();
    if (threadIdx.x < kClasses && have[threadIdx.x]) at[threadIdx.x] = atomicAdd(used + threadIdx.x, have[threadIdx.x]);
    __syncthreads();
    if (cls < kClasses) lists.rows[cls][at[cls] + pos] = i;
}

// Orders the LDS accesses of a group of lanes of one wavefront, whose LDS accesses are in order.
__device__ __forceinline__ void group_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// What the row kernels take: rows of C = L M (the listed ones, or the first `count`). FILL: a row's columns and
// values are written at cptr[i]; else its entry count. zeros: set to 1 if an exact zero is written off
// the diagonal.
struct RowProducts {
    int32_t count;
    const int32_t* rows;
    const int32_t *lptr, *lcol;
    const double* lval;
    const int32_t *mptr, *mcol;
    const double* mval;
    int32_t* cnt;
    const int32_t* cptr;
    int32_t* ccol;
    double* cval;
    int32_t* zeros;
};

// A row by G lanes in a table of S slots. Bound by latency: an entry of L costs its row bounds of M, its row and
// the table. The row bounds of G entries of L are loaded together and an entry's row of M while the one
// before it is added.
template <int G, int S, bool FILL>
__global__ __launch_bounds__(kThreads) void row_hash_kernel(RowProducts a) {
    constexpr int kRows = kThreads / G;
    __shared__ __align__(16) int32_t keys[kRows][S];
    __shared__ double vals[kRows][FILL ? S : 1];
    const int g = threadIdx.x / G, t = threadIdx.x % G;
    const int32_t at = static_cast<int32_t>(blockIdx.x) * kRows + g;
    const bool mine = at < a.count;  // uniform over the group
    const int32_t i = !mine ? 0 : a.rows ? a.rows[at] : at;
    int32_t* const key = keys[g];
    double* const val = FILL ? vals[g] : nullptr;
    for (int k = t; k < S; k += G) {
        key[k] = -1;
        if constexpr (FILL) val[k] = 0.0;
    }
    group_sync();
    const int32_t pb = mine ? a.lptr[i] : 0, np = mine ? a.lptr[i + 1] - pb : 0;
    for (int32_t e0 = 0; e0 < np; e0 += G) {
        // the next G entries of L, one per thread
        const int32_t p = pb + min(e0 + t, np - 1);
        const int32_t j = a.lcol[p];
        const int32_t mb0 = a.mptr[j], me0 = a.mptr[j + 1];
        const double lv0 = FILL ? a.lval[p] : 0.0;
        auto bounds = [&](int e, int32_t& b, int32_t& x, double& v) {
            b = __shfl(mb0, e, G);
            x = __shfl(me0, e, G);
            v = FILL ? __shfl(lv0, e, G) : 0.0;
        };
        const int32_t ne = min(np - e0, G);
        int32_t b, x, kn = 0;
        double lv, vn = 0.0;
        bounds(0, b, x, lv);
        if (t < x - b) {
            kn = a.mcol[b + t];
            if constexpr (FILL) vn = a.mval[b + t];
        }
        for (int e = 0; e < ne; ++e) {
            const int32_t bc = b, xc = x;
            const double lc = lv;
            int32_t k = kn;
            double m = vn;
            if (e + 1 < ne) {
                bounds(e + 1, b, x, lv);
                if (t < x - b) {
                    kn = a.mcol[b + t];
                    if constexpr (FILL) vn = a.mval[b + t];
                }
            }
            for (int32_t q = t; q < xc - bc; q += G) {
                if (q != t) {
                    k = a.mcol[bc + q];
                    if constexpr (FILL) m = a.mval[bc + q];
                }
                unsigned int s = static_cast<unsigned int>(k) * 2654435769u >> (32 - __builtin_ctz(S));
                for (;;) {  // ends: the table has a slot for every product
                    const int32_t old = atomicCAS(&key[s], -1, k);
                    if (old == -1 || old == k) break;
                    s = (s + 1) & (S - 1);
                }
                if constexpr (FILL) val[s] = val[s] + lc * m;  // no other thread has column k in this step
            }
            group_sync();
        }
    }
    // entries of the row, moved to the front of the table: a round's entries go to places that it or an
    // earlier round has read
    const int sh = threadIdx.x & 63 & ~(G - 1);
    const uint64_t gm = G == 64 ? ~0ull : (1ull << (G & 63)) - 1;
    int32_t u = 0;
    for (int k0 = 0; k0 < S; k0 += G) {
        const int32_t k = key[k0 + t];
        const uint64_t m = __builtin_amdgcn_ballot_w64(k >= 0) >> sh & gm;
        if constexpr (FILL) {
            const double v = val[k0 + t];
            group_sync();
            if (k >= 0) {
                const int to = u + __popcll(m & ((1ull << t) - 1));
                key[to] = k;
                val[to] = v;
            }
            group_sync();
        }
        u += __popcll(m);
    }
    if constexpr (!FILL) {
        if (t == 0 && mine) a.cnt[i] = u;
    } else {
        if (t < (4 - u % 4) % 4) key[u + t] = INT32_MAX;
        group_sync();
        if (!mine) return;
        // an entry's place is the number of smaller columns, four per read (broadcast) of the table
        const int32_t base = a.cptr[i];
        bool zero = false;
        for (int32_t r = t; r < u; r += G) {
            const int32_t k = key[r];
            int32_t rank = 0;
            for (int32_t q = 0; q < u; q += 4) {
                const int4 o = *reinterpret_cast<const int4*>(key + q);
                rank += (o.x < k) + (o.y < k) + (o.z < k) + (o.w < k);
            }
            const double v = val[r];
            a.ccol[base + rank] = k;
            a.cval[base + rank] = v;
            zero = zero || (v == 0.0 && k != i);
        }
        if (zero && a.zeros) *a.zeros = 1;
    }
}

// A long row by a workgroup of T threads, at most S products: its products are laid out in LDS in their order
// (the threads find a product's entry of L by bisection in the scanned lengths), sorted by (column, place), and
// each column's are added from its first to its last. All threads work whatever the lengths of the rows of
// M; a table takes one entry of L after the other, two products at a time where M is a prolongation, and
// ranks by the square of the row's entries. Whole call, ms, with tables of 8192 slots, sorted and
// expanding: a 90k-row grid with a hub of 3900 neighbours 15.1 / 1.6 / 5.1, with 40 of them 15.9 / 1.6 / 6.2,
// 1500 rows of 700 entries 3.5 / 1.7 / 2.9.
template <int T, int S, bool FILL>
__global__ __launch_bounds__(T) void row_sort_kernel(RowProducts a) {
    static_assert(S <= 1 << 16, "places take 16 bits of a key");
    __shared__ uint64_t keys[S];
    __shared__ double vals[FILL ? S : 1];
    __shared__ int32_t ends[T], begs[T], wsum[T / 64];
    __shared__ double lvals[FILL ? T : 1];
    const int t = threadIdx.x;
    const int32_t i = a.rows ? a.rows[blockIdx.x] : static_cast<int32_t>(blockIdx.x);
    const int32_t pb = a.lptr[i], np = a.lptr[i + 1] - pb;
    int32_t total = 0;
    for (int32_t e0 = 0; e0 < np; e0 += T) {
        int32_t len = 0, incl;
        if (e0 + t < np) {
            const int32_t j = a.lcol[pb + e0 + t], b = a.mptr[j];
            len = a.mptr[j + 1] - b;
            begs[t] = b;
            if constexpr (FILL) lvals[t] = a.lval[pb + e0 + t];
        }
        incl = len;
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t o = __shfl_up(incl, off, 64);
            if ((t & 63) >= off) incl += o;
        }
        if ((t & 63) == 63) wsum[t / 64] = incl;
        __syncthreads();
        for (int w = 0; w < t / 64; ++w) incl += wsum[w];
        ends[t] = incl;
        __syncthreads();
        const int32_t chunk = ends[T - 1];
        for (int32_t s = t; s < chunk; s += T) {
            int32_t lo = 0, hi = T - 1;  // the first entry that ends past s
            while (lo < hi) {
                const int32_t mid = (lo + hi) / 2;
                if (ends[mid] > s)
                    hi = mid;
                else
                    lo = mid + 1;
            }
            const int32_t q = begs[lo] + s - (lo > 0 ? ends[lo - 1] : 0), at = total + s;
            keys[at] = static_cast<uint64_t>(a.mcol[q]) << 16 | static_cast<uint32_t>(at);
            if constexpr (FILL) vals[at] = lvals[lo] * a.mval[q];
        }
        total += chunk;
        __syncthreads();
    }
    int32_t span = 2;
    while (span < total) span *= 2;
    for (int32_t k = total + t; k < span; k += T) keys[k] = ~0ull;
    __syncthreads();
    for (int32_t size = 2; size <= span; size *= 2)  // bitonic
        for (int32_t step = size / 2; step > 0; step /= 2) {
            for (int32_t k = t; k < span / 2; k += T) {
                const int32_t lo = 2 * k - (k & (step - 1)), hi = lo + step;
                const uint64_t x = keys[lo], y = keys[hi];
                if ((x > y) == ((lo & size) == 0)) {
                    keys[lo] = y;
                    keys[hi] = x;
                }
            }
            __syncthreads();
        }
    const int32_t base = FILL ? a.cptr[i] : 0;
    int32_t u = 0;  // entries so far
    bool zero = false;
    for (int32_t k0 = 0; k0 < total; k0 += T) {
        const int32_t k = k0 + t;
        const uint64_t c = k < total ? keys[k] >> 16 : 0;
        const bool head = k < total && (k == 0 || keys[k - 1] >> 16 != c);
        const uint64_t m = __builtin_amdgcn_ballot_w64(head);
        if ((t & 63) == 0) wsum[t / 64] = __popcll(m);
        __syncthreads();
        int32_t before = u + __popcll(m & ((1ull << (t & 63)) - 1));
        for (int w = 0; w < T / 64; ++w) {
            if (w < t / 64) before += wsum[w];
            u += wsum[w];
        }
        if constexpr (FILL)
            if (head) {
                double s = 0.0;
                for (int32_t q = k; q < total && keys[q] >> 16 == c; ++q) s = s + vals[keys[q] & 0xffff];
                a.ccol[base + before] = static_cast<int32_t>(c);
                a.cval[base + before] = s;
                zero = zero || (s == 0.0 && static_cast<int32_t>(c) != i);
            }
        __syncthreads();
    }
    if constexpr (!FILL) {
        if (t == 0) a.cnt[i] = u;
    } else {
        if (zero && a.zeros) *a.zeros = 1;
    }
}

template <bool FILL>
void launch_rows(const unsigned long long* rows, const ClassLists& lists, hipStream_t st, RowProducts a) {
    auto go = [&](auto kernel, int cls) {
        if (rows[cls] == 0) return;
        const unsigned threads = std::max(kThreads, kClassThreads[cls]), per = threads / kClassThreads[cls];
        a.count = static_cast<int32_t>(rows[cls]);
        a.rows = lists.rows[cls];
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((rows[cls] + per - 1) / per)), dim3(threads), 0, st, a);
    };
    static_assert(kHashClasses == 3 && kClasses == 5, "one launch per class");
    go(row_hash_kernel<kClassThreads[0], kClassSlots[0], FILL>, 0);
    go(row_hash_kernel<kClassThreads[1], kClassSlots[1], FILL>, 1);
    go(row_hash_kernel<kClassThreads[2], kClassSlots[2], FILL>, 2);
    go(row_sort_kernel<kClassThreads[3], kClassSlots[3], FILL>, 3);
    go(row_sort_kernel<kClassThreads[4], kClassSlots[4], FILL>, 4);
    check(hipGetLastError(), "row products");
}

// C = L * M with the pattern of every structurally generated entry; false where the expanding form is
// needed. zeros (device, set to 1 if an exact zero was written off the diagonal; null: not wanted).
bool spgemm_rows(Pool& pool, const ConstCsr& L, const ConstCsr& M, int32_t* zeros, DevCsr& C, hipStream_t st) {
    const int32_t n = L.nrows;
    int32_t* nprod = pool.get<int32_t>(n);
    auto* stats = pool.get<unsigned long long>(2 * kClasses + 2);
    auto* used = reinterpret_cast<int32_t*>(stats + kClasses + 2);
    check(vec_zero_bytes(stats, sizeof(unsigned long long) * (2 * kClasses + 2), st), "row products");
    launch(row_products_kernel, n, st, n, L.ptr, L.col, M.ptr, nprod, stats);
    check(hipGetLastError(), "row products");
    unsigned long long rows[kClasses + 2];
    check(hipMemcpyAsync(rows, stats, sizeof(rows), hipMemcpyDeviceToHost, st), "copy");
    check(hipStreamSynchronize(st), "hipStreamSynchronize");
    if (rows[kClasses] || rows[kClasses + 1] > INT32_MAX) return false;
    C.nrows = n;
    C.ncols = M.ncols;
    C.ptr = pool.get<int32_t>(static_cast<int64_t>(n) + 1);
    int32_t* cnt = pool.get<int32_t>(static_cast<int64_t>(n) + 1);
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, cnt + n, 0);
    ClassLists lists;
    bool listed = true;  // false: every row is of one class
    for (int c = 0; c < kClasses; ++c) listed = listed && rows[c] != static_cast<unsigned long long>(n);
    for (int c = 0; c < kClasses; ++c) lists.rows[c] = pool.get<int32_t>(listed ? static_cast<int64_t>(rows[c]) : 1);
    if (listed)
        launch(classify_rows_kernel, n, st, n, nprod, lists, used, cnt);
    else
        lists = ClassLists{};
    RowProducts a{0, nullptr, L.ptr, L.col, L.val, M.ptr, M.col, M.val, cnt, nullptr, nullptr, nullptr, nullptr};
    launch_rows<false>(rows, lists, st, a);
    exclusive_scan_i32(pool, cnt, C.ptr, static_cast<int64_t>(n) + 1, st);
    C.nnz = read_back(C.ptr + n, st);
    C.col = pool.get<int32_t>(C.nnz);
    C.val = pool.get<double>(C.nnz);
    a.cptr = C.ptr;
    a.ccol = C.col;
    a.cval = C.val;
    a.zeros = zeros;
    launch_rows<true>(rows, lists, st, a);
    return true;
}

// Drops exact zeros off the diagonal; the result's arrays replace C's.
DevCsr drop_zeros(Pool& pool, const DevCsr& C, hipStream_t st) {
    int32_t* crow = pool.get<int32_t>(C.nnz);
    int32_t* flag = pool.get<int32_t>(static_cast<int64_t>(C.nnz) + 1);
    int32_t* pos = pool.get<int32_t>(static_cast<int64_t>(C.nnz) + 1);
    launch(row_index_kernel, C.nrows, st, C.nrows, C.ptr, crow);
    launch(keep_flag_kernel, static_cast<int64_t>(C.nnz) + 1, st,
                       C.nnz, crow, C.col, C.val, flag);
    check(hipGetLastError(), "keep flags");
    size_t tb = 0;
    check(rocprim::exclusive_scan(nullptr, tb, flag, pos, int32_t{0}, static_cast<size_t>(C.nnz) + 1,
                                  rocprim::plus<int32_t>(), st),
          "scan size");
    void* tmp = pool.get<unsigned char>(static_cast<int64_t>(tb));
    check(rocprim::exclusive_scan(tmp, tb, flag, pos, int32_t{0}, static_cast<size_t>(C.nnz) + 1,
                                  rocprim::plus<int32_t>(), st),
          "keep positions");
    pool.put(tmp);
    const int32_t kept = read_back(pos + C.nnz, st);
    DevCsr D = C;
    if (kept != C.nnz) {
        D.nnz = kept;
        D.ptr = pool.get<int32_t>(static_cast<int64_t>(C.nrows) + 1);
        D.col = pool.get<int32_t>(kept);
        D.val = pool.get<double>(kept);
        launch(compact_kernel, C.nnz, st, C.nnz, flag, pos, C.col,
                           C.val, D.col, D.val);
        launch(remap_rowptr_kernel, static_cast<int64_t>(C.nrows) + 1, st, C.nrows, C.ptr, pos, D.ptr);
        check(hipGetLastError(), "compact");
        check(hipStreamSynchronize(st), "hipStreamSynchronize");
        pool.put(C.ptr);
        pool.put(C.col);
        pool.put(C.val);
    }
    pool.put(crow);
    pool.put(flag);
    pool.put(pos);
    return D;
}

// ---------------------------------------------------------------------------------------
// Strength and direct interpolation: one thread per row, the host setup's formulas in the
// host setup's order (entries in stored, ascending column order; every operation rounded).
// ---------------------------------------------------------------------------------------
// strong[p] = 1 when entry p (column j != i) of row i has -a_ij >= theta max_{k != i}(-a_ik)
// and that max is positive.
__global__ void strength_kernel(int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                const double* __restrict__ val, double theta, uint8_t* __restrict__ strong) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int32_t pb = ptr[i], pe = ptr[i + 1];
    double big = -INFINITY;
    bool any_off = false;
    for (int32_t p = pb; p < pe; ++p) {
        if (col[p] == i) continue;
        any_off = true;
        const double v = -val[p];
        big = big < v ? v : big;
    }
    const bool some = any_off && big > 0.0;
    const double cut = theta * big;
    for (int32_t p = pb; p < pe; ++p) strong[p] = some && col[p] != i && -val[p] >= cut ? 1 : 0;
}

// cf as int32 with a trailing 0 (its exclusive scan numbers the C points)
__global__ void cf_to_int_kernel(int32_t n, const int8_t* __restrict__ cf, int32_t* __restrict__ out) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i < n) out[i] = cf[i] != 0 ? 1 : 0;
    if (i == n) out[i] = 0;
}

// entries of P's row i: 1 for a C point, else the strong C neighbours (0: no interpolation)
__global__ void interp_count_kernel(int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                    const uint8_t* __restrict__ strong, const int8_t* __restrict__ cf,
                                    int32_t* __restrict__ cnt) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i == n) cnt[i] = 0;
    if (i >= n) return;
    if (cf[i] != 0) {
        cnt[i] = 1;
        return;
    }
    int32_t c = 0;
    for (int32_t p = ptr[i]; p < ptr[i + 1]; ++p) c += strong[p] && cf[col[p]] != 0 ? 1 : 0;
    cnt[i] = c;
}

// Direct interpolation with positive couplings lumped on the diagonal: an F row with strong C
// neighbours C_i gets w_ik = -(alpha_i a_ik) / (a_ii + sum of its positive off-diagonals), with
// alpha_i = (sum of its negative off-diagonals) / (sum of a_ik over C_i); a C row is the identity.
__global__ void interp_fill_kernel(int32_t n, const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                   const double* __restrict__ val, const uint8_t* __restrict__ strong,
                                   const int8_t* __restrict__ cf, const int32_t* __restrict__ cidx,
                                   const int32_t* __restrict__ prow, int32_t* __restrict__ pcol,
                                   double* __restrict__ pval) {
    const int32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    int32_t q = prow[i];
    if (cf[i] != 0) {
        pcol[q] = cidx[i];
        pval[q] = 1.0;
        return;
    }
    if (prow[i + 1] == q) return;
    const int32_t pb = ptr[i], pe = ptr[i + 1];
    double a_ii = 0.0;
    for (int32_t p = pb; p < pe; ++p)
        if (col[p] == i) a_ii = val[p];
    double lumped = a_ii, neg_sum = 0.0, strong_c_sum = 0.0;
    for (int32_t p = pb; p < pe; ++p) {
        const int32_t k = col[p];
        if (k == i) continue;
        const double a = val[p];
        if (a > 0.0) lumped = lumped + a;
        if (a < 0.0) neg_sum = neg_sum + a;
        if (strong[p] && cf[k] != 0) strong_c_sum = strong_c_sum + a;
    }
    const double ratio = neg_sum / strong_c_sum;
    for (int32_t p = pb; p < pe; ++p) {
        const int32_t k = col[p];
        if (!(strong[p] && cf[k] != 0)) continue;
        pcol[q] = cidx[k];
        pval[q] = -(ratio * val[p]) / lumped;
        ++q;
    }
}

// bad[0] = 1 unless (ptr, col) is a CSR pattern of n rows, nnz entries, ascending columns < n
void validate_square(Pool& pool, int32_t n, int32_t nnz, const int32_t* ptr, const int32_t* col, const char* who,
                     hipStream_t st) {
    int32_t* bad = pool.get<int32_t>(1);
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, bad, 0);
    launch(validate_csr_kernel, n, st, n, n, nnz, ptr, col, bad);
    check(hipGetLastError(), "validate");
    if (read_back(bad, st))
        throw Failure{AMGG_EINVAL, std::string(who) + ": not a CSR pattern of the stated size with ascending columns"};
    pool.put(bad);
}

}  // namespace

extern "C" int amgg_strength_device(int device, int32_t n, const int32_t* rowptr, const int32_t* col,
                                    const double* val, int32_t nnz, double theta, uint8_t* strong,
                                    amgg_alloc_fn alloc, amgg_release_fn release, void* user, void* stream) {
    return guarded([&]() -> int {
        if (n <= 0 || nnz < 0 || !rowptr || !alloc || !release || (nnz > 0 && (!col || !val || !strong)))
            return fail(AMGG_EINVAL, "amgg_strength_device: NULL argument or bad size");
        if (!(theta > 0.0 && theta < 1.0)) return fail(AMGG_EINVAL, "amgg_strength_device: theta outside (0, 1)");
        hipError_t e = hipSetDevice(device);
        if (e != hipSuccess) return hip_fail(e, "amgg_strength_device: hipSetDevice");
        const hipStream_t st = static_cast<hipStream_t>(stream);
        try {
            Pool pool(alloc, release, user, st);
            validate_square(pool, n, nnz, rowptr, col, "amgg_strength_device", st);
            launch(strength_kernel, n, st, n, rowptr, col, val, theta, strong);
            check(hipGetLastError(), "strength");
            return AMGG_OK;
        } catch (const Failure& f) {
            (void)hipStreamSynchronize(st);
            return fail(f.code, f.msg);
        }
    });
}

extern "C" int amgg_interp_device(int device, int32_t n, const int32_t* rowptr, const int32_t* col, const double* val,
                                  int32_t nnz, const uint8_t* strong, const int8_t* cf, amgg_alloc_fn alloc,
                                  amgg_release_fn release, void* user, int32_t* nc, int32_t** p_rowptr,
                                  int32_t** p_col, double** p_val, int32_t* p_nnz, void* stream) {
    return guarded([&]() -> int {
        if (n <= 0 || nnz < 0 || !rowptr || !cf || !alloc || !release || !nc || !p_rowptr || !p_col || !p_val ||
            !p_nnz || (nnz > 0 && (!col || !val || !strong)))
            return fail(AMGG_EINVAL, "amgg_interp_device: NULL argument or bad size");
        hipError_t e = hipSetDevice(device);
        if (e != hipSuccess) return hip_fail(e, "amgg_interp_device: hipSetDevice");
        const hipStream_t st = static_cast<hipStream_t>(stream);
        try {
            Pool pool(alloc, release, user, st);
            validate_square(pool, n, nnz, rowptr, col, "amgg_interp_device", st);
            int32_t* tmp = pool.get<int32_t>(static_cast<int64_t>(n) + 1);
            int32_t* cidx = pool.get<int32_t>(static_cast<int64_t>(n) + 1);
            launch(cf_to_int_kernel, static_cast<int64_t>(n) + 1, st, n, cf, tmp);
            exclusive_scan_i32(pool, tmp, cidx, static_cast<int64_t>(n) + 1, st);
            const int32_t ncoarse = read_back(cidx + n, st);
            if (ncoarse <= 0) throw Failure{AMGG_EINVAL, "amgg_interp_device: no C point"};
            int32_t* prow = pool.get<int32_t>(static_cast<int64_t>(n) + 1);
            launch(interp_count_kernel, static_cast<int64_t>(n) + 1, st, n, rowptr, col, strong, cf, tmp);
            exclusive_scan_i32(pool, tmp, prow, static_cast<int64_t>(n) + 1, st);
            const int32_t total = read_back(prow + n, st);
            pool.put(tmp);
            int32_t* pcol = pool.get<int32_t>(total);
            double* pval = pool.get<double>(total);
            launch(interp_fill_kernel, n, st, n, rowptr, col, val, strong, cf, cidx, prow, pcol, pval);
            check(hipGetLastError(), "interpolation");
            check(hipStreamSynchronize(st), "hipStreamSynchronize");
            pool.put(cidx);
            pool.keep(prow);
            pool.keep(pcol);
            pool.keep(pval);
            *nc = ncoarse;
            *p_rowptr = prow;
            *p_col = pcol;
            *p_val = pval;
            *p_nnz = total;
            return AMGG_OK;
        } catch (const Failure& f) {
            (void)hipStreamSynchronize(st);
            return fail(f.code, f.msg);
        }
    });
}

extern "C" int amgg_galerkin_device(int device, int32_t n, int32_t nc, const int32_t* a_rowptr, const int32_t* a_col,
                                    const double* a_val, int32_t a_nnz, const int32_t* p_rowptr, const int32_t* p_col,
                                    const double* p_val, int32_t p_nnz, amgg_alloc_fn alloc, amgg_release_fn release,
                                    void* user, int64_t chunk_products, int32_t** ac_rowptr, int32_t** ac_col,
                                    double** ac_val, int32_t* ac_nnz, void* stream) {
    return guarded([&]() -> int {
        if (n <= 0 || nc <= 0 || a_nnz < 0 || p_nnz < 0 || !a_rowptr || !p_rowptr || !alloc || !release ||
            !ac_rowptr || !ac_col || !ac_val || !ac_nnz || (a_nnz > 0 && (!a_col || !a_val)) ||
            (p_nnz > 0 && (!p_col || !p_val)) || chunk_products < 0)
            return fail(AMGG_EINVAL, "amgg_galerkin_device: NULL argument or bad size");
        const int64_t budget = chunk_products > 0 ? chunk_products : (int64_t{1} << 27);
        if (budget > INT32_MAX) return fail(AMGG_EINVAL, "amgg_galerkin_device: chunk_products above 2^31 - 1");
        hipError_t e = hipSetDevice(device);
        if (e != hipSuccess) return hip_fail(e, "amgg_galerkin_device: hipSetDevice");
        const hipStream_t st = static_cast<hipStream_t>(stream);
        try {
            Pool pool(alloc, release, user, st);
            int32_t* bad = pool.get<int32_t>(2);
            hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, bad, 0);
            hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, bad + 1, 0);
            launch(validate_csr_kernel, n, st, n, n, a_nnz, a_rowptr, a_col, bad);
            launch(validate_csr_kernel, n, st, n, nc, p_nnz, p_rowptr, p_col, bad + 1);
            check(hipGetLastError(), "validate");
            int32_t flags[2] = {0, 0};
            check(hipMemcpyAsync(flags, bad, sizeof(flags), hipMemcpyDeviceToHost, st), "copy");
            check(hipStreamSynchronize(st), "hipStreamSynchronize");
            if (flags[0] || flags[1])
                throw Failure{AMGG_EINVAL, std::string("amgg_galerkin_device: ") + (flags[0] ? "A" : "P") +
                                               " is not a CSR pattern of the stated size with ascending columns"};
            // R = P^T, the exact transpose (rows in ascending fine index)
            DevCsr R;
            R.nrows = nc;
            R.ncols = n;
            R.nnz = p_nnz;
            R.ptr = pool.get<int32_t>(static_cast<int64_t>(nc) + 1);
            R.col = pool.get<int32_t>(p_nnz);
            R.val = pool.get<double>(p_nnz);
            int32_t* cursor = pool.get<int32_t>(static_cast<int64_t>(nc) + 1);
            check(transpose_csr(n, nc, p_nnz, p_rowptr, p_col, p_val, R.ptr, R.col, R.val, cursor, st), "transpose");
            const ConstCsr A{n, n, a_nnz, a_rowptr, a_col, a_val};
            const ConstCsr P{n, nc, p_nnz, p_rowptr, p_col, p_val};
            // The row-wise products' temporaries (a few integers a row) stay until the call returns, each
            // release being a wait; the expanding form, whose memory the caller may bound, starts
            // without them.
            const bool expand = chunk_products > 0;  // the caller bounds the expansion
            int32_t* zeros = bad;                     // 0 again after the checks
            DevCsr AP, G, Ac;
            size_t from = pool.mark();
            if (expand || !spgemm_rows(pool, A, P, nullptr, AP, st)) {
                pool.put_since(from, nullptr);
                AP = spgemm(pool, A, P, budget, st);
                pool.put(cursor);
            }
            const ConstCsr Rc{R.nrows, R.ncols, R.nnz, R.ptr, R.col, R.val};
            const ConstCsr APc{AP.nrows, AP.ncols, AP.nnz, AP.ptr, AP.col, AP.val};
            // exact zeros off the diagonal are rare: the row-wise product tells whether there are any
            bool drop = true;
            if (!expand && spgemm_rows(pool, Rc, APc, zeros, G, st)) {
                drop = read_back(zeros, st) != 0;
            } else {
                pool.put_since(from, &AP);
                G = spgemm(pool, Rc, APc, budget, st);
            }
            if (drop) {
                pool.put_since(from, &G);  // A P and the temporaries
                pool.put(R.ptr);
                pool.put(R.col);
                pool.put(R.val);
            }
            Ac = drop ? drop_zeros(pool, G, st) : G;
            pool.keep(Ac.ptr);
            pool.keep(Ac.col);
            pool.keep(Ac.val);
            *ac_rowptr = Ac.ptr;
            *ac_col = Ac.col;
            *ac_val = Ac.val;
            *ac_nnz = Ac.nnz;
            return AMGG_OK;
        } catch (const Failure& f) {
            (void)hipStreamSynchronize(st);  // the failure is what is reported
            return fail(f.code, f.msg);
        }
    });
}
