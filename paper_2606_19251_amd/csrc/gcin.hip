// GCIN smoother-coefficient predictor on gfx950 (paper Sec. 3.2, Eqs. 6-10; App. A.1,
// Tab. 5): forward, hand-written backward and Adam.
//
// Layout. All graphs of a batch (every level of every problem, Alg. 1 steps 3-6) are
// concatenated; each graph starts on a 64-row tile boundary (pad rows carry no edges and
// are masked), so a tile belongs to exactly one graph and per-graph statistics are fixed
// order sums of per-tile partials (no atomics, bitwise reproducible). Activations are
// FP32 [N x 64] (or [N x 32]) row-major; a tile is processed by one workgroup of four groups of
// 64 (32) lanes with 16 rows each, a lane holding four neighbouring channels of four rows, so that a
// row is 16 lanes' 16-byte accesses, one coalesced 256-byte transaction.
//
// Each GCIN layer is one pass: the neighbour features are normalised and rectified on
// load (InstanceNorm + ReLU of the previous layer applied by the consumer), aggregated
// with the edge weights (A_hat = (A - D) + I), multiplied by Theta_l (64 x 64) and the
// per-tile sums of y and y^2 are emitted for the next InstanceNorm. In BF16 mode the
// 64 x 64 products run on v_mfma_f32_16x16x32_bf16 with FP32 accumulation.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include "amggnn.h"
#include "errors.hpp"
#include "gcin.h"

namespace {

// The hidden width HD (64, or 32 for the smaller variant) is a template parameter of every
// kernel below; a workgroup has 4 HD threads (4 groups of HD lanes, lane = channel).
constexpr int NL = 4;      // GCIN layers
constexpr int RO = 32;     // readout width per layer
constexpr int JK = RO * NL;
constexpr int M1 = 128, M2 = 64;
constexpr int TILE = 64;
constexpr int kAdamThreads = 256;
// Grids of the weight-gradient kernels, at most: what the chip holds of bwd_b_kernel at a time (its LDS leaves
// room for 3 or 7 workgroups per CU), and of bwd_b0_kernel, which keeps nothing but its loads in flight.
constexpr int w_blocks(int hidden) { return hidden == 64 ? 768 : 1792; }
constexpr int kW0Blocks = 1024;
constexpr int kMaxOut = 9;    // 2 d + 1 for d <= 4
constexpr float kEps = 1e-5f;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------
// parameter offsets (order documented in gcin.h)
// ------------------------------------------------------------------------------------------
struct Offs {
    int64_t convW[NL], convb[NL], gam[NL], bet[NL], roW[NL], rob[NL];
    int64_t lng, lnb, m0W, m0b, m1W, m1b, m2W, m2b, head0, total;
    int nout;
};

Offs offsets(int d, int HD) {
    Offs o{};
    int64_t k = 0;
    for (int l = 0; l < NL; ++l) {
        const int in = l == 0 ? 2 : HD;
        o.convW[l] = k; k += in * HD;
        o.convb[l] = k; k += HD;
        o.gam[l] = k; k += HD;
        o.bet[l] = k; k += HD;
    }
    o.head0 = k;
    for (int l = 0; l < NL; ++l) {
        o.roW[l] = k; k += 2 * HD * RO;
        o.rob[l] = k; k += RO;
    }
    o.nout = 2 * d + 1;
    o.lng = k; k += JK;
    o.lnb = k; k += JK;
    o.m0W = k; k += JK * M1;
    o.m0b = k; k += M1;
    o.m1W = k; k += M1 * M2;
    o.m1b = k; k += M2;
    o.m2W = k; k += M2 * o.nout;
    o.m2b = k; k += o.nout;
    o.total = k;
    return o;
}

__device__ __forceinline__ unsigned short f2bf(float f) {
    // round to nearest even (inputs are finite)
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<unsigned short>(u >> 16);
}

__device__ __forceinline__ float normrelu(float y, float mu, float rs, float ga, float be) {
    return fmaxf((y - mu) * rs * ga + be, 0.0f);
}

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>): an unrolled loop whose index is a
// constant expression (the DPP controls below have to be).
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Orders a wavefront's LDS accesses where its lanes exchange values among themselves only.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Reductions over the four groups of G lanes of 4 G lanes (16 rows of HD = 4 G channels), four values per
// lane: every exchange adds (or merges) two values' halves at once, so that three exchanges leave each
// lane with one value's total, the value reduced_channel() of its group.
template <int G>
__device__ __forceinline__ int reduced_channel() {
    const int q = static_cast<int>(threadIdx.x % (4 * G)) / G;
    return (q & 1) * 2 + q / 2;
}
// Exchanges b's lower half of every 2 S lanes with a's upper half.
template <int S>
__device__ __forceinline__ void swap_halves(unsigned int& a, unsigned int& b) {
    if constexpr (S == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else if constexpr (S == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const bool up = (threadIdx.x & S) != 0;
        const unsigned int got = __shfl_xor(up ? a : b, S, 64);
        if (up)
            a = got;
        else
            b = got;
    }
}
template <int S>
__device__ __forceinline__ double add_halves(double a, double b) {
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    swap_halves<S>(x.x, y.x);
    swap_halves<S>(x.y, y.y);
    return __builtin_bit_cast(double, x) + __builtin_bit_cast(double, y);
}
template <int G>
__device__ __forceinline__ double reduce_groups(const double (&v)[4]) {
    return add_halves<G>(add_halves<2 * G>(v[0], v[1]), add_halves<2 * G>(v[2], v[3]));
}

// Max with its arg-max, ties to the lowest node index (any combination order gives the same).
__device__ __forceinline__ void max_merge(float& mx, int32_t& am, float m2, int32_t a2) {
    if (m2 > mx || (m2 == mx && a2 < am)) {
        mx = m2;
        am = a2;
    }
}
template <int S>
__device__ __forceinline__ void max_halves(float& m, int32_t& a, float m2, int32_t a2) {
    unsigned int x = __float_as_uint(m), y = __float_as_uint(m2), i = static_cast<unsigned int>(a),
                 j = static_cast<unsigned int>(a2);
    swap_halves<S>(x, y);
    swap_halves<S>(i, j);
    m = __uint_as_float(x);
    a = static_cast<int32_t>(i);
    max_merge(m, a, __uint_as_float(y), static_cast<int32_t>(j));
}
// The result is left in mx[0], am[0].
template <int G>
__device__ __forceinline__ void reduce_groups_max(float (&mx)[4], int32_t (&am)[4]) {
    max_halves<2 * G>(mx[0], am[0], mx[1], am[1]);
    max_halves<2 * G>(mx[2], am[2], mx[3], am[3]);
    max_halves<G>(mx[0], am[0], mx[2], am[2]);
}

// Lane Q's value of each group of G lanes (16 or 8), by DPP row broadcasts (a DPP row is 16 lanes, a bank
// 4): a vector instruction or two where a shuffle goes through the LDS unit.
template <int Q, int G>
__device__ __forceinline__ int group_bcast(int v) {
    constexpr int kRowNewBcast = 0x150;
    if constexpr (G == 16) {
        return __builtin_amdgcn_update_dpp(0, v, kRowNewBcast + Q, 0xf, 0xf, true);
    } else {
        const int lo = __builtin_amdgcn_update_dpp(0, v, kRowNewBcast + Q, 0xf, 0x3, true);
        return __builtin_amdgcn_update_dpp(lo, v, kRowNewBcast + 8 + Q, 0xf, 0xc, false);
    }
}
template <int Q, int G>
__device__ __forceinline__ float group_bcast(float v) {
    return __builtin_bit_cast(float, group_bcast<Q, G>(__builtin_bit_cast(int, v)));
}

// Aggregation over the stored entries of rows of the batched graph with 16-byte gathers: group q of
// G = HD / 4 lanes (of the HD lanes that own rows [r0, r0 + 16)) owns the rows [r0 + 4 q, r0 + 4 q + 4)
// and lane p of the group holds channels 4 p .. 4 p + 3, so that one load instruction brings 64 / G
// neighbour rows. Each row's entries are visited in stored order. A group's lanes hold its next G
// entries (column, weight, row); eight gathers are in flight at a time, and the next entries load
// meanwhile. What is bound here is instructions and latency, not bytes, so the steps are straight-line
// code: entries are broadcast by DPP, a slot past the group's end has weight 0 and ends no row, and
// whether any group ends a row at a step is a scalar test of a mask formed once per G entries. rp is the
// lane's row pointer, ptr[g0 + min(p, 4)] of the group's first row g0; init() is called once the first
// entries are on their way. use(w, v) gets what load(column) returned; with PAIR, load brings two
// floats per node, which each lane then loads for the entry it holds (one load instruction per G entries
// instead of one per entry: the address units take a wavefront's lanes four a cycle, whatever they
// load). done(i) is called after the last entry of the group's row i = 0..3 and never for a row without
// entries (the caller presets those).
constexpr int kBatchX4 = 8;

template <int G, bool PAIR, class Init, class Load, class Use, class Done>
__device__ __forceinline__ void visit_rows_x4(int rp, const int32_t* __restrict__ col, const float* __restrict__ w,
                                              Init init, Load load, Use use, Done done) {
    static_assert(G == 16 || G == 8, "groups of 16 (64 channels) or 8 (32 channels) lanes");
    const int p = static_cast<int>(threadIdx.x % G);
    const int32_t b0 = group_bcast<0, G>(rp), b1 = group_bcast<1, G>(rp), b2 = group_bcast<2, G>(rp),
                  b3 = group_bcast<3, G>(rp), b4 = group_bcast<4, G>(rp);
    const int32_t last = max(b4 - 1, 0);
    int32_t longest = 0;  // entries of the wavefront's longest group
    static_for<64 / G>([&](auto q) { longest = max(longest, __builtin_amdgcn_readlane(b4 - b0, q * G)); });
    int32_t e = b0 + p;
    int cl = col[min(e, last)];
    float wl = w[min(e, last)];
    init();
    for (int32_t base = 0; base < longest; base += G, e += G) {
        const int ccur = cl;
        const float wcur = e < b4 ? wl : 0.0f;
        const int ri = (e >= b1) + (e >= b2) + (e >= b3);
        const int32_t rend = ri == 0 ? b1 : ri == 1 ? b2 : ri == 2 ? b3 : b4;
        const int info = e + 1 == rend ? 4 + ri : 0;
        const uint64_t ends = __builtin_amdgcn_ballot_w64(info != 0);
        if (base + G < longest) {
            cl = col[min(e + G, last)];
            wl = w[min(e + G, last)];
        }
        constexpr uint64_t kFirst = G == 16 ? 0x0001000100010001ull : 0x0101010101010101ull;
        float2 own = make_float2(0.0f, 0.0f);
        if constexpr (PAIR) own = load(ccur);
        static_for<G / kBatchX4>([&](auto half) {
            constexpr int H = half * kBatchX4;
            if (H > 0 && base + H >= longest) return;
            decltype(load(0)) vj[kBatchX4];
            if constexpr (!PAIR) static_for<kBatchX4>([&](auto q) { vj[q] = load(group_bcast<H + q, G>(ccur)); });
            static_for<kBatchX4>([&](auto q) {
                if (q > 0 && base + H + q >= longest) return;
                if constexpr (PAIR)
                    use(group_bcast<H + q, G>(wcur),
                        make_float2(group_bcast<H + q, G>(own.x), group_bcast<H + q, G>(own.y)));
                else
                    use(group_bcast<H + q, G>(wcur), vj[q]);
                if (ends & (kFirst << (H + q))) {
                    const int f = group_bcast<H + q, G>(info);
                    if (f != 0) done(f - 4);
                }
            });
        });
    }
}

// Whether one group of the wavefront has nearly all of its entries (rp as above): a hub row, whose group then
// has eight gathers in flight and the others none.
template <int G>
__device__ __forceinline__ bool one_group_walks(int rp) {
    const int32_t mine = group_bcast<4, G>(rp) - group_bcast<0, G>(rp);
    int32_t longest = 0, all = 0;
    static_for<64 / G>([&](auto q) {
        const int32_t n = __builtin_amdgcn_readlane(mine, q * G);
        longest = max(longest, n);
        all += n;
    });
    return longest > 512 && longest > all / 4 * 3;
}

// The same sums one row after the other, a channel per lane of the HD lanes that own rows [r0, r0 + 16), with
// HD / 2 gathers in flight: load(column) brings the lane's channel, put(i, sum) is called for every row. The
// sums are those of visit_rows_x4 bit for bit (stored order, fused products).
template <int HD, class Load, class Put>
__device__ __forceinline__ void visit_rows_one(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                               const float* __restrict__ w, int32_t r0, Load load, Put put) {
    constexpr int B = HD / 2;
    const int l = static_cast<int>(threadIdx.x % B);
    auto lane = [](auto v, int q) {
        if constexpr (HD == 64)
            return __builtin_bit_cast(decltype(v), __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), q));
        else
            return __shfl(v, q, HD);
    };
    for (int i = 0; i < 16; ++i) {
        const int32_t b = ptr[r0 + i], n = ptr[r0 + i + 1] - b;
        float sum = 0.0f;
        int cl = 0;
        float wl = 0.0f;
        if (n > 0) {
            cl = col[b + min(l, n - 1)];
            wl = w[b + min(l, n - 1)];
        }
        for (int32_t k = 0; k < n; k += B) {
            float v[B];
#pragma unroll
            for (int q = 0; q < B; ++q) v[q] = load(lane(cl, q));
            const float wcur = wl;
            if (k + B < n) {
                cl = col[b + min(k + B + l, n - 1)];
                wl = w[b + min(k + B + l, n - 1)];
            }
#pragma unroll
            for (int q = 0; q < B; ++q)
                if (k + q < n) sum += lane(wcur, q) * v[q];
        }
        put(i, sum);
    }
}

// Bounds of a group's rows for the callers of visit_rows_x4 that preset rows without entries.
template <class Empty>
__device__ __forceinline__ void for_empty_rows(const int32_t* __restrict__ ptr, int32_t g0, Empty empty) {
    for (int i = 0; i < 4; ++i)
        if (ptr[g0 + i] == ptr[g0 + i + 1]) empty(i);
}

// Sum over the 4 wavefronts of a workgroup, per channel (lane), into out[c] (thread wave 0).
template <int HD>
__device__ __forceinline__ double wave4_sum(double v, double (*sh)[HD]) {
    const int wv = threadIdx.x / HD, c = threadIdx.x % HD;
    sh[wv][c] = v;
    __syncthreads();
    const double s = sh[0][c] + sh[1][c] + sh[2][c] + sh[3][c];
    __syncthreads();
    return s;
}

// ------------------------------------------------------------------------------------------
// batch construction
// ------------------------------------------------------------------------------------------
// One launch builds the batched graph of every level: a workgroup owns one 64-row tile (four threads
// per row) and looks its graph's arrays up. It writes the rows' pointers and degree features (pad rows
// of a graph's last tile carry no entries), marks the rows' entries in an LDS map and copies the
// entries with unit stride (columns shifted to the graph's first batch row, weights a_ij, 1 for the
// self-loop of A_hat, whose entry also writes the a_ii feature). A copy: bound by memory on large
// levels, by the latency of its few dependent loads on small ones, which is why the levels share one
// launch (one launch per level of 256-row workgroups took 157 us on the hierarchy of 998k tetrahedral
// cells, 83 of them on levels below 25k rows, and 28 us more for the pad rows; this one takes 85). In a
// tile whose entries do not fit the map (more than 64 per row on average) an entry finds its row by
// bisection in the rows' ends (copied row by row, four threads each, a hub row of 5000 entries made the
// batch of its 20k-row graph 209 us; 37 so).
struct FillGraph {
    const int32_t* rp;
    const int32_t* cl;
    const double* va;
    int32_t n, row0, e0;  // rows; first batch row and first batch entry
};
constexpr int kFillCap = 4096;
constexpr int kFillChunk = 4;  // entries per thread whose loads are issued together

__global__ __launch_bounds__(256) void fill_graph_kernel(int ntiles, const int32_t* __restrict__ tile_graph,
                                                        const FillGraph* __restrict__ fg, int32_t* __restrict__ ptr,
                                                        int32_t* __restrict__ col, float* __restrict__ w,
                                                        float* __restrict__ x0) {
    __shared__ uint8_t rowof[kFillCap];
    __shared__ int32_t ends[TILE];  // of the rows' entries, from the tile's first entry
    const int t = static_cast<int>(threadIdx.x);
    const FillGraph g = fg[tile_graph[blockIdx.x]];
    const int32_t r0 = static_cast<int32_t>(blockIdx.x) * TILE - g.row0;  // rows of the level matrix
    const int32_t r1 = min(r0 + TILE, g.n);
    const int32_t b0 = g.rp[r0];
    const int32_t ne = g.rp[r1] - b0;
    const bool fits = ne <= kFillCap;
    const int lr = t / 4, q = t % 4;
    const int32_t i = r0 + lr;
    int32_t b = 0, e = 0;
    if (i < r1) {
        b = g.rp[i];
        e = g.rp[i + 1];
        if (fits)
            for (int32_t k = b - b0 + q; k < e - b0; k += 4) rowof[k] = static_cast<uint8_t>(lr);
    } else {
        b = e = g.rp[g.n];  // a pad row
    }
    if (q == 0) {
        ends[lr] = e - b0;
        ptr[g.row0 + i] = g.e0 + b;
        x0[2 * (g.row0 + i)] = 0.0f;  // a_ii; the diagonal entry writes it below
        x0[2 * (g.row0 + i) + 1] = i < r1 ? static_cast<float>(e - b - 1) : 0.0f;
        if (static_cast<int>(blockIdx.x) == ntiles - 1 && lr == TILE - 1) ptr[g.row0 + i + 1] = g.e0 + e;
    }
    __syncthreads();
    auto row_of = [&](int32_t k) -> int32_t {
        if (fits) return rowof[k];
        int32_t r = 0;  // rows that end at or before entry k
#pragma unroll
        for (int step = TILE / 2; step > 0; step /= 2)
            if (ends[r + step - 1] <= k) r += step;
        return r;
    };
    for (int32_t base = 0; base < ne; base += kFillChunk * 256) {
        int32_t j[kFillChunk];
        double a[kFillChunk];
#pragma unroll
        for (int u = 0; u < kFillChunk; ++u) {
            const int32_t p = b0 + min(base + t + u * 256, ne - 1);
            j[u] = g.cl[p];
            a[u] = g.va[p];
        }
#pragma unroll
        for (int u = 0; u < kFillChunk; ++u) {
            const int32_t k = base + t + u * 256;
            if (k < ne) {
                const int32_t row = r0 + row_of(k);
                col[g.e0 + b0 + k] = g.row0 + j[u];
                if (j[u] == row) {
                    w[g.e0 + b0 + k] = 1.0f;  // self-loop of A_hat
                    x0[2 * (g.row0 + row)] = static_cast<float>(a[u]);
                } else {
                    w[g.e0 + b0 + k] = static_cast<float>(a[u]);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// forward
// ------------------------------------------------------------------------------------------
// Output of layer 0 at a node from its two aggregated input features h = (A_hat x0)_i:
// y_c = b0_c + h0 W0[0][c] + h1 W0[1][c]. The input features span two dimensions, so y is never
// stored: every consumer (the layer's statistics and pooling, layer 1's aggregation, the
// backward) forms it from h with this one expression, 8 bytes per node instead of 4 HD.
__device__ __forceinline__ float y0_of(float2 h, float w0, float w1, float bb) {
    return __builtin_fmaf(h.y, w1, __builtin_fmaf(h.x, w0, bb));
}

__device__ __forceinline__ float4 y0_of4(float2 h, const float4& w0, const float4& w1, const float4& bb) {
    return make_float4(y0_of(h, w0.x, w1.x, bb.x), y0_of(h, w0.y, w1.y, bb.y), y0_of(h, w0.z, w1.z, bb.z),
                       y0_of(h, w0.w, w1.w, bb.w));
}

// Layer 0 of a tile: H0 = A_hat x0 (two features per node; 4 HD / 64 lanes per row, each summing
// every such entry of the row, combined in a fixed butterfly) and the per-tile sums of y and
// y^2 for the InstanceNorm statistics.
template <int HD>
__global__ __launch_bounds__(4 * HD) void layer0_kernel(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                    const float* __restrict__ w, const float* __restrict__ x0,
                                                    const int32_t* __restrict__ tile_graph,
                                                    const int32_t* __restrict__ gend, const float* __restrict__ W0,
                                                    const float* __restrict__ b0, float* __restrict__ H0,
                                                    double* __restrict__ tstat) {
    constexpr int LPR = 4 * HD / TILE;
    __shared__ double sh[4][HD];
    __shared__ float2 hs[TILE];
    const int tile = blockIdx.x, wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int32_t end = gend[tile_graph[tile]];
    {
        const int lr = threadIdx.x / LPR, q = threadIdx.x % LPR;
        const int32_t row = tile * TILE + lr;
        float h0 = 0.0f, h1 = 0.0f;
        if (row < end) {
            const int32_t pe = ptr[row + 1];
            for (int32_t k = ptr[row] + q; k < pe; k += LPR) {
                const float wk = w[k];
                const float2 xv = *reinterpret_cast<const float2*>(x0 + 2 * static_cast<int64_t>(col[k]));
                h0 = __builtin_fmaf(wk, xv.x, h0);
                h1 = __builtin_fmaf(wk, xv.y, h1);
            }
        }
#pragma unroll
        for (int off = 1; off < LPR; off <<= 1) {
            h0 += __shfl_xor(h0, off, LPR);
            h1 += __shfl_xor(h1, off, LPR);
        }
        if (q == 0) {
            const float2 hv = make_float2(h0, h1);
            hs[lr] = hv;
            reinterpret_cast<float2*>(H0)[row] = hv;
        }
    }
    __syncthreads();
    const float w0 = W0[c], w1 = W0[HD + c], bb = b0[c];
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int lr = wv * 16 + r;
        if (tile * TILE + lr < end) {
            const float y = y0_of(hs[lr], w0, w1, bb);
            s1 += y;
            s2 += static_cast<double>(y) * y;
        }
    }
    s1 = wave4_sum(s1, sh);
    s2 = wave4_sum(s2, sh);
    if (wv == 0) {
        tstat[tile * 2 * HD + c] = s1;
        tstat[tile * 2 * HD + HD + c] = s2;
    }
}

// y (64 values of `rows` in LDS tile A[64][65]) times B (64 x 64) -> D tile [64][65] in LDS.
// FP32: lane c computes column c. BF16: v_mfma_f32_16x16x32_bf16 on the wavefront's 16 rows;
// Bt is the bf16 copy of B stored [col][k] (k contiguous) in LDS.
//
// SPLIT: A is passed as a_hi + a_lo, two bf16 numbers (16 significant bits), with one MFMA
// each. The aggregated features of a GCIN layer have a per-graph mean that is large next to
// their spread across nodes (the raw features a_ii, deg(i) are not centred), and the
// InstanceNorm that follows subtracts that mean: rounding each node's A row to a single bf16
// would be amplified by |A| / std(A) in the normalised output. Rounding of the weights is
// not amplified (it moves the mean and the rows alike), so B stays single bf16.
__device__ __forceinline__ void split_bf16(float x, unsigned short& hi, unsigned short& lo) {
    hi = f2bf(x);
    lo = f2bf(x - __uint_as_float(static_cast<unsigned int>(hi) << 16));
}

// The same for two (finite) numbers by the packed conversion, which rounds to nearest even as f2bf
// does, in a third of the instructions.
__device__ __forceinline__ void split_bf16_pair(float x0, float x1, unsigned int& hi, unsigned int& lo) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    hi = __builtin_bit_cast(unsigned int, __builtin_convertvector((f32x2{x0, x1}), bf16x2));
    const f32x2 r{x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xFFFF0000u)};
    lo = __builtin_bit_cast(unsigned int, __builtin_convertvector(r, bf16x2));
}

// D = A B, a group of HD lanes its 16 rows. FP32: B from memory (Bf); MFMA: bf16 parts of both (B as Bt).
template <int HD, bool MFMA, int LD = HD + 1>
__device__ __forceinline__ void tile_gemm(const float (*A)[LD], const float* __restrict__ Bf,
                                          const unsigned short (*Bt)[HD + 8], float (*D)[LD]) {
    static_assert(!MFMA || HD == 64, "the MFMA tiling is written for 64 channels");
    const int wv = threadIdx.x / HD, lane = threadIdx.x % HD;
    if constexpr (!MFMA) {
        // column `lane` of B in registers, 32 rows of it at a time, and the rows of A as broadcasts
        float acc[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
        for (int k0 = 0; k0 < HD; k0 += 32) {
            float bc[32];
#pragma unroll
            for (int k = 0; k < 32; ++k) bc[k] = Bf[(k0 + k) * HD + lane];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float* ar = &A[wv * 16 + r][k0];
                if constexpr (LD % 4 == 0) {
#pragma unroll
                    for (int k = 0; k < 32; k += 4) {
                        const float4 a = *reinterpret_cast<const float4*>(ar + k);
                        acc[r] += a.x * bc[k];
                        acc[r] += a.y * bc[k + 1];
                        acc[r] += a.z * bc[k + 2];
                        acc[r] += a.w * bc[k + 3];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 32; ++k) acc[r] += ar[k] * bc[k];
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) D[wv * 16 + r][lane] = acc[r];
    } else {
        const int i = lane % 16, kq = (lane / 16) * 8;
        f32x4 acc[4];
        for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int ks = 0; ks < HD; ks += 32) {
            u16x8 av;
            for (int e = 0; e < 8; ++e) av[e] = f2bf(A[wv * 16 + i][ks + kq + e]);
            const bf16x8 a = __builtin_bit_cast(bf16x8, av);
            for (int nb = 0; nb < 4; ++nb) {
                u16x8 bv;
                for (int e = 0; e < 8; ++e) bv[e] = Bt[nb * 16 + i][ks + kq + e];
                const bf16x8 b = __builtin_bit_cast(bf16x8, bv);
                acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[nb], 0, 0, 0);
            }
        }
        for (int nb = 0; nb < 4; ++nb)
            for (int e = 0; e < 4; ++e) D[wv * 16 + (lane / 16) * 4 + e][nb * 16 + i] = acc[nb][e];
    }
}

// The wavefront's 16 rows of A (64 channels, LD apart) times B on MFMA, A split as above: acc[nb][e] is the
// row 4 (lane / 16) + e and the column 4 (lane % 16) + nb, so that a lane's four blocks are neighbouring
// columns. B's bf16 hi parts and its lo parts (added with SPLITB) are read from global memory,
// [column][k] (formed once per forward by weights_bf16_kernel): every tile shares them, so they
// stay in cache and take no LDS. SPLITB: a_hi b_lo is added as well (a_lo b_lo is below FP32
// resolution): an FP32-accurate product on the BF16 MFMA units, used where the result feeds
// non-smooth operations (ReLU masks, arg-max pooling) whose gradients must match an FP32/FP64
// evaluation.
template <int HD, bool SPLITB, int LD>
__device__ __forceinline__ void tile_product(const float (*A)[LD], const unsigned short* __restrict__ Bg,
                                             f32x4 (&acc)[4]) {
    static_assert(HD == 64, "the MFMA tiling is written for 64 channels");
    const int wv = threadIdx.x / HD, lane = threadIdx.x % HD;
    const int i = lane % 16, kq = (lane / 16) * 8;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < HD; ks += 32) {
        const float* ar = &A[wv * 16 + i][ks + kq];
        const f32x4 a0 = *reinterpret_cast<const f32x4*>(ar), a1 = *reinterpret_cast<const f32x4*>(ar + 4);
        u32x4 av, alv;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            unsigned int h, l;
            split_bf16_pair(a0[2 * e], a0[2 * e + 1], h, l);
            av[e] = h;
            alv[e] = l;
            split_bf16_pair(a1[2 * e], a1[2 * e + 1], h, l);
            av[2 + e] = h;
            alv[2 + e] = l;
        }
        const bf16x8 a = __builtin_bit_cast(bf16x8, av), al = __builtin_bit_cast(bf16x8, alv);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const unsigned short* bp = Bg + (4 * i + nb) * HD + ks + kq;
            const bf16x8 b = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(bp));
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[nb], 0, 0, 0);
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b, acc[nb], 0, 0, 0);
            if constexpr (SPLITB) {
                const bf16x8 bl = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(bp + HD * HD));
                acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc[nb], 0, 0, 0);
            }
        }
    }
}

// bf16 copy of a 64 x 64 FP32 matrix M (row-major) for tile_gemm's product with M^T.
template <int HD>
__device__ __forceinline__ void stage_bf16(const float* __restrict__ M, unsigned short (*Bt)[HD + 8]) {
    for (int e = threadIdx.x; e < HD * HD; e += 4 * HD) Bt[e / HD][e % HD] = f2bf(M[e]);
}

// Entry e of the weights W ([k][col]) as tile_product reads them: bf16 hi part at [col][k], lo part HD^2 on.
template <int HD>
__device__ __forceinline__ void weight_parts(const float* __restrict__ W, int e, unsigned short* hi) {
    const int k = e / HD, c = e % HD;
    unsigned short h, lo;
    split_bf16(W[e], h, lo);
    hi[c * HD + k] = h;
    hi[HD * HD + c * HD + k] = lo;
}

// bf16 hi / lo parts of the 64 x 64 weights of layers 1 .. NL-1, transposed ([col][k]) for
// tile_product: blocks (l - 1, *) form layer l into wbf + (l - 1) 2 HD^2 (hi) and
// the HD^2 entries after it (lo). One element per thread: with one workgroup per layer its 16 rounds
// of dependent loads took 13 us, spread over 16 workgroups 3.
template <int HD>
__global__ __launch_bounds__(256) void weights_bf16_kernel(const float* __restrict__ P, Offs o,
                                                         unsigned short* __restrict__ wbf) {
    const int l = blockIdx.x + 1;
    const float* W = P + o.convW[l];
    unsigned short* hi = wbf + static_cast<int64_t>(blockIdx.x) * 2 * HD * HD;
    const int e = static_cast<int>(blockIdx.y) * 256 + threadIdx.x;
    if (e >= HD * HD) return;
    weight_parts<HD>(W, e, hi);
}

// Tile of a workgroup. Workgroups go to the 8 XCDs in turn, each with an L2 of its own: within every 256
// tiles an XCD takes 32 neighbouring ones, whose rows gather mostly each other's neighbours (layers of
// the 998k-cell hierarchy 476 -> 457 us). One contiguous range per XCD would give one of them the
// coarse levels with their long rows.
__device__ __forceinline__ int dealt_tile() {
    constexpr int kRun = 32, kXcd = 8;
    const int b = blockIdx.x, r = b % (kRun * kXcd), base = b - r;
    if (base + kRun * kXcd > static_cast<int>(gridDim.x)) return b;  // the last, partial 256
    return base + (r % kXcd) * kRun + r / kXcd;
}

// A layer above the first, one tile per workgroup. Layer 1, whose input is formed from 8 bytes per node,
// is bound by the vector instructions of the walk (23 an entry, of which 16 normalise it; 95 % busy);
// the others by the gathers' traffic from the L2s (256 bytes an entry at about 9 TB/s). On the
// 998k-cell hierarchy (1.64M nodes, 14.5M entries) layer 1 went from 468 to 360 us and the others from
// 500 to 462 against a form that passed the batch's entries through LDS shuffles, kept the rows' own
// inputs in LDS and summed the tile one row at a time.
// Y0: the layer below is layer 0, whose output is formed from H0 (y0_of) instead of read from Yp. Off: type
// of the byte offsets into Yp (32 bits where they suffice).
template <int HD, bool MFMA, bool X3, bool Y0, typename Off>
__global__ __launch_bounds__(4 * HD, MFMA && (Y0 || X3) ? 5 : 4) void layer_kernel(
                                                   const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                   const float* __restrict__ w, const int32_t* __restrict__ tile_graph,
                                                   const int32_t* __restrict__ gend, const float* __restrict__ Yp,
                                                   const float* __restrict__ H0, const float* __restrict__ W0,
                                                   const float* __restrict__ b0,
                                                   const float* __restrict__ mup, const float* __restrict__ rsp,
                                                   const float* __restrict__ gam, const float* __restrict__ bet,
                                                   const float* __restrict__ W, const float* __restrict__ b,
                                                   const unsigned short* __restrict__ wbf,
                                                   float* __restrict__ Hout, float* __restrict__ Y,
                                                   double* __restrict__ tstat, double* __restrict__ psum,
                                                   float* __restrict__ pmax, int32_t* __restrict__ parg) {
    // The kernel also forms the per-tile readout partials of the layer below (psum / pmax / parg
    // as pool_tile_kernel writes them) from the tile's own rows of that layer, which the gathers have
    // just brought into cache, so the layer below needs no pooling pass.
    // The product overwrites the aggregates in place: every group of HD lanes reads only its own 16
    // rows of Hs and writes the same rows, each output after all of its row's reads (the
    // stores depend on them), so one tile buffer serves both and the wavefronts of a tile meet only
    // at the end, when the buffer takes the per-tile reductions.
    constexpr int LD = HD + 4;  // rows stay aligned to 16 bytes
    __shared__ __align__(16) float Hs[TILE][LD];  // aggregates, products, then the reductions
    constexpr int G = HD / 4;
    const int tile = dealt_tile(), wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int32_t r0 = tile * TILE + wv * 16;
    const int32_t g0 = r0 + 4 * (c / G);  // the first row of the lane's group (see visit_rows_x4)
    const int rp = ptr[g0 + min(static_cast<int>(threadIdx.x % G), 4)];  // first in the chain of loads
    const int g = tile_graph[tile];
    const int32_t end = gend[g];
    const int c4 = 4 * static_cast<int>(threadIdx.x % G);  // the lane's channels: c4 .. c4 + 3
    float* const hs = &Hs[g0 - tile * TILE][c4];
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(hs + i * LD) = make_float4(0.f, 0.f, 0.f, 0.f);
    if (Hout)
        for_empty_rows(ptr, g0, [&](int i) {
            *reinterpret_cast<float4*>(Hout + static_cast<int64_t>(g0 + i) * HD + c4) = make_float4(0.f, 0.f, 0.f, 0.f);
        });
    float4 mu4, rs4, ga4, be4;
    float4 w04 = make_float4(0.f, 0.f, 0.f, 0.f), w14 = w04, bb4 = w04;
    float4 h4 = make_float4(0.f, 0.f, 0.f, 0.f);
    visit_rows_x4<G, Y0>(
        rp, col, w,
        [&] {
            mu4 = *reinterpret_cast<const float4*>(mup + g * HD + c4);
            rs4 = *reinterpret_cast<const float4*>(rsp + g * HD + c4);
            ga4 = *reinterpret_cast<const float4*>(gam + c4);
            be4 = *reinterpret_cast<const float4*>(bet + c4);
            if constexpr (Y0) {
                w04 = *reinterpret_cast<const float4*>(W0 + c4);
                w14 = *reinterpret_cast<const float4*>(W0 + HD + c4);
                bb4 = *reinterpret_cast<const float4*>(b0 + c4);
            }
        },
        [&](int32_t j) {
            if constexpr (Y0) {
                return reinterpret_cast<const float2*>(H0)[j];
            } else {
                const Off at = static_cast<Off>(j) * (HD * 4) + c4 * 4;
                return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(Yp) + at);
            }
        },
        [&](float wp, const auto& in) {
            float4 v;
            if constexpr (Y0)
                v = make_float4(y0_of(in, w04.x, w14.x, bb4.x), y0_of(in, w04.y, w14.y, bb4.y),
                                y0_of(in, w04.z, w14.z, bb4.z), y0_of(in, w04.w, w14.w, bb4.w));
            else
                v = in;
            h4.x += wp * normrelu(v.x, mu4.x, rs4.x, ga4.x, be4.x);
            h4.y += wp * normrelu(v.y, mu4.y, rs4.y, ga4.y, be4.y);
            h4.z += wp * normrelu(v.z, mu4.z, rs4.z, ga4.z, be4.z);
            h4.w += wp * normrelu(v.w, mu4.w, rs4.w, ga4.w, be4.w);
        },
        [&](int i) {
            *reinterpret_cast<float4*>(hs + i * LD) = h4;
            if (Hout) *reinterpret_cast<float4*>(Hout + static_cast<int64_t>(g0 + i) * HD + c4) = h4;
            h4 = make_float4(0.f, 0.f, 0.f, 0.f);
        });
    // From here on a lane holds the same rows g0 .. g0 + 3 and channels c4 .. c4 + 3 as in the walk:
    // the product's column block nb covers the channels 4 i + nb, so that its 16 results per lane
    // are four rows of four neighbouring channels.
    float4 xv[4];  // the rows' own inputs, loaded while the product runs
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (Y0)
            xv[e] = y0_of4(reinterpret_cast<const float2*>(H0)[g0 + e], w04, w14, bb4);
        else
            xv[e] = *reinterpret_cast<const float4*>(Yp + static_cast<int64_t>(g0 + e) * HD + c4);
    }
    const float4 b4 = *reinterpret_cast<const float4*>(b + c4);
    wave_sync();
    float4 yv[4];
    if constexpr (MFMA) {
        f32x4 acc[4];
        tile_product<HD, X3, LD>(Hs, wbf, acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) yv[e] = make_float4(acc[0][e], acc[1][e], acc[2][e], acc[3][e]);
    } else {
        tile_gemm<HD, false, LD>(Hs, W, nullptr, Hs);
        wave_sync();
#pragma unroll
        for (int e = 0; e < 4; ++e) yv[e] = *reinterpret_cast<const float4*>(hs + e * LD);
    }
    // y of the lane's rows, the sums of y and y^2 and the readout partials of the layer below (sum,
    // max and first arg-max of x per channel): over the lane's rows, then the 16 rows of the HD
    // lanes, then the tile, in a fixed order
    double s1[4] = {}, s2[4] = {}, ps[4] = {};
    float mx[4];
    int32_t am[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        mx[k] = -INFINITY;
        am[k] = INT32_MAX;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int32_t row = g0 + e;
        const bool ok = row < end;
        const float y[4] = {ok ? yv[e].x + b4.x : 0.0f, ok ? yv[e].y + b4.y : 0.0f, ok ? yv[e].z + b4.z : 0.0f,
                            ok ? yv[e].w + b4.w : 0.0f};
        const float x[4] = {normrelu(xv[e].x, mu4.x, rs4.x, ga4.x, be4.x), normrelu(xv[e].y, mu4.y, rs4.y, ga4.y, be4.y),
                            normrelu(xv[e].z, mu4.z, rs4.z, ga4.z, be4.z), normrelu(xv[e].w, mu4.w, rs4.w, ga4.w, be4.w)};
        *reinterpret_cast<float4*>(Y + static_cast<int64_t>(row) * HD + c4) = make_float4(y[0], y[1], y[2], y[3]);
        if (!ok) continue;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s1[k] += y[k];
            s2[k] += static_cast<double>(y[k]) * y[k];
            ps[k] += x[k];
            if (x[k] > mx[k]) {
                mx[k] = x[k];
                am[k] = row;
            }
        }
    }
    const int cc = c4 + reduced_channel<G>();
    const double t1 = reduce_groups<G>(s1), t2 = reduce_groups<G>(s2), tp = reduce_groups<G>(ps);
    reduce_groups_max<G>(mx, am);
    // each group of HD lanes puts its partials where its rows of the tile were, once all its lanes have read
    // them; the first adds them up in order
    wave_sync();
    auto part = [&](int k) { return reinterpret_cast<double*>(&Hs[16 * k][0]); };
    static_assert(16 * LD * sizeof(float) >= HD * (3 * sizeof(double) + sizeof(float) + sizeof(int32_t)), "they fit");
    {
        double* r = part(wv);
        r[cc] = t1;
        r[HD + cc] = t2;
        r[2 * HD + cc] = tp;
        float* rm = reinterpret_cast<float*>(r + 3 * HD);
        rm[cc] = mx[0];
        reinterpret_cast<int32_t*>(rm + HD)[cc] = am[0];
    }
    __syncthreads();
    if (wv == 0) {
        tstat[tile * 2 * HD + c] = part(0)[c] + part(1)[c] + part(2)[c] + part(3)[c];
        tstat[tile * 2 * HD + HD + c] = part(0)[HD + c] + part(1)[HD + c] + part(2)[HD + c] + part(3)[HD + c];
        psum[tile * HD + c] = part(0)[2 * HD + c] + part(1)[2 * HD + c] + part(2)[2 * HD + c] + part(3)[2 * HD + c];
        float m = -INFINITY;
        int32_t a = INT32_MAX;
        for (int k = 0; k < 4; ++k) {
            const float* rm = reinterpret_cast<const float*>(part(k) + 3 * HD);
            max_merge(m, a, rm[c], reinterpret_cast<const int32_t*>(rm + HD)[c]);
        }
        pmax[tile * HD + c] = m;
        parg[tile * HD + c] = a;
    }
}

// Per-graph reductions over tiles run in two fixed-order stages so that large graphs (the fine
// level has n/64 tiles) are spread over many workgroups: stage 1 sums the tiles of each chunk
// (at most kChunkTiles consecutive tiles of one graph, chunks counted from the graph's first
// tile), stage 2 the chunks of each graph. In both, group w of the workgroup's kSumGroups groups of HD lanes
// sums items w, w + kSumGroups, ... in order and the groups' sums are added in group order:
// deterministic, and a graph's result does not depend on the other graphs of the batch. The loads decide the
// time, so kAhead items' loads are issued together, all that a full chunk gives a group (with 4 groups a chunk
// took four such rounds, 7.5 us against 4.7 on 625 tiles of 32 channels), and what can be summed apart
// (y, y^2, the readout, the backward's four sums; blockIdx.y) gets its own workgroup. The statistics of
// a layer and the readout of the layer below it share their launches, and where every graph is one
// chunk, stage 1 finishes it and there is no stage 2. On the 998k-cell hierarchy the forward's
// reductions went from 16 launches and 180 us to 10 and 92, on the 32-mesh training batch from 16 and
// 130 to 5 and 44, the backward's sums from 8 and 48 to 4 and 33.
constexpr int kChunkTiles = 256;
constexpr int kAhead = 16;
constexpr int kSumGroups = 16;

// Sum of in[i][c] over the items i0 <= i < i1 as above, rows `stride` apart; valid in group 0.
template <int HD>
__device__ __forceinline__ double sum_items(const double* __restrict__ in, int64_t stride, int32_t i0, int32_t i1,
                                            int wv, int c, double (*sh)[HD]) {
    double s = 0.0;
    for (int32_t i = i0 + wv; i < i1; i += kSumGroups * kAhead) {
        double v[kAhead];  // a slot past the end re-reads the last item and is not used
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = in[min(i + kSumGroups * u, i1 - 1) * stride + c];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (i + kSumGroups * u < i1) s += v[u];
    }
    sh[wv][c] = s;
    __syncthreads();
    if (wv != 0) return s;
#pragma unroll
    for (int w = 1; w < kSumGroups; ++w) s += sh[w][c];
    return s;
}

// Mean and 1/sqrt(biased variance + eps) of a graph's channel from its sums of y and y^2.
__device__ __forceinline__ void norm_of(double s1, double s2, double n, float* mu, float* rstd) {
    const double m = s1 / n;
    double var = s2 / n - m * m;
    if (var < 0.0) var = 0.0;
    *mu = static_cast<float>(m);
    *rstd = static_cast<float>(1.0 / sqrt(var + static_cast<double>(kEps)));
}

// Sum, max and arg-max over the items as sum_items takes them; valid in group 0.
template <int HD>
__device__ __forceinline__ void pool_items(const double* __restrict__ isum, const float* __restrict__ imax,
                                           const int32_t* __restrict__ iarg, int32_t i0, int32_t i1, int wv, int c,
                                           double& s, float& mx, int32_t& am) {
    __shared__ double ss[kSumGroups][HD];
    __shared__ float sm[kSumGroups][HD];
    __shared__ int32_t sa[kSumGroups][HD];
    s = 0.0;
    mx = -INFINITY;
    am = INT32_MAX;
    for (int32_t i = i0 + wv; i < i1; i += kSumGroups * kAhead) {
        double vs[kAhead];
        float vm[kAhead];
        int32_t va[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t e = static_cast<int64_t>(min(i + kSumGroups * u, i1 - 1)) * HD + c;
            vs[u] = isum[e];
            vm[u] = imax[e];
            va[u] = iarg[e];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (i + kSumGroups * u < i1) {
                s += vs[u];
                max_merge(mx, am, vm[u], va[u]);
            }
    }
    ss[wv][c] = s;
    sm[wv][c] = mx;
    sa[wv][c] = am;
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int w = 1; w < kSumGroups; ++w) {
        s += ss[w][c];
        max_merge(mx, am, sm[w][c], sa[w][c]);
    }
}

// What a reduction of the forward takes and writes: the statistics of layer `layer` (stats) and the
// readout of layer `layer` - 1 or of the last layer (pool).
struct Reduce {
    const double* tstat;  // per tile (stage 1) or chunk (stage 2)
    const double* psum;
    const float* pmax;
    const int32_t* parg;
    double* cstat;        // stage 1: per chunk
    double* csum;
    float* cmax;
    int32_t* carg;
    const float* gcnt;    // the stage that finishes: per graph
    float *mu, *rstd, *pooled;
    int32_t* argmax;
    int pool_layer;
};

// FINAL: blockIdx.x is a graph and the items are its own (its tiles where it is one chunk, else its
// chunks); otherwise a chunk and its tiles. blockIdx.y + first selects the part: 0 = statistics (the
// first stage takes y and y^2 apart, 0 and 1), then the readout.
template <int HD, bool FINAL>
__global__ __launch_bounds__(kSumGroups * HD) void reduce_kernel(const int32_t* __restrict__ bounds, Reduce r, int first) {
    __shared__ double sh[2][kSumGroups][HD];
    constexpr int NSTAT = FINAL ? 1 : 2;
    const int k = blockIdx.x, wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int part = blockIdx.y + first;
    const int32_t i0 = bounds[k], i1 = bounds[k + 1];
    if (part < NSTAT) {
        if constexpr (FINAL) {
            const double s1 = sum_items<HD>(r.tstat, 2 * HD, i0, i1, wv, c, sh[0]);
            const double s2 = sum_items<HD>(r.tstat + HD, 2 * HD, i0, i1, wv, c, sh[1]);
            if (wv == 0) norm_of(s1, s2, r.gcnt[k], r.mu + k * HD + c, r.rstd + k * HD + c);
        } else {
            const double s = sum_items<HD>(r.tstat + part * HD, 2 * HD, i0, i1, wv, c, sh[0]);
            if (wv == 0) r.cstat[(static_cast<int64_t>(k) * 2 + part) * HD + c] = s;
        }
    } else {
        double s;
        float mx;
        int32_t am;
        pool_items<HD>(r.psum, r.pmax, r.parg, i0, i1, wv, c, s, mx, am);
        if (wv != 0) return;
        if constexpr (FINAL) {
            r.pooled[(k * NL + r.pool_layer) * 2 * HD + c] = static_cast<float>(s / r.gcnt[k]);
            r.pooled[(k * NL + r.pool_layer) * 2 * HD + HD + c] = mx;
            r.argmax[(k * NL + r.pool_layer) * HD + c] = am;
        } else {
            r.csum[static_cast<int64_t>(k) * HD + c] = s;
            r.cmax[static_cast<int64_t>(k) * HD + c] = mx;
            r.carg[static_cast<int64_t>(k) * HD + c] = am;
        }
    }
}

// The sums of the backward's four quantities j = blockIdx.y over a graph (FINAL) or a chunk, as above:
// out[k][j][c], or per graph the means of dxhat and dxhat*xhat (j = 0, 1) and the gamma / beta
// gradients (j = 2, 3).
template <int HD, bool FINAL>
__global__ __launch_bounds__(kSumGroups * HD) void bwd_sum_kernel(const double* __restrict__ in,
                                                                  const int32_t* __restrict__ bounds,
                                                                  double* __restrict__ out,
                                                                  const float* __restrict__ gcnt,
                                                                  float* __restrict__ gmean, double* __restrict__ ggb) {
    __shared__ double sh[kSumGroups][HD];
    const int k = blockIdx.x, j = blockIdx.y, wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const double s = sum_items<HD>(in + j * HD, 4 * HD, bounds[k], bounds[k + 1], wv, c, sh);
    if (wv != 0) return;
    if constexpr (!FINAL)
        out[(static_cast<int64_t>(k) * 4 + j) * HD + c] = s;
    else if (j < 2)
        gmean[(k * 2 + j) * HD + c] = static_cast<float>(s / gcnt[k]);
    else
        ggb[(k * 2 + j - 2) * HD + c] = s;
}

// Per tile: sum, max and first arg-max of x = ReLU(IN(y)) per channel (the last layer's readout).
template <int HD>
__global__ __launch_bounds__(4 * HD) void pool_tile_kernel(const int32_t* __restrict__ tile_graph,
                                                       const int32_t* __restrict__ gend, const float* __restrict__ Y,
                                                       const float* __restrict__ mu, const float* __restrict__ rstd,
                                                       const float* __restrict__ gam, const float* __restrict__ bet,
                                                       double* __restrict__ tsum, float* __restrict__ tmax,
                                                       int32_t* __restrict__ targ) {
    __shared__ double sh[4][HD];
    __shared__ float smax[4][HD];
    __shared__ int32_t sarg[4][HD];
    const int tile = blockIdx.x, wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int g = tile_graph[tile];
    const int32_t end = gend[g];
    const float m = mu[g * HD + c], rs = rstd[g * HD + c], ga = gam[c], be = bet[c];
    double s = 0.0;
    float mx = -INFINITY;
    int32_t am = INT32_MAX;
    float yv[16];  // the 16 rows' loads are issued together
    const int32_t r0 = tile * TILE + wv * 16;
#pragma unroll
    for (int r = 0; r < 16; ++r) yv[r] = r0 + r < end ? Y[static_cast<int64_t>(r0 + r) * HD + c] : 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int32_t row = tile * TILE + wv * 16 + r;
        if (row < end) {
            const float x = normrelu(yv[r], m, rs, ga, be);
            s += x;
            if (x > mx) {
                mx = x;
                am = row;
            }
        }
    }
    smax[wv][c] = mx;
    sarg[wv][c] = am;
    s = wave4_sum(s, sh);
    if (wv == 0) {
        for (int k = 1; k < 4; ++k)
            if (smax[k][c] > mx) {
                mx = smax[k][c];
                am = sarg[k][c];
            }
        tsum[tile * HD + c] = s;
        tmax[tile * HD + c] = mx;
        targ[tile * HD + c] = am;
    }
}

__device__ __forceinline__ float block128_sum(float v, float* red) {
    // 128 threads
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = 64; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    const float r = red[0];
    __syncthreads();
    return r;
}

struct HeadSave {
    float* z;    // [G][128] readout concatenation
    float* ln;   // [G][2]   mean, rstd
    float* s;    // [G][128] sigmoid output
    float* a1;   // [G][128]
    float* a2;   // [G][64]
};

// Readout, LayerNorm, sigmoid and predictive MLP of one graph per workgroup (128 threads).
// Each output is one sequential sum over weights in memory: 32 of its loads are issued together.
template <int HD>
__global__ __launch_bounds__(128) void head_fwd_kernel(const float* __restrict__ P, Offs o,
                                                       const float* __restrict__ pooled, HeadSave hs,
                                                       float* __restrict__ out) {
    __shared__ float p[NL * 2 * HD], z[JK], s[JK], a1[M1], a2[M2], red[128];
    const int g = blockIdx.x, t = threadIdx.x;
    for (int k = t; k < NL * 2 * HD; k += 128) p[k] = pooled[g * NL * 2 * HD + k];
    __syncthreads();
    {
        const int l = t / RO, oo = t % RO;
        float acc = P[o.rob[l] + oo];
#pragma unroll 32
        for (int k = 0; k < 2 * HD; ++k) acc += p[l * 2 * HD + k] * P[o.roW[l] + k * RO + oo];
        z[t] = acc;
    }
    __syncthreads();
    const float m = block128_sum(z[t], red) / JK;
    const float dz = z[t] - m;
    const float v = block128_sum(dz * dz, red) / JK;
    const float rs = 1.0f / sqrtf(v + kEps);
    const float zn = dz * rs * P[o.lng + t] + P[o.lnb + t];
    s[t] = 1.0f / (1.0f + expf(-zn));
    __syncthreads();
    {
        float acc = P[o.m0b + t];
#pragma unroll 32
        for (int k = 0; k < JK; ++k) acc += s[k] * P[o.m0W + k * M1 + t];
        a1[t] = fmaxf(acc, 0.0f);
    }
    __syncthreads();
    if (t < M2) {
        float acc = P[o.m1b + t];
#pragma unroll 32
        for (int k = 0; k < M1; ++k) acc += a1[k] * P[o.m1W + k * M2 + t];
        a2[t] = fmaxf(acc, 0.0f);
    }
    __syncthreads();
    if (t < o.nout) {
        float acc = P[o.m2b + t];
#pragma unroll 32
        for (int k = 0; k < M2; ++k) acc += a2[k] * P[o.m2W + k * o.nout + t];
        out[g * o.nout + t] = acc;
    }
    hs.z[g * JK + t] = z[t];
    hs.s[g * JK + t] = s[t];
    hs.a1[g * M1 + t] = a1[t];
    if (t < M2) hs.a2[g * M2 + t] = a2[t];
    if (t == 0) {
        hs.ln[2 * g] = m;
        hs.ln[2 * g + 1] = rs;
    }
}

// ------------------------------------------------------------------------------------------
// backward
// ------------------------------------------------------------------------------------------
// acc + sum_q d[q] w[q], q in order, w in memory: 16-byte loads, issued together.
template <int N>
__device__ __forceinline__ float row_dot(const float* d, const float* __restrict__ w, float acc) {
    float4 v[N / 4];
#pragma unroll
    for (int q = 0; q < N / 4; ++q) v[q] = reinterpret_cast<const float4*>(w)[q];
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {
        acc += d[4 * q] * v[q].x;
        acc += d[4 * q + 1] * v[q].y;
        acc += d[4 * q + 2] * v[q].z;
        acc += d[4 * q + 3] * v[q].w;
    }
    return acc;
}

// Head backward of one graph; writes this graph's head-parameter gradients (relative to
// o.head0) into gh[g][*] and the pooled-feature gradients into dpooled[g]. Bound by the chain of products
// with the transposed weights, where every thread reads a row of its own, by 16 bytes, and the parameter
// gradients, outer products whose column stays a thread's own, by 16 rows at a time (153 graphs: 28 us with
// both by single floats, 19 here).
template <int HD>
__global__ __launch_bounds__(128) void head_bwd_kernel(const float* __restrict__ P, Offs o,
                                                       const float* __restrict__ pooled, HeadSave hs,
                                                       const float* __restrict__ dout, float* __restrict__ gh,
                                                       int64_t ghstride, float* __restrict__ dpooled) {
    __shared__ float p[NL * 2 * HD], s[JK], a1[M1], a2[M2], d2[M2], d1[M1], dzv[JK], red[128], dov[kMaxOut];
    const int g = blockIdx.x, t = threadIdx.x;
    float* const gbase = gh + g * ghstride;
    auto G = [&](int64_t off) -> float& { return gbase[off - o.head0]; };  // absolute parameter offsets
    // the gradient a d^T of a weight matrix at `off`, rows x cols (cols divides 128)
    auto outer = [&](int64_t off, const float* a, int rows, const float* d, int cols) {
        const float mine = d[t % cols];
        float* const to = &G(off) + t;
#pragma unroll 16
        for (int i = 0; i < rows * cols / 128; ++i) to[i * 128] = a[i * (128 / cols) + t / cols] * mine;
    };
    for (int k = t; k < NL * 2 * HD; k += 128) p[k] = pooled[g * NL * 2 * HD + k];
    s[t] = hs.s[g * JK + t];
    a1[t] = hs.a1[g * M1 + t];
    if (t < M2) a2[t] = hs.a2[g * M2 + t];
    if (t < o.nout) dov[t] = dout[g * o.nout + t];
    __syncthreads();
    // out = a2 W3 + b3
    if (t < o.nout) G(o.m2b + t) = dov[t];
    for (int e = t; e < M2 * o.nout; e += 128) G(o.m2W + e) = a2[e / o.nout] * dov[e % o.nout];
    if (t < M2) {
        float acc = 0.0f;
        for (int q = 0; q < o.nout; ++q) acc += dov[q] * P[o.m2W + t * o.nout + q];
        d2[t] = a2[t] > 0.0f ? acc : 0.0f;
    }
    __syncthreads();
    // a2 = relu(a1 W2 + b2)
    if (t < M2) G(o.m1b + t) = d2[t];
    outer(o.m1W, a1, M1, d2, M2);
    {
        const float acc = row_dot<M2>(d2, P + o.m1W + t * M2, 0.0f);
        d1[t] = a1[t] > 0.0f ? acc : 0.0f;
    }
    __syncthreads();
    // a1 = relu(s W1 + b1)
    float ds = 0.0f;
#pragma unroll
    for (int q = 0; q < M1; q += 64) ds = row_dot<64>(d1 + q, P + o.m0W + t * M1 + q, ds);
    G(o.m0b + t) = d1[t];
    outer(o.m0W, s, JK, d1, M1);
    // s = sigmoid(zn), zn = zhat gamma + beta, zhat = (z - m) rstd
    const float dzn = ds * s[t] * (1.0f - s[t]);
    const float m = hs.ln[2 * g], rs = hs.ln[2 * g + 1];
    const float zh = (hs.z[g * JK + t] - m) * rs;
    G(o.lng + t) = dzn * zh;
    G(o.lnb + t) = dzn;
    const float dzh = dzn * P[o.lng + t];
    const float mean_a = block128_sum(dzh, red) / JK;
    const float mean_b = block128_sum(dzh * zh, red) / JK;
    dzv[t] = rs * (dzh - mean_a - zh * mean_b);
    __syncthreads();
    // z[l*32+o] = rob_l[o] + sum_k p_l[k] roW_l[k][o]
    for (int l = 0; l < NL; ++l) {
        if (t < RO) G(o.rob[l] + t) = dzv[l * RO + t];
        outer(o.roW[l], p + l * 2 * HD, 2 * HD, dzv + l * RO, RO);
        for (int k = t; k < 2 * HD; k += 128) {
            dpooled[(g * NL + l) * 2 * HD + k] = row_dot<RO>(dzv + l * RO, P + o.roW[l] + k * RO, 0.0f);
        }
    }
}

// Layer backward, first half, per tile: dX from pooling (mean and arg-max) and, below the last
// layer, from the next layer's aggregation (A_hat^T dH = A_hat dH, A symmetric); ReLU and the
// affine part of InstanceNorm; per-tile sums for the normalisation backward and gamma/beta. The walk and the
// split of rows and channels over the lanes are the layer kernel's, and so is what bounds it: the
// gathers of dH and, on large batches, Y in and dxhat out (422k nodes, four layers: 389 us with one channel per lane
// and the sums passed through LDS one by one, 323 here).
template <int HD, bool Y0, typename Off>
__global__ __launch_bounds__(4 * HD, 5) void bwd_a_kernel(const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                   const float* __restrict__ w, const int32_t* __restrict__ tile_graph,
                                                   const int32_t* __restrict__ gend, const float* __restrict__ gcnt,
                                                   const float* __restrict__ Y, const float* __restrict__ H0,
                                                   const float* __restrict__ W0, const float* __restrict__ b0,
                                                   const float* __restrict__ mu,
                                                   const float* __restrict__ rstd, const float* __restrict__ gam,
                                                   const float* __restrict__ bet, const float* __restrict__ dpooled,
                                                   const int32_t* __restrict__ argmax, int layer,
                                                   const float* __restrict__ dHn, float* __restrict__ dxh,
                                                   double* __restrict__ tb) {
    constexpr int LD = HD + 4, G = HD / 4;
    __shared__ __align__(16) float aggs[TILE][LD];  // per row: sum of w * dH of the layer above; then the reductions
    const int tile = dealt_tile(), wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int32_t r0 = tile * TILE + wv * 16;
    const int32_t g0 = r0 + 4 * (c / G);  // the first row of the lane's group (see visit_rows_x4)
    const int rp = dHn ? ptr[g0 + min(static_cast<int>(threadIdx.x % G), 4)] : 0;
    const int g = tile_graph[tile];
    const int32_t end = gend[g];
    const int c4 = 4 * static_cast<int>(threadIdx.x % G);  // the lane's channels: c4 .. c4 + 3
    float* const mine = &aggs[g0 - tile * TILE][c4];
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(mine + i * LD) = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 yv[4];  // the rows' own y, loaded while the aggregation runs
    auto own = [&] {
        float4 w04, w14, bb4;
        if constexpr (Y0) {
            w04 = *reinterpret_cast<const float4*>(W0 + c4);
            w14 = *reinterpret_cast<const float4*>(W0 + HD + c4);
            bb4 = *reinterpret_cast<const float4*>(b0 + c4);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (Y0)
                yv[e] = y0_of4(reinterpret_cast<const float2*>(H0)[g0 + e], w04, w14, bb4);
            else
                yv[e] = *reinterpret_cast<const float4*>(Y + static_cast<int64_t>(g0 + e) * HD + c4);
        }
    };
    if (dHn && one_group_walks<G>(rp)) {
        // (a 20k-row graph with a hub of 5000 neighbours, whole backward: 1.21 ms by the walk below, 0.89 here;
        // of 19000 4.17 and 2.77)
        own();
        visit_rows_one<HD>(
            ptr, col, w, r0, [&](int32_t j) { return dHn[static_cast<int64_t>(j) * HD + c]; },
            [&](int i, float v) { aggs[wv * 16 + i][c] = v; });
        wave_sync();
    } else if (dHn) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        visit_rows_x4<G, false>(
            rp, col, w, own,
            [&](int32_t j) {
                const Off at = static_cast<Off>(j) * (HD * 4) + c4 * 4;
                return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(dHn) + at);
            },
            [&](float wp, const float4& v) {
                acc.x += wp * v.x;
                acc.y += wp * v.y;
                acc.z += wp * v.z;
                acc.w += wp * v.w;
            },
            [&](int i) {  // read back below by the same lane
                *reinterpret_cast<float4*>(mine + i * LD) = acc;
                acc = make_float4(0.f, 0.f, 0.f, 0.f);
            });
    } else {
        own();
    }
    const auto four = [](const float4& v, float (&o)[4]) {
        o[0] = v.x;
        o[1] = v.y;
        o[2] = v.z;
        o[3] = v.w;
    };
    float m[4], rs[4], ga[4], be[4], dmean[4], dmax[4];
    four(*reinterpret_cast<const float4*>(mu + g * HD + c4), m);
    four(*reinterpret_cast<const float4*>(rstd + g * HD + c4), rs);
    four(*reinterpret_cast<const float4*>(gam + c4), ga);
    four(*reinterpret_cast<const float4*>(bet + c4), be);
    const float* dp = dpooled + static_cast<int64_t>(g * NL + layer) * 2 * HD + c4;
    four(*reinterpret_cast<const float4*>(dp), dmean);
    four(*reinterpret_cast<const float4*>(dp + HD), dmax);
    const int4 am4 = *reinterpret_cast<const int4*>(argmax + (g * NL + layer) * HD + c4);
    const int32_t am[4] = {am4.x, am4.y, am4.z, am4.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) dmean[k] /= gcnt[g];
    double sa[4] = {}, sb[4] = {}, sg[4] = {}, sbe[4] = {};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int32_t row = g0 + e;
        float y[4], ag[4], d[4];
        four(yv[e], y);
        four(*reinterpret_cast<const float4*>(mine + e * LD), ag);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d[k] = 0.0f;
            if (row >= end) continue;
            const float dx = dmean[k] + (row == am[k] ? dmax[k] : 0.0f) + ag[k];
            const float xh = (y[k] - m[k]) * rs[k];
            const float xn = xh * ga[k] + be[k];
            const float dxn = xn > 0.0f ? dx : 0.0f;
            d[k] = dxn * ga[k];
            sa[k] += d[k];
            sb[k] += static_cast<double>(d[k]) * xh;
            sg[k] += static_cast<double>(dxn) * xh;
            sbe[k] += dxn;
        }
        *reinterpret_cast<float4*>(dxh + static_cast<int64_t>(row) * HD + c4) = make_float4(d[0], d[1], d[2], d[3]);
    }
    // over the 16 rows of the HD lanes, then over the tile, in a fixed order (as in layer_kernel)
    const int cc = c4 + reduced_channel<G>();
    const double t[4] = {reduce_groups<G>(sa), reduce_groups<G>(sb), reduce_groups<G>(sg), reduce_groups<G>(sbe)};
    auto part = [&](int k) { return reinterpret_cast<double*>(&aggs[16 * k][0]); };
    static_assert(16 * LD * sizeof(float) >= 4 * HD * sizeof(double), "they fit");
    wave_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q) part(wv)[q * HD + cc] = t[q];
    __syncthreads();
    if (wv == 0)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            tb[tile * 4 * HD + q * HD + c] =
                part(0)[q * HD + c] + part(1)[q * HD + c] + part(2)[q * HD + c] + part(3)[q * HD + c];
}

// Layer backward, second half. dY = rstd (dxhat - mean(dxhat) - xhat mean(dxhat xhat));
// dH = dY W^T (stored for the layer below); partial dW = H^T dY and db = sum dY
// accumulated over the tiles a workgroup visits (fixed grid of w_blocks, fixed order). With MFMA it is
// bound by its four arrays (422k nodes: 432 MB in 92 us, 101 with 512
// workgroups). In FP32 by the LDS reads of the products: a thread
// keeps its row of W and reads rows of dY and H as 16-byte broadcasts (36.5k nodes of 32 channels: 41 us
// with W read per row and two rounds of tiles, 14 now).
template <int HD, bool MFMA>
__global__ __launch_bounds__(4 * HD) void bwd_b_kernel(int ntiles, const int32_t* __restrict__ tile_graph,
                                                   const int32_t* __restrict__ gend, const float* __restrict__ Y,
                                                   const float* __restrict__ mu, const float* __restrict__ rstd,
                                                   const float* __restrict__ gmean, const float* __restrict__ dxh,
                                                   const float* __restrict__ H, const float* __restrict__ W,
                                                   float* __restrict__ dH, float* __restrict__ wpart,
                                                   double* __restrict__ bpart) {
    constexpr int LD = HD + (MFMA ? 1 : 4);  // FP32: rows stay aligned to 16 bytes
    __shared__ __align__(16) float dYs[TILE][LD];
    __shared__ __align__(16) float Hs[TILE][LD];
    float (*Ds)[LD] = Hs;  // the dH product is formed after dW no longer needs Hs
    __shared__ unsigned short Bt[MFMA ? HD : 1][HD + 8];
    __shared__ double sh[4][HD];
    const int wv = threadIdx.x / HD, c = threadIdx.x % HD;
    static_assert(!MFMA || HD == 64, "the MFMA tiling is written for 64 channels");
    constexpr int NW = HD / 4;  // dW entries per thread
    if constexpr (MFMA) stage_bf16<HD>(W, Bt);  // dH = dY W^T: B[c'][k] = W[k][c'] read as rows of W
    float wr[MFMA ? 1 : HD];                           // FP32: row c of W
    if constexpr (!MFMA)
#pragma unroll
        for (int q = 0; q < HD; q += 4) {
            const float4 v = *reinterpret_cast<const float4*>(W + c * HD + q);
            wr[q] = v.x;
            wr[q + 1] = v.y;
            wr[q + 2] = v.z;
            wr[q + 3] = v.w;
        }
    // FP32: a thread owns the entries k = NW wv + q of column c of dW
    float accw[NW];
    for (int q = 0; q < NW; ++q) accw[q] = 0.0f;
    double accb = 0.0;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int g = tile_graph[tile];
        const int32_t end = gend[g];
        const float m = mu[g * HD + c], rs = rstd[g * HD + c];
        const float ma = gmean[g * 2 * HD + c], mb = gmean[g * 2 * HD + HD + c];
        // eight rows at a time, their loads issued together
        for (int r8 = 0; r8 < 16; r8 += 8) {
            float yv[8], dv[8], hv[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int32_t row = tile * TILE + wv * 16 + r8 + r;
                const int64_t k = static_cast<int64_t>(row) * HD + c;
                const bool ok = row < end;
                yv[r] = ok ? Y[k] : 0.0f;
                dv[r] = ok ? dxh[k] : 0.0f;
                hv[r] = ok ? H[k] : 0.0f;
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int lr = wv * 16 + r8 + r;
                const int32_t row = tile * TILE + lr;
                float dy = 0.0f;
                if (row < end) {
                    const float xh = (yv[r] - m) * rs;
                    dy = rs * (dv[r] - ma - xh * mb);
                }
                dYs[lr][c] = dy;
                Hs[lr][c] = hv[r];
                accb += dy;
            }
        }
        __syncthreads();
        // dW[k][c'] += sum_rows H[row][k] dY[row][c']
        if constexpr (!MFMA) {
            float acc[NW];
#pragma unroll
            for (int q = 0; q < NW; ++q) acc[q] = 0.0f;
#pragma unroll 4
            for (int r = 0; r < TILE; ++r) {
                const float dy = dYs[r][c];
#pragma unroll
                for (int q = 0; q < NW; q += 4) {
                    const float4 h = *reinterpret_cast<const float4*>(&Hs[r][wv * NW + q]);
                    acc[q] += h.x * dy;
                    acc[q + 1] += h.y * dy;
                    acc[q + 2] += h.z * dy;
                    acc[q + 3] += h.w * dy;
                }
            }
#pragma unroll
            for (int q = 0; q < NW; ++q) accw[q] += acc[q];
        } else {
            // 64 x 64 = (H^T)(64 x 64 rows) (dY): wavefront wv owns output rows k in [16 wv, 16 wv + 16)
            const int lane = c, i = lane % 16, kq = (lane / 16) * 8;
            f32x4 acc[4];
            for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int ks = 0; ks < TILE; ks += 32) {
                // H^T is the uncentred operand here as in the forward product: split it
                u16x8 av, alv;
                for (int e = 0; e < 8; ++e) {
                    unsigned short h, l;
                    split_bf16(Hs[ks + kq + e][wv * 16 + i], h, l);
                    av[e] = h;
                    alv[e] = l;
                }
                const bf16x8 a = __builtin_bit_cast(bf16x8, av);
                const bf16x8 al = __builtin_bit_cast(bf16x8, alv);
                for (int nb = 0; nb < 4; ++nb) {
                    u16x8 bv;
                    for (int e = 0; e < 8; ++e) bv[e] = f2bf(dYs[ks + kq + e][nb * 16 + i]);
                    const bf16x8 b = __builtin_bit_cast(bf16x8, bv);
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[nb], 0, 0, 0);
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b, acc[nb], 0, 0, 0);
                }
            }
            // lane holds rows k = 16 wv + 4 (lane/16) + e, column 16 nb + i; map to accw slots
            for (int nb = 0; nb < 4; ++nb)
                for (int e = 0; e < 4; ++e) accw[nb * 4 + e] += acc[nb][e];
        }
        // dH = dY W^T
        if constexpr (!MFMA) {
            for (int r = 0; r < 16; ++r) {
                const int lr = wv * 16 + r;
                const int32_t row = tile * TILE + lr;
                float acc = 0.0f;
#pragma unroll
                for (int q = 0; q < HD; q += 4) {
                    const float4 d = *reinterpret_cast<const float4*>(&dYs[lr][q]);
                    acc += d.x * wr[q];
                    acc += d.y * wr[q + 1];
                    acc += d.z * wr[q + 2];
                    acc += d.w * wr[q + 3];
                }
                dH[static_cast<int64_t>(row) * HD + c] = row < end ? acc : 0.0f;
            }
        } else {  // into the rows of Hs
            __syncthreads();
            tile_gemm<HD, true>(dYs, W, Bt, Ds);
            __syncthreads();
            for (int r = 0; r < 16; ++r) {
                const int lr = wv * 16 + r;
                const int32_t row = tile * TILE + lr;
                dH[static_cast<int64_t>(row) * HD + c] = row < end ? Ds[lr][c] : 0.0f;
            }
        }
        __syncthreads();
    }
    // write this workgroup's partials in plain [k][c] order
    float* const wp = wpart + static_cast<int64_t>(blockIdx.x) * HD * HD;
    if constexpr (MFMA) {
        const int lane = c, i = lane % 16;
        for (int nb = 0; nb < 4; ++nb)
            for (int e = 0; e < 4; ++e) {
                const int k = wv * 16 + (lane / 16) * 4 + e, cc = nb * 16 + i;
                wp[k * HD + cc] = accw[nb * 4 + e];
            }
    } else {
#pragma unroll
        for (int q = 0; q < NW; ++q) wp[(wv * NW + q) * HD + c] = accw[q];
    }
    accb = wave4_sum(accb, sh);
    if (wv == 0) bpart[blockIdx.x * HD + c] = accb;
}

// The same for layer 0, whose input is two features per node and whose dH nobody needs: a stream over dxhat
// (Y formed from H0), the lanes' rows and channels as in bwd_a_kernel and the sums in FP64 registers until
// the end; no LDS tile and no barrier per tile. (422k nodes: 115 us as the general kernel with
// two input channels, 20 here.)
template <int HD>
__global__ __launch_bounds__(4 * HD) void bwd_b0_kernel(int ntiles, const int32_t* __restrict__ tile_graph,
                                                    const int32_t* __restrict__ gend, const float* __restrict__ H0,
                                                    const float* __restrict__ W0, const float* __restrict__ b0,
                                                    const float* __restrict__ mu, const float* __restrict__ rstd,
                                                    const float* __restrict__ gmean, const float* __restrict__ dxh,
                                                    float* __restrict__ wpart, double* __restrict__ bpart) {
    constexpr int G = HD / 4;
    __shared__ double sh[4][3][HD];
    const int wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int c4 = 4 * static_cast<int>(threadIdx.x % G);
    const float4 w0 = *reinterpret_cast<const float4*>(W0 + c4), w1 = *reinterpret_cast<const float4*>(W0 + HD + c4),
                 bb = *reinterpret_cast<const float4*>(b0 + c4);
    double s0[4] = {}, s1[4] = {}, sb[4] = {};
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int32_t g0 = tile * TILE + wv * 16 + 4 * (c / G);
        float4 dv[4];
        float2 hv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dv[e] = *reinterpret_cast<const float4*>(dxh + static_cast<int64_t>(g0 + e) * HD + c4);
            hv[e] = reinterpret_cast<const float2*>(H0)[g0 + e];
        }
        const int g = tile_graph[tile];
        const int32_t end = gend[g];
        const float4 m = *reinterpret_cast<const float4*>(mu + g * HD + c4);
        const float4 rs = *reinterpret_cast<const float4*>(rstd + g * HD + c4);
        const float4 ma = *reinterpret_cast<const float4*>(gmean + g * 2 * HD + c4);
        const float4 mb = *reinterpret_cast<const float4*>(gmean + g * 2 * HD + HD + c4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (g0 + e >= end) continue;
            const float4 y = y0_of4(hv[e], w0, w1, bb);
            const float dy[4] = {rs.x * (dv[e].x - ma.x - (y.x - m.x) * rs.x * mb.x),
                                 rs.y * (dv[e].y - ma.y - (y.y - m.y) * rs.y * mb.y),
                                 rs.z * (dv[e].z - ma.z - (y.z - m.z) * rs.z * mb.z),
                                 rs.w * (dv[e].w - ma.w - (y.w - m.w) * rs.w * mb.w)};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s0[k] += static_cast<double>(hv[e].x) * dy[k];
                s1[k] += static_cast<double>(hv[e].y) * dy[k];
                sb[k] += dy[k];
            }
        }
    }
    const int cc = c4 + reduced_channel<G>();
    sh[wv][0][cc] = reduce_groups<G>(s0);
    sh[wv][1][cc] = reduce_groups<G>(s1);
    sh[wv][2][cc] = reduce_groups<G>(sb);
    __syncthreads();
    if (wv < 3) {
        const double v = sh[0][wv][c] + sh[1][wv][c] + sh[2][wv][c] + sh[3][wv][c];
        if (wv < 2)
            wpart[(static_cast<int64_t>(blockIdx.x) * 2 + wv) * HD + c] = static_cast<float>(v);
        else
            bpart[static_cast<int64_t>(blockIdx.x) * HD + c] = v;
    }
}

// One workgroup: A B by the layer kernel's products, over the same tile and with the same rows and columns per
// lane: D1 in FP32, D2 by MFMA with B in bf16 (hi parts), D3 with B's lo parts too. Any of them may be null.
__global__ __launch_bounds__(256) void tile_gemm_check_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                              float* __restrict__ D1, float* __restrict__ D2,
                                                              float* __restrict__ D3) {
    constexpr int HD = 64, NT = 256, LD = HD + 4, G = HD / 4;
    __shared__ __align__(16) float Hs[TILE][LD];
    __shared__ __align__(16) unsigned short wbf[2 * HD * HD];
    for (int e = threadIdx.x; e < TILE * HD; e += NT) Hs[e / HD][e % HD] = A[e];
    for (int e = threadIdx.x; e < HD * HD; e += NT) weight_parts<HD>(B, e, wbf);
    __syncthreads();
    const int wv = threadIdx.x / HD, c = threadIdx.x % HD;
    const int row0 = wv * 16 + 4 * (c / G), c4 = 4 * static_cast<int>(threadIdx.x % G);
    auto write = [&](float* D, const f32x4 (&acc)[4]) {
        for (int e = 0; e < 4; ++e)
            for (int nb = 0; nb < 4; ++nb) D[(row0 + e) * HD + c4 + nb] = acc[nb][e];
    };
    f32x4 acc[4];
    if (D2) {
        tile_product<HD, false, LD>(Hs, wbf, acc);
        write(D2, acc);
    }
    if (D3) {
        tile_product<HD, true, LD>(Hs, wbf, acc);
        write(D3, acc);
    }
    if (D1) {
        wave_sync();
        tile_gemm<HD, false, LD>(Hs, B, nullptr, Hs);
        wave_sync();
        for (int e = 0; e < 4; ++e)
            for (int k = 0; k < 4; ++k) D1[(row0 + e) * HD + c4 + k] = Hs[row0 + e][c4 + k];
    }
}

// out[e] = sum over the `parts` partial arrays (stride `stride`) of part[k][e], e < count, in FP64 and in a
// fixed order: 32 neighbouring outputs per workgroup (one 128-byte line of floats a part), whose eight groups
// of threads sum every eighth part. The sums of a layer's backward share one launch: they take a few us each
// and a launch nearly as long. (32-mesh training batch, 153 graphs: 17 launches and 145 us with a wavefront
// per output, 4 and 28 us.)
struct PartJob {
    const void* part;
    float* out;
    int64_t stride;
    int parts, count, block0;
    bool f64;
};
struct PartJobs {
    static constexpr int kMax = 5;
    PartJob job[kMax];
    int n = 0, blocks = 0;
    template <typename T>
    void add(const T* part, int parts, int64_t stride, int64_t count, float* out) {
        if (count <= 0) return;
        job[n++] = {part, out, stride, parts, static_cast<int>(count), blocks, sizeof(T) == sizeof(double)};
        blocks += static_cast<int>((count + 31) / 32);
    }
};

template <typename T>
__device__ __forceinline__ double sum_parts(const PartJob& j, int64_t e, int slot) {
    constexpr int kFly = 8;
    const T* p = static_cast<const T*>(j.part) + e;
    double s = 0.0;
    int k = slot;
    for (; k + 8 * (kFly - 1) < j.parts; k += 8 * kFly) {
        T v[kFly];
#pragma unroll
        for (int q = 0; q < kFly; ++q) v[q] = p[(k + 8 * q) * j.stride];
#pragma unroll
        for (int q = 0; q < kFly; ++q) s += static_cast<double>(v[q]);
    }
    for (; k < j.parts; k += 8) s += static_cast<double>(p[k * j.stride]);
    return s;
}

__global__ __launch_bounds__(256) void reduce_parts_kernel(PartJobs js) {
    __shared__ double sh[8][32];
    int i = 0;
    while (i + 1 < js.n && static_cast<int>(blockIdx.x) >= js.job[i + 1].block0) ++i;
    const PartJob j = js.job[i];
    const int lane = threadIdx.x % 32, slot = threadIdx.x / 32;
    const int64_t e = (static_cast<int64_t>(blockIdx.x) - j.block0) * 32 + lane;
    double s = 0.0;
    if (e < j.count) s = j.f64 ? sum_parts<double>(j, e, slot) : sum_parts<float>(j, e, slot);
    sh[slot][lane] = s;
    __syncthreads();
    if (slot != 0 || e >= j.count) return;
#pragma unroll
    for (int q = 1; q < 8; ++q) s += sh[q][lane];
    j.out[e] = static_cast<float>(s);
}

// ------------------------------------------------------------------------------------------
// Adam
// ------------------------------------------------------------------------------------------
constexpr int kAdamBlocks = 256;

__global__ __launch_bounds__(kAdamThreads) void sumsq_kernel(const float* __restrict__ g, int64_t n,
                                                             double* __restrict__ part) {
    constexpr int NT = kAdamThreads;
    __shared__ double red[NT];
    double s = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * NT + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * NT)
        s += static_cast<double>(g[i]) * g[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = NT / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void clipcoef_kernel(const double* __restrict__ part, float clip, double* __restrict__ scal,
                                float* __restrict__ gnorm_out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double s = 0.0;
    for (int k = 0; k < kAdamBlocks; ++k) s += part[k];
    const double nrm = sqrt(s);
    double coef = 1.0;
    if (clip > 0.0f) {
        coef = static_cast<double>(clip) / (nrm + 1e-6);
        if (coef > 1.0) coef = 1.0;
    }
    scal[0] = coef;
    scal[1] = nrm;
    if (gnorm_out) gnorm_out[0] = static_cast<float>(nrm);
}

__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float bc1,
                            float bc2, const double* __restrict__ scal) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = static_cast<float>(g[i] * scal[0]);
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

inline dim3 grid_of(int64_t n, int block) { return dim3(static_cast<unsigned>((n + block - 1) / block)); }

}  // namespace

// ------------------------------------------------------------------------------------------
// batch object
// ------------------------------------------------------------------------------------------
struct gcin_batch {
    int G = 0;
    int64_t N = 0, E = 0;
    int ntiles = 0;
    std::vector<int32_t> goff, gend, gtile, gn;
    std::vector<int32_t> cbound, gchunk;  // chunk tile bounds [nchunks + 1], graph chunk bounds [G + 1]
    int nchunks = 0;
    // device
    // tables, one contiguous part of the workspace that is uploaded at once
    int32_t *d_gend = nullptr, *d_tile_graph = nullptr;
    int32_t *d_cbound = nullptr, *d_gchunk = nullptr;
    FillGraph* d_fill = nullptr;
    size_t table_bytes = 0;
    double* cbuf = nullptr;  // chunk partial sums (up to 4 HD doubles per chunk)
    float* cmax = nullptr;
    int32_t* carg = nullptr;
    float* d_gcnt = nullptr;
    int32_t *ptr = nullptr, *col = nullptr;
    float *w = nullptr, *x0 = nullptr, *H0 = nullptr;
    unsigned short* wbf = nullptr;  // bf16 hi / lo parts of the weights of layers 1 .. NL-1
    float* Y[NL] = {};
    float* H[NL] = {};
    double* tstat = nullptr;
    float* mu[NL] = {};
    float* rstd[NL] = {};
    double* tpsum = nullptr;
    float* tpmax = nullptr;
    int32_t* tparg = nullptr;
    float* pooled = nullptr;
    int32_t* argmax = nullptr;
    HeadSave hs{};
    float *dpooled = nullptr, *ghead = nullptr, *dxh = nullptr, *dHa = nullptr, *dHb = nullptr;
    double* tb = nullptr;
    float* gmean = nullptr;
    double* ggb = nullptr;
    float* wpart = nullptr;
    double* bpart = nullptr;
    int64_t ghstride = 0;
    int last_degree = -1;
    int hd = 64;         // hidden width
    bool infer = false;  // forward only: no activations kept for a backward (GCIN_INFERENCE)
};

namespace {

struct Carve {
    uintptr_t base;
    size_t off = 0;
    template <class T>
    T* take(size_t count) {
        off = (off + 255) & ~static_cast<size_t>(255);
        T* p = reinterpret_cast<T*>(base + off);
        off += (count ? count : 1) * sizeof(T);
        return p;
    }
};

size_t layout_batch(gcin_batch* b, uintptr_t base) {
    Carve cv{base};
    const size_t G = b->G, N = b->N, E = b->E, T = b->ntiles, HD = b->hd;
    b->d_gend = cv.take<int32_t>(G);
    b->d_tile_graph = cv.take<int32_t>(T);
    b->d_gcnt = cv.take<float>(G);
    b->d_cbound = cv.take<int32_t>(static_cast<size_t>(b->nchunks) + 1);
    b->d_gchunk = cv.take<int32_t>(G + 1);
    b->d_fill = cv.take<FillGraph>(G);
    b->table_bytes = cv.off;
    b->cbuf = cv.take<double>(static_cast<size_t>(b->nchunks) * 4 * HD);
    b->cmax = cv.take<float>(static_cast<size_t>(b->nchunks) * HD);
    b->carg = cv.take<int32_t>(static_cast<size_t>(b->nchunks) * HD);
    b->ptr = cv.take<int32_t>(N + 1);
    b->col = cv.take<int32_t>(E);
    b->w = cv.take<float>(E);
    b->x0 = cv.take<float>(2 * N);
    b->H0 = cv.take<float>(2 * N);
    for (int l = 0; l < NL; ++l) {
        // forward only: a layer reads the layer below and its pooling reads the layer itself, so
        // two activation buffers in turn suffice (layers 1, 2, then 3 in layer 1's) and the
        // aggregates are not kept
        // layer 0's output is formed from H0 where needed and never stored
        b->Y[l] = l == 0 ? nullptr : b->infer && l >= 3 ? b->Y[l - 2] : cv.take<float>(N * HD);
        b->H[l] = l == 0 || b->infer ? nullptr : cv.take<float>(N * HD);
        b->mu[l] = cv.take<float>(G * HD);
        b->rstd[l] = cv.take<float>(G * HD);
    }
    b->tstat = cv.take<double>(T * 2 * HD);
    b->tpsum = cv.take<double>(T * HD);
    b->tpmax = cv.take<float>(T * HD);
    b->tparg = cv.take<int32_t>(T * HD);
    b->pooled = cv.take<float>(G * NL * 2 * HD);
    b->argmax = cv.take<int32_t>(G * NL * HD);
    b->hs.z = cv.take<float>(G * JK);
    b->hs.ln = cv.take<float>(G * 2);
    b->hs.s = cv.take<float>(G * JK);
    b->hs.a1 = cv.take<float>(G * M1);
    b->hs.a2 = cv.take<float>(G * M2);
    b->wbf = cv.take<unsigned short>(static_cast<size_t>(NL - 1) * 2 * HD * HD);
    if (b->infer) return (cv.off + 255) & ~static_cast<size_t>(255);  // no backward buffers
    b->dpooled = cv.take<float>(G * NL * 2 * HD);
    const Offs o4 = offsets(AMGG_MAX_DEGREE, b->hd);
    b->ghstride = ((o4.total - o4.head0) + 63) / 64 * 64;
    b->ghead = cv.take<float>(G * b->ghstride);
    b->dxh = cv.take<float>(N * HD);
    b->dHa = cv.take<float>(N * HD);
    b->dHb = cv.take<float>(N * HD);
    b->tb = cv.take<double>(T * 4 * HD);
    b->gmean = cv.take<float>(G * 2 * HD);
    b->ggb = cv.take<double>(G * 2 * HD);
    b->wpart = cv.take<float>(std::max<size_t>(static_cast<size_t>(w_blocks(HD)) * HD, kW0Blocks * 2) * HD);
    b->bpart = cv.take<double>(static_cast<size_t>(std::max(w_blocks(HD), kW0Blocks)) * HD);
    return (cv.off + 255) & ~static_cast<size_t>(255);
}

int plan_batch(gcin_batch* b, int ngraphs, const int32_t* n, const int32_t* nnz) {
    if (ngraphs < 1 || ngraphs > GCIN_MAX_GRAPHS) return amgg::fail(AMGG_EINVAL, "gcin: ngraphs out of range");
    b->G = ngraphs;
    b->goff.assign(ngraphs + 1, 0);
    b->gend.assign(ngraphs, 0);
    b->gtile.assign(ngraphs + 1, 0);
    b->gn.assign(ngraphs, 0);
    int64_t rows = 0, edges = 0;
    for (int g = 0; g < ngraphs; ++g) {
        if (n[g] < 1 || nnz[g] < n[g]) return amgg::fail(AMGG_EINVAL, "gcin: a graph has n < 1 or nnz < n");
        b->goff[g] = static_cast<int32_t>(rows);
        b->gend[g] = static_cast<int32_t>(rows + n[g]);
        b->gtile[g] = static_cast<int32_t>(rows / TILE);
        b->gn[g] = n[g];
        rows += (static_cast<int64_t>(n[g]) + TILE - 1) / TILE * TILE;
        edges += nnz[g];
        if (rows > INT32_MAX / 2 || edges > INT32_MAX / 2) return amgg::fail(AMGG_EINVAL, "gcin: batch too large");
    }
    b->goff[ngraphs] = static_cast<int32_t>(rows);
    b->gtile[ngraphs] = static_cast<int32_t>(rows / TILE);
    b->cbound.clear();
    b->gchunk.assign(ngraphs + 1, 0);
    for (int g = 0; g < ngraphs; ++g) {
        b->gchunk[g] = static_cast<int32_t>(b->cbound.size());
        for (int32_t t = b->gtile[g]; t < b->gtile[g + 1]; t += kChunkTiles) b->cbound.push_back(t);
    }
    b->gchunk[ngraphs] = static_cast<int32_t>(b->cbound.size());
    b->nchunks = static_cast<int>(b->cbound.size());
    b->cbound.push_back(b->gtile[ngraphs]);
    b->N = rows;
    b->E = edges;
    b->ntiles = static_cast<int>(rows / TILE);
    return AMGG_OK;
}

int hip_err(hipError_t e, const char* where) {
    return amgg::fail(AMGG_EHIP, std::string(where) + ": " + hipGetErrorString(e));
}

}  // namespace

static bool hidden_ok(int hidden) { return hidden == 64 || hidden == 32; }

extern "C" int64_t gcin_param_count_hidden(int degree, int hidden) {
    if (degree < 1 || degree > AMGG_MAX_DEGREE || !hidden_ok(hidden)) return -1;
    return offsets(degree, hidden).total;
}

extern "C" int64_t gcin_param_count(int degree) { return gcin_param_count_hidden(degree, 64); }

extern "C" int gcin_batch_workspace_bytes_ex(int hidden, int flags, int ngraphs, const int32_t* n, const int32_t* nnz,
                                             size_t* bytes) {
    return amgg::guarded([&]() -> int {
        if (!n || !nnz || !bytes) return amgg::fail(AMGG_EINVAL, "gcin_batch_workspace_bytes: null argument");
        if (!hidden_ok(hidden)) return amgg::fail(AMGG_EINVAL, "gcin_batch_workspace_bytes: hidden must be 64 or 32");
        if (flags & ~GCIN_INFERENCE) return amgg::fail(AMGG_EINVAL, "gcin_batch_workspace_bytes: unknown flag");
        gcin_batch b;
        b.hd = hidden;
        b.infer = (flags & GCIN_INFERENCE) != 0;
        int rc = plan_batch(&b, ngraphs, n, nnz);
        if (rc) return rc;
        *bytes = layout_batch(&b, 0);
        return AMGG_OK;
    });
}

extern "C" int gcin_batch_workspace_bytes_hidden(int hidden, int ngraphs, const int32_t* n, const int32_t* nnz,
                                                 size_t* bytes) {
    return gcin_batch_workspace_bytes_ex(hidden, 0, ngraphs, n, nnz, bytes);
}

extern "C" int gcin_batch_workspace_bytes(int ngraphs, const int32_t* n, const int32_t* nnz, size_t* bytes) {
    return gcin_batch_workspace_bytes_hidden(64, ngraphs, n, nnz, bytes);
}

extern "C" int gcin_batch_create_ex(int hidden, int flags, int ngraphs, const gcin_graph* graphs, void* workspace,
                                    size_t ws_bytes, void* stream, gcin_batch** out) {
    return amgg::guarded([&]() -> int {
        if (!hidden_ok(hidden)) return amgg::fail(AMGG_EINVAL, "gcin_batch_create: hidden must be 64 or 32");
        if (flags & ~GCIN_INFERENCE) return amgg::fail(AMGG_EINVAL, "gcin_batch_create: unknown flag");
        if (!graphs || !out || !workspace) return amgg::fail(AMGG_EINVAL, "gcin_batch_create: null argument");
        if (reinterpret_cast<uintptr_t>(workspace) & 255u)
            return amgg::fail(AMGG_EWORKSPACE, "gcin_batch_create: workspace not 256-byte aligned");
        if (ngraphs < 1 || ngraphs > GCIN_MAX_GRAPHS) return amgg::fail(AMGG_EINVAL, "gcin_batch_create: ngraphs out of range");
        std::vector<int32_t> n(ngraphs), z(ngraphs);
        for (int g = 0; g < ngraphs; ++g) {
            n[g] = graphs[g].n;
            z[g] = graphs[g].nnz;
            if (!graphs[g].rowptr || !graphs[g].col || !graphs[g].val)
                return amgg::fail(AMGG_EINVAL, "gcin_batch_create: null graph array");
        }
        auto* b = new gcin_batch();
        b->hd = hidden;
        b->infer = (flags & GCIN_INFERENCE) != 0;
        int rc = plan_batch(b, ngraphs, n.data(), z.data());
        if (rc) {
            delete b;
            return rc;
        }
        const size_t need = layout_batch(b, 0);
        if (ws_bytes < need) {
            delete b;
            return amgg::fail(AMGG_EWORKSPACE, "gcin_batch_create: workspace too small");
        }
        layout_batch(b, reinterpret_cast<uintptr_t>(workspace));
        hipStream_t st = static_cast<hipStream_t>(stream);
        // tables, laid out on the host as in the workspace and uploaded in one copy
        std::vector<unsigned char> tab(b->table_bytes);
        auto host = [&](auto* dev) {
            return reinterpret_cast<std::remove_reference_t<decltype(dev)>>(
                tab.data() + (reinterpret_cast<uintptr_t>(dev) - reinterpret_cast<uintptr_t>(workspace)));
        };
        int32_t *gend = host(b->d_gend), *tile_graph = host(b->d_tile_graph);
        float* cnt = host(b->d_gcnt);
        FillGraph* fill = host(b->d_fill);
        int64_t e0 = 0;
        for (int g = 0; g < ngraphs; ++g) {
            gend[g] = b->gend[g];
            for (int t = b->gtile[g]; t < b->gtile[g + 1]; ++t) tile_graph[t] = g;
            cnt[g] = static_cast<float>(b->gn[g]);
            fill[g] = FillGraph{graphs[g].rowptr, graphs[g].col, graphs[g].val, n[g], b->goff[g],
                                static_cast<int32_t>(e0)};
            e0 += z[g];
        }
        std::memcpy(host(b->d_cbound), b->cbound.data(), sizeof(int32_t) * b->cbound.size());
        std::memcpy(host(b->d_gchunk), b->gchunk.data(), sizeof(int32_t) * b->gchunk.size());
        hipError_t e = hipMemcpyAsync(workspace, tab.data(), tab.size(), hipMemcpyHostToDevice, st);
        if (e == hipSuccess) {
            fill_graph_kernel<<<b->ntiles, 256, 0, st>>>(b->ntiles, b->d_tile_graph, b->d_fill, b->ptr, b->col, b->w,
                                                         b->x0);
            e = hipGetLastError();
        }
        // the host tables must stay alive until the copy completes, the graphs' arrays until they are read
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            delete b;
            return hip_err(e, "gcin_batch_create");
        }
        *out = b;
        return AMGG_OK;
    });
}

extern "C" int gcin_batch_create_hidden(int hidden, int ngraphs, const gcin_graph* graphs, void* workspace,
                                        size_t ws_bytes, void* stream, gcin_batch** out) {
    return gcin_batch_create_ex(hidden, 0, ngraphs, graphs, workspace, ws_bytes, stream, out);
}

extern "C" int gcin_batch_create(int ngraphs, const gcin_graph* graphs, void* workspace, size_t ws_bytes, void* stream,
                                 gcin_batch** out) {
    return gcin_batch_create_hidden(64, ngraphs, graphs, workspace, ws_bytes, stream, out);
}

extern "C" int gcin_batch_destroy(gcin_batch* b) {
    delete b;
    return AMGG_OK;
}

namespace {

// The tile products run on MFMA for 64 channels; the 32-channel variant keeps them in FP32.
template <int HD>
void forward_impl(gcin_batch* b, int degree, int precision, const float* P, float* coeffs_out, hipStream_t st) {
    constexpr int NT = 4 * HD;
    const Offs o = offsets(degree, HD);
    const int T = b->ntiles, G = b->G;
    const float *W0 = P + o.convW[0], *b0 = P + o.convb[0];
    layer0_kernel<HD><<<T, NT, 0, st>>>(b->ptr, b->col, b->w, b->x0, b->d_tile_graph, b->d_gend, W0, b0, b->H0,
                                        b->tstat);
    // Statistics of layer l, then its readout, which feeds no later layer: pooling each layer as
    // soon as its statistics exist leaves every result as it is and lets an inference-only batch
    // reuse the buffer of layer l - 1 for layer l + 1. The readout partials of layer l are formed
    // by the kernel of layer l + 1 (from its tile's own rows of the layer below), the last layer's by a
    // pooling pass; the per-graph reductions of a layer's statistics and of the readout below it
    // share their launches (reduce_kernel).
    const int C = b->nchunks;
    const bool one = C == G;  // every graph is one chunk
    auto reduce = [&](int stat_layer, int pool_layer) {  // -1: none
        Reduce r{b->tstat, b->tpsum, b->tpmax, b->tparg, b->cbuf, b->cbuf + static_cast<int64_t>(C) * 2 * HD, b->cmax,
                 b->carg, b->d_gcnt, stat_layer < 0 ? nullptr : b->mu[stat_layer],
                 stat_layer < 0 ? nullptr : b->rstd[stat_layer], b->pooled, b->argmax, pool_layer};
        const int stat = stat_layer >= 0, pool = pool_layer >= 0;
        if (one) {
            reduce_kernel<HD, true><<<dim3(G, stat + pool), kSumGroups * HD, 0, st>>>(b->d_cbound, r, 1 - stat);
            return;
        }
        reduce_kernel<HD, false><<<dim3(C, 2 * stat + pool), kSumGroups * HD, 0, st>>>(b->d_cbound, r, 2 - 2 * stat);
        r.tstat = r.cstat;
        r.psum = r.csum;
        r.pmax = r.cmax;
        r.parg = r.carg;
        reduce_kernel<HD, true><<<dim3(G, stat + pool), kSumGroups * HD, 0, st>>>(b->d_gchunk, r, 1 - stat);
    };
    reduce(0, -1);
    const bool mfma = HD == 64 && precision != GCIN_FP32;
    if (mfma) weights_bf16_kernel<HD><<<dim3(NL - 1, HD * HD / 256), 256, 0, st>>>(P, o, b->wbf);
    for (int l = 1; l < NL; ++l) {
        const bool y0 = l == 1;
        auto pick = [&](auto off) {
            using Off = decltype(off);
            if constexpr (HD == 64) {
                if (precision == GCIN_BF16X3)
                    return y0 ? layer_kernel<HD, true, true, true, uint32_t> : layer_kernel<HD, true, true, false, Off>;
                if (precision == GCIN_BF16)
                    return y0 ? layer_kernel<HD, true, false, true, uint32_t> : layer_kernel<HD, true, false, false, Off>;
            }
            return y0 ? layer_kernel<HD, false, false, true, uint32_t> : layer_kernel<HD, false, false, false, Off>;
        };
        auto kern = b->N * HD * 4 <= UINT32_MAX ? pick(uint32_t{}) : pick(uint64_t{});
        kern<<<T, NT, 0, st>>>(b->ptr, b->col, b->w, b->d_tile_graph, b->d_gend, b->Y[l - 1], b->H0, W0, b0,
                               b->mu[l - 1], b->rstd[l - 1], P + o.gam[l - 1], P + o.bet[l - 1], P + o.convW[l],
                               P + o.convb[l], b->wbf + static_cast<int64_t>(l - 1) * 2 * HD * HD, b->H[l], b->Y[l],
                               b->tstat, b->tpsum, b->tpmax, b->tparg);
        reduce(l, l - 1);
    }
    pool_tile_kernel<HD><<<T, NT, 0, st>>>(b->d_tile_graph, b->d_gend, b->Y[NL - 1], b->mu[NL - 1], b->rstd[NL - 1],
                                           P + o.gam[NL - 1], P + o.bet[NL - 1], b->tpsum, b->tpmax, b->tparg);
    reduce(-1, NL - 1);
    head_fwd_kernel<HD><<<G, 128, 0, st>>>(P, o, b->pooled, b->hs, coeffs_out);
}

template <int HD>
void backward_impl(gcin_batch* b, int degree, int precision, const float* P, const float* dcoeffs, float* grads,
                   hipStream_t st) {
    constexpr int NT = 4 * HD;
    const Offs o = offsets(degree, HD);
    const int T = b->ntiles, G = b->G;
    head_bwd_kernel<HD><<<G, 128, 0, st>>>(P, o, b->pooled, b->hs, dcoeffs, b->ghead, b->ghstride, b->dpooled);
    PartJobs sums;  // of the parameter gradients: the head's (over the graphs) with the last layer's
    sums.add(b->ghead, G, b->ghstride, o.total - o.head0, grads + o.head0);
    float* dHn = nullptr;  // dH of the layer above (for the aggregation backward)
    float* bufs[2] = {b->dHa, b->dHb};
    for (int l = NL - 1; l >= 0; --l) {
        const float *W0 = P + o.convW[0], *b0 = P + o.convb[0];
        auto pick = [&](auto off) {
            return l == 0 ? bwd_a_kernel<HD, true, decltype(off)> : bwd_a_kernel<HD, false, decltype(off)>;
        };
        (b->N * HD * 4 <= UINT32_MAX ? pick(uint32_t{}) : pick(uint64_t{}))<<<T, NT, 0, st>>>(
            b->ptr, b->col, b->w, b->d_tile_graph, b->d_gend, b->d_gcnt, b->Y[l], b->H0, W0, b0, b->mu[l], b->rstd[l],
            P + o.gam[l], P + o.bet[l], b->dpooled, b->argmax, l, dHn, b->dxh, b->tb);
        const bool one = b->nchunks == G;  // every graph is one chunk
        if (!one)
            bwd_sum_kernel<HD, false><<<dim3(b->nchunks, 4), kSumGroups * HD, 0, st>>>(b->tb, b->d_cbound, b->cbuf,
                                                                                       nullptr, nullptr, nullptr);
        bwd_sum_kernel<HD, true><<<dim3(G, 4), kSumGroups * HD, 0, st>>>(
            one ? b->tb : b->cbuf, one ? b->d_cbound : b->d_gchunk, nullptr, b->d_gcnt, b->gmean, b->ggb);
        sums.add(b->ggb, G, 2 * HD, HD, grads + o.gam[l]);
        sums.add(b->ggb + HD, G, 2 * HD, HD, grads + o.bet[l]);
        float* dHout = l > 0 ? bufs[l & 1] : nullptr;
        const int grid = std::min(T, l > 0 ? w_blocks(HD) : kW0Blocks);
        if (l == 0) {
            bwd_b0_kernel<HD><<<grid, NT, 0, st>>>(T, b->d_tile_graph, b->d_gend, b->H0, W0, b0, b->mu[l], b->rstd[l],
                                                   b->gmean, b->dxh, b->wpart, b->bpart);
            sums.add(b->wpart, grid, 2 * HD, 2 * HD, grads + o.convW[l]);
        } else {
            auto kern = bwd_b_kernel<HD, false>;
            if constexpr (HD == 64)
                if (precision != GCIN_FP32) kern = bwd_b_kernel<HD, true>;
            kern<<<grid, NT, 0, st>>>(T, b->d_tile_graph, b->d_gend, b->Y[l], b->mu[l], b->rstd[l], b->gmean, b->dxh,
                                      b->H[l], P + o.convW[l], dHout, b->wpart, b->bpart);
            sums.add(b->wpart, grid, HD * HD, HD * HD, grads + o.convW[l]);
        }
        sums.add(b->bpart, grid, HD, HD, grads + o.convb[l]);
        reduce_parts_kernel<<<sums.blocks, 256, 0, st>>>(sums);
        sums = PartJobs{};
        dHn = dHout;
    }
}

}  // namespace

extern "C" int gcin_forward(gcin_batch* b, int degree, int precision, const float* P, float* coeffs_out, void* stream) {
    return amgg::guarded([&]() -> int {
        if (!b || !P || !coeffs_out) return amgg::fail(AMGG_EINVAL, "gcin_forward: null argument");
        if (degree < 1 || degree > AMGG_MAX_DEGREE) return amgg::fail(AMGG_EINVAL, "gcin_forward: degree out of range");
        if (precision < GCIN_FP32 || precision > GCIN_BF16X3) return amgg::fail(AMGG_EINVAL, "gcin_forward: bad precision");
        hipStream_t st = static_cast<hipStream_t>(stream);
        if (b->hd == 32)
            forward_impl<32>(b, degree, precision, P, coeffs_out, st);
        else
            forward_impl<64>(b, degree, precision, P, coeffs_out, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_err(e, "gcin_forward");
        b->last_degree = degree;
        return AMGG_OK;
    });
}

extern "C" int gcin_backward(gcin_batch* b, int degree, int precision, const float* P, const float* dcoeffs,
                             float* grads, void* stream) {
    return amgg::guarded([&]() -> int {
        if (!b || !P || !dcoeffs || !grads) return amgg::fail(AMGG_EINVAL, "gcin_backward: null argument");
        if (b->infer) return amgg::fail(AMGG_ESTATE, "gcin_backward: the batch was created for inference only");
        if (degree != b->last_degree) return amgg::fail(AMGG_ESTATE, "gcin_backward: no forward pass of this degree");
        if (precision < GCIN_FP32 || precision > GCIN_BF16X3) return amgg::fail(AMGG_EINVAL, "gcin_backward: bad precision");
        hipStream_t st = static_cast<hipStream_t>(stream);
        if (b->hd == 32)
            backward_impl<32>(b, degree, precision, P, dcoeffs, grads, st);
        else
            backward_impl<64>(b, degree, precision, P, dcoeffs, grads, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_err(e, "gcin_backward");
        return AMGG_OK;
    });
}

extern "C" int gcin_tile_gemm_check(const float* A, const float* B, float* D_fp32, float* D_bf16, void* stream) {
    if (!A || !B || !D_fp32 || !D_bf16) return amgg::fail(AMGG_EINVAL, "gcin_tile_gemm_check: null argument");
    tile_gemm_check_kernel<<<1, 256, 0, static_cast<hipStream_t>(stream)>>>(A, B, D_fp32, D_bf16, nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e, "gcin_tile_gemm_check");
    return AMGG_OK;
}

extern "C" int gcin_tile_gemm_check_x3(const float* A, const float* B, float* D, void* stream) {
    if (!A || !B || !D) return amgg::fail(AMGG_EINVAL, "gcin_tile_gemm_check_x3: null argument");
    tile_gemm_check_kernel<<<1, 256, 0, static_cast<hipStream_t>(stream)>>>(A, B, nullptr, nullptr, D);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_err(e, "gcin_tile_gemm_check_x3");
    return AMGG_OK;
}

constexpr size_t kAdamScratchDoubles = kAdamBlocks + 8;  // partial sums of ||g||^2, then the clip scalars

extern "C" size_t adam_scratch_bytes(void) { return sizeof(double) * kAdamScratchDoubles; }

namespace {
// The three launches of one Adam step; `work` holds kAdamScratchDoubles doubles of device memory.
// Every entry of `work` that is read was written earlier in the same step (each partial by its
// workgroup, the scalars by the one-thread kernel), so it needs no clearing between calls.
hipError_t adam_launch(float* params, const float* grads, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, int step, float clip, float* gnorm_out, double* work, hipStream_t st) {
    double* part = work;
    double* scal = part + kAdamBlocks;
    sumsq_kernel<<<kAdamBlocks, kAdamThreads, 0, st>>>(grads, n, part);
    clipcoef_kernel<<<1, 1, 0, st>>>(part, clip, scal, gnorm_out);
    const float bc1 = 1.0f - std::pow(b1, static_cast<float>(step));
    const float bc2 = 1.0f - std::pow(b2, static_cast<float>(step));
    adam_kernel<<<grid_of(n, 256), 256, 0, st>>>(params, grads, m, v, n, lr, b1, b2, eps, bc1, bc2, scal);
    return hipGetLastError();
}

bool adam_args_ok(const float* params, const float* grads, const float* m, const float* v, int64_t n, int step) {
    return params && grads && m && v && n > 0 && step >= 1;
}
}  // namespace

extern "C" int adam_step(float* params, const float* grads, float* m, float* v, int64_t n, float lr, float b1, float b2,
                         float eps, int step, float clip, float* gnorm_out, void* workspace, void* stream) {
    return amgg::guarded([&]() -> int {
        if (!adam_args_ok(params, grads, m, v, n, step) || !workspace)
            return amgg::fail(AMGG_EINVAL, "adam_step: bad argument");
        const hipError_t e = adam_launch(params, grads, m, v, n, lr, b1, b2, eps, step, clip, gnorm_out,
                                         static_cast<double*>(workspace), static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return hip_err(e, "adam_step");
        return AMGG_OK;
    });
}

// ------------------------------------------------------------------------------------------
// Adam step without any allocation: the step's scratch (kAdamScratchDoubles doubles) is this
// file-scope device array, one copy per GPU, held until the process ends. Host code never
// passes `scratch` itself to a kernel (on the host it names a stand-in, not device memory):
// it uses the address hipGetSymbolAddress returns on each device, looked up once per device.
// ------------------------------------------------------------------------------------------
static __device__ __align__(256) double scratch[kAdamScratchDoubles];
static_assert(sizeof(scratch) == sizeof(double) * kAdamScratchDoubles, "one Adam step's scratch, whatever n");

namespace {
std::mutex g_scratch_mu;
double* g_scratch_ptr[64] = {};  // per device ordinal: the address of `scratch` on that device

// Address of `scratch` on `device`, looked up on the first call for that device with the device
// current (the caller's current device is restored afterwards).
hipError_t scratch_on(int device, double** out) {
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int prev = -1;
        hipError_t e = hipGetDevice(&prev);
        if (e == hipSuccess && prev != device) e = hipSetDevice(device);
        void* p = nullptr;
        if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (prev >= 0 && prev != device) {
            const hipError_t e2 = hipSetDevice(prev);
            if (e == hipSuccess) e = e2;
        }
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = static_cast<double*>(p);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}
}  // namespace

extern "C" int adam_step_noalloc(float* params, const float* grads, float* m, float* v, int64_t n, float lr,
                                 float b1, float b2, float eps, int step, float clip, float* gnorm_out,
                                 void* stream) {
    return amgg::guarded([&]() -> int {
        if (!adam_args_ok(params, grads, m, v, n, step)) return amgg::fail(AMGG_EINVAL, "adam_step_noalloc: bad argument");
        const hipStream_t st = static_cast<hipStream_t>(stream);
        int device = -1;
        hipError_t e = st ? hipStreamGetDevice(st, &device) : hipGetDevice(&device);
        double* work = nullptr;
        if (e == hipSuccess) e = scratch_on(device, &work);
        if (e == hipSuccess) e = adam_launch(params, grads, m, v, n, lr, b1, b2, eps, step, clip, gnorm_out, work, st);
        if (e != hipSuccess) return hip_err(e, "adam_step_noalloc");
        return AMGG_OK;
    });
}
