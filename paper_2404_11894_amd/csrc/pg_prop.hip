// pg_prop.hip -- iterated aggregation + propagation and the output to pixels.
//
// Paper eqs. ag-mf, rte-pg and rte-mff: the indirect part of the scattered
// radiance is re-aggregated from the neighbours' incoming indirect radiance,
// the constant direct part is added, and the result is propagated one edge
// back along each path.  With delta tracking the propagation factor
// transmittance / free-flight pdf equals 1/sigma_t at the collision, which
// turns sigma_s * phase into albedo * phase, so propagation is a shift:
//   y_i = b_i + albedo_i sum_j w_ij L(j),   L(v) = y(succ v), 0 at a path's end.
//
// Two schedules, identical arithmetic:
//  * two-pass: a sparse matrix-vector product over the spatially sorted rows
//    (neighbour gathers stay within a few grid cells), then the shift as one
//    gather per vertex;
//  * shifted: the rows are pre-arranged in predecessor order, row v holding
//    albedo_u w_u. and b_u of its successor u, so one pass per iteration
//    computes L directly.
// Both are sparse gathers bound by HBM bandwidth (about 0.5 flop per byte).
#include <algorithm>
#include <cmath>

#include "pg_internal.h"

namespace pg {

// Rows in path order, as callers hold them.  One group of KP lanes per row, lane =
// edge: the row's column ids and weights are read as contiguous, coalesced
// segments, each lane gathers one x value, and the group reduces.
//
// succ NULL: y_i is stored at i.  With succ the propagation is part of the store: in
// path order the predecessor of i is i - 1 where it has one, so row i stores at
// i - 1, a path's last vertex gets 0, and y is x of the next iteration, each entry
// written once.  One launch an iteration instead of two and no pass over y: a call
// over 29 thousand vertices (K = 8, D = 8), bound by its launches, 76 -> 48 us.
template <int KP>
__global__ __launch_bounds__(kBlock) void k_spmv(int64_t N, int K, const int32_t* __restrict__ col,
                                                 const float* __restrict__ w, const float* __restrict__ x,
                                                 const float* __restrict__ b, const float* __restrict__ alpha,
                                                 const int32_t* __restrict__ succ, float* __restrict__ y) {
    constexpr int GR = kBlock / KP;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int lane = threadIdx.x % KP;
    const int64_t i = tile * GR + threadIdx.x / KP;
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
    if (i < N && lane < K) {
        const int64_t e = i * K + lane;
        const int64_t j = col[e];
        const float ww = w[e];
        if ((uint64_t)j < (uint64_t)N) {   // ids from callers are not trusted
            ax = ww * x[3 * j];
            ay = ww * x[3 * j + 1];
            az = ww * x[3 * j + 2];
        }
    }
    ax = group_sum<KP>(ax);
    ay = group_sum<KP>(ay);
    az = group_sum<KP>(az);
    if (i >= N || lane != 0) return;
    int64_t to = i;
    if (succ) {
        if (succ[i] < 0) st3(y, i, f3{0.f, 0.f, 0.f});
        if (i == 0 || succ[i - 1] < 0) return;
        to = i - 1;
    }
    const float a = alpha[i];
    st3(y, to, f3{fmaf(a, ax, b[3 * i]), fmaf(a, ay, b[3 * i + 1]), fmaf(a, az, b[3 * i + 2])});
}

hipError_t launch_spmv(int64_t N, int K, const int32_t* col, const float* w, const float* x, const float* b,
                       const float* alpha, const int32_t* succ, float* y, hipStream_t s) {
    if (N == 0) return hipSuccess;
    dispatch_kp(K, [&](auto kp) {
        constexpr int KP = decltype(kp)::value;
        hipLaunchKernelGGL(k_spmv<KP>, dim3((unsigned)div_up(N, kBlock / KP)), dim3(kBlock), 0, s, N, K, col, w,
                           x, b, alpha, succ, y);
    });
    return hipGetLastError();
}

// One thread per row over the sliced-ELL layout: each wave owns one slice of
// 64 rows and reads four edges of each of its rows per 16-byte load (1 KiB
// contiguous per wave).  rowmask (nullable): rows with rowmask[i] < 0 output
// 0.  alpha NULL means 1.  SCATTER: the row's result is stored at
// y[rowmask[i]] (the predecessor) and rows with rowmask[i] < 0 are skipped;
// otherwise such rows store 0 at y[i].
//
// Blocks run in plain launch order (all XCDs sweep the same region of the
// sorted rows together, which measured faster here than giving each XCD its
// own contiguous range), and the edge ids and weights, read exactly once, are
// loaded non-temporally so they do not displace the gathered vector in L2.
template <int KT, bool SCATTER, int BS>
__global__ __launch_bounds__(BS) void k_spmv_ell(int64_t N, int K, const int32_t* __restrict__ col,
                                                 const float* __restrict__ w, const float* __restrict__ x,
                                                 const float* __restrict__ b, const float* __restrict__ alpha,
                                                 const int32_t* __restrict__ rowmask, float* __restrict__ y,
                                                 int group) {
    const int64_t tile = grouped_tile(blockIdx.x, gridDim.x, group);
    const int64_t i = tile * BS + threadIdx.x;
    if (i >= N) return;
    int64_t dst = i;
    if (rowmask) {
        dst = rowmask[i];
        if (dst < 0) {
            if (!SCATTER) st3(y, i, f3{0.f, 0.f, 0.f});
            return;
        }
        if (!SCATTER) dst = i;
    }
    const f3 z = ell_row_sum<KT>(i, K, col, w, x);
    const f3 bb = ld3(b, i);
    const float a = alpha ? alpha[i] : 1.0f;
    st3_nt(y, dst, f3{fmaf(a, z.x, bb.x), fmaf(a, z.y, bb.y), fmaf(a, z.z, bb.z)});
}

template <bool SCATTER>
static void go_spmv_ell(int64_t N, int K, const int32_t* col, const float* w, const float* x, const float* b,
                        const float* alpha, const int32_t* rowmask, float* y, hipStream_t s, int tile, int group) {
    dispatch_tile(tile, [&](auto bs) {
        constexpr int BS = decltype(bs)::value;
        dim3 grid((unsigned)div_up(N, BS)), block(BS);
        dispatch_k4(K, [&](auto kt) {
            constexpr int KT = decltype(kt)::value;
            hipLaunchKernelGGL((k_spmv_ell<KT, SCATTER, BS>), grid, block, 0, s, N, K, col, w, x, b, alpha, rowmask,
                               y, group);
        });
    });
}

hipError_t launch_spmv_ell(int64_t N, int K, const int32_t* col, const float* w, const float* x, const float* b,
                           const float* alpha, const int32_t* rowmask, float* y, hipStream_t s, int tile,
                           int tile_group) {
    if (N == 0) return hipSuccess;
    go_spmv_ell<false>(N, K, col, w, x, b, alpha, rowmask, y, s, tile, tile_group);
    return hipGetLastError();
}

hipError_t launch_spmv_scatter(int64_t N, int K, const int32_t* col, const float* w, const float* x,
                               const float* b, const float* alpha, const int32_t* pred, float* xn, hipStream_t s) {
    if (N == 0) return hipSuccess;
    go_spmv_ell<true>(N, K, col, w, x, b, alpha, pred, xn, s, 0, 0);
    return hipGetLastError();
}

// ------------------------------------------------- compact edge ids ---
// One wave per 64-row slice: each lane counts its row's escaped offsets, a
// wave prefix sum gives the row's start in the slice's escape list (slot 0),
// and the row's octets are written as 16-byte stores.  Rows past N keep
// offset 0 in every slot.
__global__ __launch_bounds__(kBlock) void k_c16_build(int64_t N, int K, const int32_t* __restrict__ col,
                                                      int16_t* __restrict__ c16, uint32_t* __restrict__ cnt,
                                                      uint16_t* __restrict__ row_start,
                                                      const int32_t* __restrict__ place) {
    if (place && *place == kPlaceRows) return;   // there is no sliced ELL
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nsl = div_up(N, kSlice);
    if ((i >> 6) >= nsl) return;   // whole waves leave together (a slice is one wave)
    const int K4 = ell_k4(K), K8 = c16_k8(K);
    const int l0 = row_start ? 0 : 1;
    uint32_t n = 0;
    if (i < N)
        for (int l = l0; l < K4; ++l) {
            const int64_t off = (int64_t)col[eidx(i, l, K)] - i;
            n += (off < -32767 || off > 32767) ? 1u : 0u;
        }
    uint32_t inc = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    const uint32_t start = inc - n;
    if (row_start && i < N) row_start[i] = (uint16_t)start;
    const int64_t b16 = c16_row(i, K);
    for (int o = 0; 8 * o < K8; ++o) {
        int32_t words[4];
        for (int h = 0; h < 4; ++h) {
            int32_t v[2];
            for (int e = 0; e < 2; ++e) {
                const int l = 8 * o + 2 * h + e;
                int32_t val = 0;
                if (l == 0 && !row_start) {
                    val = (int32_t)(start & 0xffffu);
                } else if (i < N && l < K4) {
                    const int64_t off = (int64_t)col[eidx(i, l, K)] - i;
                    val = (off < -32767 || off > 32767) ? kC16Escape : (int32_t)off;
                }
                v[e] = val & 0xffff;
            }
            words[h] = v[0] | (v[1] << 16);
        }
        *reinterpret_cast<i32x4*>(c16 + b16 + o * kOctStride) = i32x4{words[0], words[1], words[2], words[3]};
    }
    if (lane == kWave - 1) cnt[i >> 6] = inc;
}

// Escaped ids of each row at its slice's list start + its slot-0 start.
__global__ __launch_bounds__(kBlock) void k_c16_escapes(int64_t N, int K, const int32_t* __restrict__ col,
                                                        const int16_t* __restrict__ c16,
                                                        const uint32_t* __restrict__ c16_base,
                                                        const uint16_t* __restrict__ row_start,
                                                        int32_t* __restrict__ ovf,
                                                        const int32_t* __restrict__ place) {
    if (place && *place == kPlaceRows) return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= N) return;
    int64_t p = (int64_t)c16_base[i >> 6] + (row_start ? row_start[i] : (uint16_t)c16[c16_row(i, K)]);
    const int K4 = ell_k4(K);
    for (int l = row_start ? 0 : 1; l < K4; ++l) {
        const int32_t j = col[eidx(i, l, K)];
        const int64_t off = (int64_t)j - i;
        if (off < -32767 || off > 32767) ovf[p++] = j;
    }
}

hipError_t launch_c16_build(int64_t N, int K, const int32_t* col, int16_t* c16, uint32_t* cnt, uint32_t* c16_base,
                            uint32_t* partials, int32_t* ovf, hipStream_t s, uint16_t* start,
                            const int32_t* place) {
    if (N == 0) return hipSuccess;
    const int64_t nsl = div_up(N, kSlice);
    hipLaunchKernelGGL(k_c16_build, dim3((unsigned)div_up(nsl * kSlice, kBlock)), dim3(kBlock), 0, s, N, K, col,
                       c16, cnt, start, place);
    hipError_t e = launch_scan_exclusive(cnt, c16_base, nsl, partials, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_c16_escapes, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, K, col, c16,
                       c16_base, (const uint16_t*)start, ovf, place);
    return hipGetLastError();
}

// The two-pass aggregation over the compact ids: the same rows, slots and
// arithmetic as k_spmv_ell, so the same results bit for bit, with 2 bytes per
// id streamed instead of 4 (plus the few escaped ids).
template <int KT, int BS, bool NT>
__global__ __launch_bounds__(BS) void k_spmv_c16(int64_t N, int K, const int16_t* __restrict__ c16,
                                                 const uint32_t* __restrict__ c16_base,
                                                 const int32_t* __restrict__ ovf, const float* __restrict__ w,
                                                 const float* __restrict__ x, const float* __restrict__ b,
                                                 const float* __restrict__ alpha, float* __restrict__ y, int group) {
    const int64_t tile = grouped_tile(blockIdx.x, gridDim.x, group);
    const int64_t i = tile * BS + threadIdx.x;
    if (i >= N) return;
    const f3 z = c16_row_sum<KT>(i, K, c16, c16_base, ovf, w, x);
    const f3 bb = ld3(b, i);
    const float a = alpha ? alpha[i] : 1.0f;
    st3_iter<NT>(y, i, f3{fmaf(a, z.x, bb.x), fmaf(a, z.y, bb.y), fmaf(a, z.z, bb.z)});
}

hipError_t launch_spmv_c16(int64_t N, int K, const int16_t* c16, const uint32_t* c16_base, const int32_t* ovf,
                           const int32_t* col, const float* w, const float* x, const float* b, const float* alpha,
                           float* y, hipStream_t s, int tile, int tile_group) {
    if (N == 0) return hipSuccess;
    if (ell_k4(K) > 32) return launch_spmv_ell(N, K, col, w, x, b, alpha, nullptr, y, s, tile, tile_group);
    dispatch_tile(tile, [&](auto bs) {
        constexpr int BS = decltype(bs)::value;
        dim3 grid((unsigned)div_up(N, BS)), block(BS);
        dispatch_k4(K, [&](auto kt) {
            constexpr int KT = decltype(kt)::value;
            if constexpr (KT > 0)
                dispatch_nt(N, [&](auto nt) {
                    hipLaunchKernelGGL((k_spmv_c16<KT, BS, decltype(nt)::value>), grid, block, 0, s, N, K, c16,
                                       c16_base, ovf, w, x, b, alpha, y, tile_group);
                });
        });
    });
    return hipGetLastError();
}

// A caller's CSR must have the k-nearest layout, row i = [i K, (i+1) K):
// the kernels of pg_edges / pg_propagate index col and w as i K + l.
__global__ __launch_bounds__(kBlock) void k_check_rows(int64_t N, int K, const int64_t* __restrict__ row_ptr,
                                                       int32_t* flag) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i <= N && row_ptr[i] != i * (int64_t)K) set_flag(flag, kFlagRows);
}

hipError_t launch_check_rows(int64_t N, int K, const int64_t* row_ptr, int32_t* flag, hipStream_t s) {
    hipLaunchKernelGGL(k_check_rows, dim3((unsigned)div_up(N + 1, kBlock)), dim3(kBlock), 0, s, N, K, row_ptr,
                       flag);
    return hipGetLastError();
}

// ------------------------------------- a caller's graph in sorted order ---
// pg_propagate takes rows and ids in path order, where neighbours lie anywhere
// in memory: every gathered x costs a cache line of its own (5M vertices, K =
// 16: 970 us an iteration, 1.1 TB/s of the bytes it needs).  Moved once to the
// spatially sorted order, the iteration runs as the render's does (product 141 us,
// shift 25 us).
//
// Where a graph's ids are near each other in path order already, that is as fast
// there (the identity in place of the permutation); where they are far in space
// too, no order helps, and from kPlaceRowsMinN vertices on the caller's own rows are
// read (below, the test in each iteration costs more than it saves).  Which it is, a
// sample says: the share of edges farther than a compact id reaches, in path order,
// and that of edges longer than half the radius of the vertices that an XCD works on
// at a time (65536; in space).  5M vertices, K = 16, D = 64, in path order / always
// sorted / so: neighbours 92 / 16.8 / 16.9 ms, ids within 40 rows 26 / 99 / 9.8, ids at
// random 92 / 106 / 94; D = 3: 4.3 / 2.6 / 2.6, 1.26 / 6.9 / 1.20, 4.5 / 8.4 / 4.7.  At 1M,
// D = 64, ids at random: 13.6 / 15.8 / 15.3.
constexpr int kPlaceSamples = 128, kPlaceLanes = 8, kPlaceMaxK = 32;
constexpr int64_t kPlaceRowsMinN = 1 << 21;
__global__ __launch_bounds__(kPlaceSamples* kPlaceLanes) void k_place(int64_t N, int K, int D,
                                                                      const int32_t* __restrict__ col,
                                                                      const float* __restrict__ pos, float reach,
                                                                      bool rows, int32_t* __restrict__ place) {
    constexpr int M = kPlaceMaxK / kPlaceLanes;
    __shared__ int edges, far_path, far_space;
    if (threadIdx.x == 0) edges = far_path = far_space = 0;
    __syncthreads();
    const int64_t i = (int64_t)(threadIdx.x / kPlaceLanes) * N / kPlaceSamples;
    const f3 p = ld3(pos, i);
    int32_t j[M];   // all ids in flight, then all positions: two waits for memory
    f3 q[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int l = threadIdx.x % kPlaceLanes + m * kPlaceLanes;
        j[m] = l < K ? col[i * K + l] : -1;
    }
#pragma unroll
    for (int m = 0; m < M; ++m) q[m] = ld3(pos, (uint32_t)j[m] < (uint32_t)N ? j[m] : i);
    int n = 0, fp = 0, fs = 0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const bool ok = (uint32_t)j[m] < (uint32_t)N;
        n += ok;
        fp += ok && (j[m] - i < -32767 || j[m] - i > 32767);
        fs += !(fabsf(q[m].x - p.x) <= reach && fabsf(q[m].y - p.y) <= reach && fabsf(q[m].z - p.z) <= reach);
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        n += __shfl_xor(n, o, kWave);
        fp += __shfl_xor(fp, o, kWave);
        fs += __shfl_xor(fs, o, kWave);
    }
    if (threadIdx.x % kWave == 0) {
        atomicAdd(&edges, n);
        atomicAdd(&far_path, fp);
        atomicAdd(&far_space, fs);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    // moving an edge costs about what two iterations save where it is brought near
    const bool sorted = (int64_t)(far_path - far_space) * D >= 2 * edges;
    *place = sorted ? kPlaceSorted : (rows && 2 * far_path >= edges ? kPlaceRows : kPlacePaths);
}

hipError_t launch_place(int64_t N, int K, int D, const int32_t* col, const float* pos, int32_t* place, hipStream_t s) {
    const float reach = 0.25f * cbrtf(65536.0f / (float)N);
    hipLaunchKernelGGL(k_place, dim3(1), dim3(kPlaceSamples * kPlaceLanes), 0, s, N, K, D, col, pos, reach,
                       N >= kPlaceRowsMinN, place);
    return hipGetLastError();
}

// Row s of the sliced ELL = row perm[s] of the caller's, ids through inv, with
// b, L_0, albedo and successors beside it.  Ids from callers are not trusted:
// one out of range points at row N, which holds 0, with weight 0 (x has N + 1
// rows); the padding slots hold the row itself and are left out of the sums.  One thread per quad, a row's
// quads in neighbouring lanes, so its 4 K bytes are read from whole lines.
__global__ __launch_bounds__(kBlock) void k_relayout(int64_t N, int K, const int32_t* __restrict__ perm,
                                                     const int32_t* __restrict__ inv, const int32_t* __restrict__ col,
                                                     const float* __restrict__ w, const float* __restrict__ b,
                                                     const float* __restrict__ x0, const float* __restrict__ alpha,
                                                     const int32_t* __restrict__ succ, int32_t* __restrict__ scol,
                                                     float* __restrict__ sw, float* __restrict__ sb,
                                                     float* __restrict__ sx, float* __restrict__ salpha,
                                                     int32_t* __restrict__ ssucc, const int32_t* __restrict__ place) {
    const int nq = ell_k4(K) / 4;
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t == 0) st3(sx, N, f3{0.f, 0.f, 0.f});
    const int64_t s = t / nq;
    if (s >= N) return;
    const int q = (int)(t - s * nq);
    const int64_t v = perm[s];
    const int64_t row = v * (int64_t)K;
    if (*place != kPlaceRows) {
        int32_t j[4];
        float ww[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int l = 4 * q + c;
            j[c] = l < K ? col[row + l] : -1;
            ww[c] = l < K ? w[row + l] : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool ok = (uint32_t)j[c] < (uint32_t)N;
            j[c] = ok ? inv[j[c]] : (4 * q + c < K ? (int32_t)N : (int32_t)s);
            ww[c] = ok ? ww[c] : 0.0f;
        }
        const int64_t e = ell_row(s, K) + q * kQuadStride;
        *reinterpret_cast<i32x4*>(scol + e) = i32x4{j[0], j[1], j[2], j[3]};
        *reinterpret_cast<f32x4*>(sw + e) = f32x4{ww[0], ww[1], ww[2], ww[3]};
    }
    if (q != 0) return;
    st3(sb, s, ld3(b, v));
    st3(sx, s, ld3(x0, v));
    salpha[s] = alpha[v];
    const int32_t u = succ[v];
    ssucc[s] = u >= 0 ? inv[u] : -1;
}

hipError_t launch_relayout(int64_t N, int K, const int32_t* perm, const int32_t* inv, const int32_t* col,
                           const float* w, const float* b, const float* x0, const float* alpha,
                           const int32_t* succ, int32_t* scol, float* sw, float* sb, float* sx, float* salpha,
                           int32_t* ssucc, const int32_t* place, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_relayout, dim3((unsigned)div_up(N * (ell_k4(K) / 4), kBlock)), dim3(kBlock), 0, s, N, K, perm,
                       inv, col, w, b, x0, alpha, succ, scol, sw, sb, sx, salpha, ssucc, place);
    return hipGetLastError();
}

// The rows of a block as k_spmv takes them, a group of KP lanes each, over the
// caller's arrays.
template <int KP, int BS>
__device__ __forceinline__ void spmv_rows(int64_t N, int K, const int32_t* __restrict__ col,
                                          const float* __restrict__ w, const float* __restrict__ x,
                                          const float* __restrict__ b, const float* __restrict__ alpha,
                                          float* __restrict__ y) {
#pragma clang fp contract(off)
    constexpr int GR = BS / KP, U = KP < 4 ? KP : 4;   // U rows of a group in flight
    const int lane = threadIdx.x % KP;
    const int64_t first = (int64_t)blockIdx.x * BS + threadIdx.x / KP;
    for (int r = 0; r < KP; r += U) {
        f3 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = first + (r + u) * GR;
            a[u] = f3{0.f, 0.f, 0.f};
            if (i < N && lane < K) {
                const int64_t e = i * K + lane;
                const int64_t j = col[e];
                const float ww = w[e];
                if (j >= 0 && j < N) {
                    const f3 xv = ld3(x, j);
                    a[u] = f3{ww * xv.x, ww * xv.y, ww * xv.z};
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = first + (r + u) * GR;
            const f3 z{group_sum<KP>(a[u].x), group_sum<KP>(a[u].y), group_sum<KP>(a[u].z)};
            if (i >= N || lane != 0) continue;
            const f3 bb = ld3(b, i);
            const float al = alpha[i];
            st3(y, i, f3{fmaf(al, z.x, bb.x), fmaf(al, z.y, bb.y), fmaf(al, z.z, bb.z)});
        }
    }
}

// One thread per row over the compact ids, every product rounded and the K
// products added pairwise in the order of k_spmv's lane reduction (slot l with
// slot l + KP/2, then KP/4, ..., the slots past K contributing 0), so the two
// give the same results bit for bit.  Left to itself the compiler interleaves
// gathers and products (73 registers at K = 16, 210 us on 5M vertices); with all
// gathers issued first (86 registers) it takes 141 us.
template <int KT, int BS, bool NT, bool ROWS>
__global__ __launch_bounds__(BS) void k_spmv_sorted(int64_t N, int K, const int16_t* __restrict__ c16,
                                                    const uint16_t* __restrict__ start,
                                                    const uint32_t* __restrict__ c16_base,
                                                    const int32_t* __restrict__ ovf, const float* __restrict__ w,
                                                    const float* __restrict__ x, const float* __restrict__ b,
                                                    const float* __restrict__ alpha, float* __restrict__ y,
                                                    const int32_t* __restrict__ col_rows,
                                                    const float* __restrict__ w_rows,
                                                    const int32_t* __restrict__ place) {
#pragma clang fp contract(off)
    constexpr int NQ = KT / 4, KP = KT <= 4 ? 4 : (KT <= 8 ? 8 : (KT <= 16 ? 16 : 32));
    if (ROWS && *place == kPlaceRows) {
        spmv_rows<KP, BS>(N, K, col_rows, w_rows, x, b, alpha, y);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= N) return;
    const int64_t base = ell_row(i, K);
    f32x4 ww[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) ww[q] = ld_quad_nt(w + base + q * kQuadStride);
    int32_t j[KT];
    c16_row_ids<KT, true>(i, K, c16, c16_base, ovf, j, start);
    f3 a[KP];
#pragma unroll
    for (int l = 0; l < KT; ++l) a[l] = ld3(x, j[l]);
    __builtin_amdgcn_sched_barrier(0);   // every gather in flight before the first product
#pragma unroll
    for (int l = 0; l < KP; ++l) {
        const float wl = l < KT ? ww[(l < KT ? l : 0) >> 2][l & 3] : 0.0f;
        a[l] = l < K && l < KT ? f3{wl * a[l].x, wl * a[l].y, wl * a[l].z} : f3{0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int o = KP / 2; o > 0; o >>= 1)
#pragma unroll
        for (int l = 0; l < o; ++l) a[l] = f3{a[l].x + a[l + o].x, a[l].y + a[l + o].y, a[l].z + a[l + o].z};
    const f3 bb = ld3(b, i);
    const float al = alpha[i];
    st3_iter<NT>(y, i, f3{fmaf(al, a[0].x, bb.x), fmaf(al, a[0].y, bb.y), fmaf(al, a[0].z, bb.z)});
}

hipError_t launch_spmv_sorted(int64_t N, int K, const int16_t* c16, const uint16_t* start, const uint32_t* c16_base,
                              const int32_t* ovf, const float* w, const float* x, const float* b, const float* alpha,
                              float* y, const int32_t* col_rows, const float* w_rows, const int32_t* place,
                              hipStream_t s) {
    if (N == 0) return hipSuccess;
    constexpr int BS = 512;   // as the render's aggregation over the compact ids
    dispatch_k4(K, [&](auto kt) {
        constexpr int KT = decltype(kt)::value;
        if constexpr (KT > 0)
            dispatch_nt(N, [&](auto nt) {
                auto go = [&](auto rows) {
                    hipLaunchKernelGGL((k_spmv_sorted<KT, BS, decltype(nt)::value, decltype(rows)::value>),
                                       dim3((unsigned)div_up(N, BS)), dim3(BS), 0, s, N, K, c16, start, c16_base, ovf,
                                       w, x, b, alpha, y, col_rows, w_rows, place);
                };
                if (N >= kPlaceRowsMinN) go(std::true_type{});
                else go(std::false_type{});
            });
    });
    return hipGetLastError();
}

// L(v) = y(succ v), 0 at a path's end.  Two vertices per thread, strided by
// the grid so every access stays coalesced, for two independent gathers; the
// successor ids (read once) are streamed.
// Every load is unconditional (indices clamped to a valid element, the value
// masked afterwards), so both successor ids and then both gathers are in
// flight together instead of each waiting at a branch.
constexpr int kShiftPer = 2;
template <int BS, bool NT>
__global__ __launch_bounds__(BS) void k_shift(int64_t N, const int32_t* __restrict__ succ,
                                              const float* __restrict__ y, float* __restrict__ x) {
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t v0 = tile * (int64_t)BS * kShiftPer + threadIdx.x;
    int32_t u[kShiftPer];
#pragma unroll
    for (int k = 0; k < kShiftPer; ++k) {
        const int64_t v = v0 + (int64_t)k * BS;
        u[k] = __builtin_nontemporal_load(succ + (v < N ? v : N - 1));
    }
    f3 val[kShiftPer];
#pragma unroll
    for (int k = 0; k < kShiftPer; ++k) val[k] = ld3(y, u[k] > 0 ? u[k] : 0);
    // an empty asm that takes every gathered value keeps the compiler from
    // sinking one vertex's loads into its guarded store (which serialises
    // the two load chains)
    asm volatile("" ::"v"(val[0].x), "v"(val[0].y), "v"(val[0].z), "v"(val[1].x), "v"(val[1].y), "v"(val[1].z));
    static_assert(kShiftPer == 2, "the asm above names two vertices");
#pragma unroll
    for (int k = 0; k < kShiftPer; ++k) {
        const int64_t v = v0 + (int64_t)k * BS;
        if (u[k] < 0) val[k] = f3{0.f, 0.f, 0.f};
        if (v < N) st3_iter<NT>(x, v, val[k]);
    }
}

hipError_t launch_shift(int64_t N, const int32_t* succ, const float* y, float* x, hipStream_t s, int tile) {
    if (N == 0) return hipSuccess;
    dispatch_tile(tile, [&](auto bs) {
        constexpr int BS = decltype(bs)::value;
        dispatch_nt(N, [&](auto nt) {
            hipLaunchKernelGGL((k_shift<BS, decltype(nt)::value>), dim3((unsigned)div_up(N, (int64_t)BS * kShiftPer)),
                               dim3(BS), 0, s, N, succ, y, x);
        });
    });
    return hipGetLastError();
}

// Row v of the shifted operator = albedo_u * row u of W, constant c_v = b_u,
// u = succ(v); a row without successor keeps zero weights (self columns).
// All slots of the row's quads are written (the padding slots of W hold
// (u, 0), so they become weight-0 slots here too).
__global__ __launch_bounds__(kBlock) void k_shifted_build(int64_t N, int K, const int32_t* __restrict__ succ,
                                                          const int32_t* __restrict__ col,
                                                          const float* __restrict__ w, const float* __restrict__ b,
                                                          const float* __restrict__ alpha,
                                                          int32_t* __restrict__ mcol, float* __restrict__ mw,
                                                          float* __restrict__ c) {
    const int K4 = ell_k4(K);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N * (int64_t)K4) return;
    const int64_t v = t / K4;
    const int k = (int)(t - v * K4);
    const int64_t u = succ[v];
    const int64_t e = eidx(v, k, K);
    if (u >= 0) {
        mcol[e] = col[eidx(u, k, K)];
        mw[e] = alpha[u] * w[eidx(u, k, K)];
    } else {
        mcol[e] = (int32_t)v;
        mw[e] = 0.0f;
    }
    if (k == 0) st3(c, v, u >= 0 ? ld3(b, u) : f3{0.f, 0.f, 0.f});
}

hipError_t launch_shifted_build(int64_t N, int K, const int32_t* succ, const int32_t* col, const float* w,
                                const float* b, const float* alpha, int32_t* mcol, float* mw, float* c,
                                hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_shifted_build, dim3((unsigned)div_up(N * (int64_t)ell_k4(K), kBlock)), dim3(kBlock), 0, s,
                       N, K, succ, col, w, b, alpha, mcol, mw, c);
    return hipGetLastError();
}

hipError_t launch_spmv_shifted(int64_t N, int K, const int32_t* succ, const int32_t* mcol, const float* mw,
                               const float* c, const float* x, float* xn, hipStream_t s) {
    return launch_spmv_ell(N, K, mcol, mw, x, c, nullptr, succ, xn, s);
}

// ------------------------------------------------------------- pixels ---
// o_p as in the "Final output" paragraph with the non-aggregated direct term at
// the first vertex ("Handling direct Light") -- or the estimate of the extra
// samples recorded there -- and that vertex's volume emission.  inv == NULL:
// local ids are path-order ids; r == NULL / alpha == NULL: computed from the
// path records.
//
// S groups of KP lanes per pixel, inside one wave: group g takes the samples g,
// g + S, ... of the pixel, lane l of it the l-th neighbour of the sample's first
// vertex.  Bound by the latency of offset -> id -> neighbour -> value: one
// thread per pixel walked spp K such chains (31 us for 4096 pixels at 4 samples,
// k = 8; 886 us for 512 x 512 at k = 16); with the neighbours and samples side
// by side a wave waits for one (5 and 225 us).  Products and sums are in double
// precision, hidden behind the loads: in single precision, split over lanes, the
// image was 4% further off than by one thread's chain of fused operations.
//
// Extra samples at the first vertex are read by all lanes of the group, from
// kExtraSpread of them on: the records of a path lie side by side, which one lane
// reads line by line (512 x 512 at 4 samples, k = 16: 16 extra samples 0.57 -> 0.25
// ms; two 0.23 either way, one 0.20 and 0.22).
constexpr int kExtraSpread = 3;
template <int KP, int S, bool SPREAD>
__global__ __launch_bounds__(kBlock) void k_pixels(int64_t px0, pg_paths P, Consts c, const int32_t* __restrict__ inv,
                                                   const int32_t* __restrict__ col, const float* __restrict__ w,
                                                   const float* __restrict__ x, const float* __restrict__ dpt,
                                                   const float* __restrict__ r, const float* __restrict__ alpha,
                                                   float* __restrict__ image, int32_t* flag) {
    constexpr int W = KP * S;   // lanes per pixel, a power of two <= 64
    const int lane = threadIdx.x % KP, grp = threadIdx.x % W / KP;
    const int64_t npix = (int64_t)P.width * P.height;
    const int64_t N = P.n_vertices;
    const int K = c.K;
    const int64_t px = px0 + ((int64_t)blockIdx.x * kBlock + threadIdx.x) / W;
    double sx = 0.0, sy = 0.0, sz = 0.0;
    for (int k0 = 0; k0 < P.spp; k0 += S) {   // the same trips on every lane: all take part in the sums
        const int k = k0 + grp;
        const int64_t p = px * P.spp + k;
        const bool path = px < npix && k < P.spp;
        int64_t a = 0;
        bool on = false;
        if (path) {
            a = P.path_offsets[p];
            const int64_t e = P.path_offsets[p + 1];
            on = e > a;
            if (on && (a < 0 || e > N)) {
                if (lane == 0) set_flag(flag, kFlagOffsets);
                on = false;
            }
        }
        const int64_t s0 = on ? (inv ? (int64_t)inv[a] : a) : 0;
        double ix = 0.0, iy = 0.0, iz = 0.0;
        if (c.final_gather == 0) {
            if (on && lane < K) {
                const int64_t e = inv ? eidx(s0, lane, K) : s0 * K + lane;
                const int64_t j = col[e];
                if (j < 0 || j >= N) {
                    set_flag(flag, kFlagIndex);
                } else {
                    const double ww = w[e];
                    const f3 xv = ld3(x, j);
                    ix = ww * xv.x;
                    iy = ww * xv.y;
                    iz = ww * xv.z;
                }
            }
            ix = group_sum<KP>(ix);
            iy = group_sum<KP>(iy);
            iz = group_sum<KP>(iz);
        } else if (on && lane == 0) {
            double rr;
            if (r) {
                rr = r[s0];
            } else {
                const f3 t = ld3(P.dir_in, a), wo = ld3(P.dir_out, a);
                const float u = one_minus_cos(t, wo);
                rr = c.rho(u) / c.pdf(u);
            }
            ix = rr * x[3 * s0];
            iy = rr * x[3 * s0 + 1];
            iz = rr * x[3 * s0 + 2];
        }
        f3 spread{0.f, 0.f, 0.f};
        if (SPREAD && on)
            spread = extra_direct<KP>(P, p, a, ld3(P.dir_in, a), c.rho, c.g, c.sun, c.env_pdf, nullptr, lane);
        if (lane != 0) continue;
        if (path) {
            sx += P.e_cam[3 * p];
            sy += P.e_cam[3 * p + 1];
            sz += P.e_cam[3 * p + 2];
        }
        if (!on) continue;
        float al;
        if (alpha) {
            al = alpha[s0];
        } else if (P.albedo_grid) {
            uint32_t idx[8];
            float tw[8];
            trilerp_corners(P.albedo_grid_res, P.pos[3 * a], P.pos[3 * a + 1], P.pos[3 * a + 2], idx, tw);
            al = 0.0f;
            for (int q = 0; q < 8; ++q) al = fmaf(tw[q], P.albedo_grid[idx[q]], al);
        } else {
            al = P.albedo[a];
        }
        if (P.l_emit) {   // volume emission of the first vertex, seen by the camera unscattered
            sx += P.l_emit[3 * a];
            sy += P.l_emit[3 * a + 1];
            sz += P.l_emit[3 * a + 2];
        }
        f3 dd = SPREAD ? spread : ld3(dpt, s0);
        if (!SPREAD && P.n_extra > 0)
            dd = extra_direct(P, p, a, ld3(P.dir_in, a), c.rho, c.g, c.sun, c.env_pdf, nullptr);
        sx = fma((double)al, (double)dd.x + ix, sx);
        sy = fma((double)al, (double)dd.y + iy, sy);
        sz = fma((double)al, (double)dd.z + iz, sz);
    }
    // the groups' sums (held by their lanes 0)
#pragma unroll
    for (int o = KP; o < W; o <<= 1) {
        sx += __shfl_xor(sx, o, kWave);
        sy += __shfl_xor(sy, o, kWave);
        sz += __shfl_xor(sz, o, kWave);
    }
    if (px >= npix || lane != 0 || grp != 0) return;
    const double inv_spp = (double)(1.0f / (float)P.spp);   // the factor of the output's adjoint
    image[3 * px] = (float)(sx * inv_spp);
    image[3 * px + 1] = (float)(sy * inv_spp);
    image[3 * px + 2] = (float)(sz * inv_spp);
}

// A launch has fewer than 2^32 threads: an image of more goes in pieces (a loop over
// the pixels in the kernel cost 6%).
constexpr int64_t kMaxBlocks = (int64_t(1) << 32) / kBlock - 1;

hipError_t launch_pixels(const pg_paths& paths, const Consts& c, const int32_t* inv, const int32_t* col,
                         const float* w, const float* x, const float* dpt, const float* r, const float* alpha,
                         float* image, int32_t* flag, hipStream_t s) {
    const int64_t npix = (int64_t)paths.width * paths.height;
    if (npix == 0) return hipSuccess;
    auto go = [&](auto kp, auto sg) {
        constexpr int KP = decltype(kp)::value, S = decltype(sg)::value;
        constexpr int64_t kRow = kBlock / (KP * S), kAll = kMaxBlocks * kRow;   // pixels of a block, of a launch
        auto launch = [&](auto spread) {
            for (int64_t px0 = 0; px0 < npix; px0 += kAll)
                hipLaunchKernelGGL((k_pixels<KP, S, decltype(spread)::value>),
                                   dim3((unsigned)div_up(std::min(npix - px0, kAll), kRow)), dim3(kBlock), 0, s, px0,
                                   paths, c, inv, col, w, x, dpt, r, alpha, image, flag);
        };
        if (KP > 1 && paths.n_extra >= kExtraSpread) launch(std::bool_constant<(KP > 1)>{});
        else launch(std::false_type{});
    };
    // The own sample's term (final_gather 1) has no neighbours, so lanes only for the
    // extra samples, eight from five of them on (1920 x 1080, one / eight lanes: none 0.035
    // ms and, with K = 8 lanes, 0.11; four 0.11 / 0.22; eight 0.49 / 0.24; 16 1.72 / 0.31).
    const int lanes = c.final_gather == 0 ? c.K : paths.n_extra >= 5 ? 8 : 1;
    dispatch_kp(lanes, [&](auto kp) {   // up to four samples side by side, as many as fit a wave
        constexpr int KP = decltype(kp)::value, S4 = KP <= 16 ? 4 : 64 / KP, S2 = KP <= 32 ? 2 : 1;
        if (paths.spp >= 3) go(kp, std::integral_constant<int, S4>{});
        else if (paths.spp == 2) go(kp, std::integral_constant<int, S2>{});
        else go(kp, std::integral_constant<int, 1>{});
    });
    return hipGetLastError();
}

// ----------------------------------------------------------- utilities ---

// gather:  dst[i] = src[idx[i]];  scatter: dst[idx[i]] = src[i]   (float3 rows)
__global__ __launch_bounds__(kBlock) void k_permute3(int64_t N, const int32_t* __restrict__ idx,
                                                     const float* __restrict__ src, float* __restrict__ dst,
                                                     int gather) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int64_t j = idx[i];
    if (gather) st3(dst, i, ld3(src, j));
    else st3(dst, j, ld3(src, i));
}

hipError_t launch_permute3(int64_t N, const int32_t* idx, const float* src, float* dst, int gather,
                           hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_permute3, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, idx, src, dst,
                       gather);
    return hipGetLastError();
}

// Fill bytes with a 32-bit pattern (a kernel, not a memset node, so the
// sequence can be captured in a graph).
__global__ __launch_bounds__(kBlock) void k_fill(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_fill(void* p, size_t bytes, hipStream_t s) {
    const int64_t n = (int64_t)(bytes / 4);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)div_up(n, kBlock)), dim3(kBlock), 0, s, (uint32_t*)p, n, 0u);
    return hipGetLastError();
}

hipError_t launch_fill_value(void* p, size_t bytes, uint32_t v, hipStream_t s) {
    const int64_t n = (int64_t)(bytes / 4);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)div_up(n, kBlock)), dim3(kBlock), 0, s, (uint32_t*)p, n, v);
    return hipGetLastError();
}

}  // namespace pg
