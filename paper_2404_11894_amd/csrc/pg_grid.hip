// pg_grid.hip -- uniform-grid build (counting sort) and exact k-nearest-
// neighbour query on quantised integer coordinates.
//
// The paper builds a hash grid over the shading points and searches the
// neighbouring bins (Sec. "Rendering System", path graph solver).  Here the
// neighbourhood of vertex i is exact: i first, then the K-1 nearest others by
// (squared distance of the 20-bit quantised positions, path-order id).
//
// Grid: cell = q >> shift per axis, G = 2^(20-shift) cells per axis.  The
// vertices are sorted by the position of their cell along the Hilbert curve,
// so neighbouring cells are close in memory (the gathers of the kNN, the
// edge weights and every propagation step stay in a small window); a row-major
// table gives each cell's [start, end) in that order without re-encoding during
// the search.  Counting sort = atomic
// histogram (which also yields each vertex's rank inside its cell) +
// exclusive scan + scatter.  The order of vertices inside a cell is not
// deterministic; nothing downstream depends on it (every comparison breaks
// ties by path-order id).
#include "pg_internal.h"

namespace pg {

__device__ inline uint32_t quant(float x) {
    float s = floorf(x * 1048576.0f);   // exact: scaling by 2^20
    if (!(s >= 0.0f)) s = 0.0f;          // also NaN
    if (s > (float)kQMax) s = (float)kQMax;
    return (uint32_t)s;
}

__device__ __forceinline__ void count_vertex(int64_t i, float x, float y, float z, int shift,
                                             uint32_t* __restrict__ count, uint32_t* __restrict__ cellid,
                                             uint32_t* __restrict__ rank, int32_t* flag) {
    if (!(x >= 0.0f && x <= 1.0f && y >= 0.0f && y <= 1.0f && z >= 0.0f && z <= 1.0f)) set_flag(flag, kFlagPos);
    uint32_t c = hilbert3(quant(x) >> shift, quant(y) >> shift, quant(z) >> shift, kQBits - shift);
    cellid[i] = c;
    rank[i] = atomicAdd(&count[c], 1u);
}

__global__ __launch_bounds__(kBlock) void k_quantize_count(int64_t N, const float* __restrict__ pos, int shift,
                                                           uint32_t* __restrict__ count,
                                                           uint32_t* __restrict__ cellid,
                                                           uint32_t* __restrict__ rank, int32_t* flag,
                                                           const int32_t* __restrict__ as_given) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N || (as_given && *as_given != 0)) return;
    count_vertex(i, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], shift, count, cellid, rank, flag);
}

hipError_t launch_quantize_count(int64_t N, const float* pos, int shift, uint32_t* count, uint32_t* cellid,
                                 uint32_t* rank, int32_t* flag, hipStream_t s, const int32_t* as_given) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_quantize_count, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, pos, shift,
                       count, cellid, rank, flag, as_given);
    return hipGetLastError();
}

// range[(z G + y) G + x] = [start, end) of cell (x, y, z), from the exclusive
// scan `start` of the counts in Hilbert order.  Row-major, so that the search
// reaches the cell at a wave-uniform offset with one scalar add.
__global__ __launch_bounds__(kBlock) void k_cell_range(int64_t ncells, int shift, const uint32_t* __restrict__ start,
                                                       uint2* __restrict__ range) {
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= ncells) return;
    const int lg = kQBits - shift;
    const uint32_t u = (uint32_t)m, mask = (1u << lg) - 1u;
    const uint32_t h = hilbert3(u & mask, (u >> lg) & mask, u >> (2 * lg), lg);
    range[m] = make_uint2(start[h], start[h + 1]);
}

hipError_t launch_cell_range(int64_t ncells, int shift, const uint32_t* start, uint2* range, hipStream_t s) {
    hipLaunchKernelGGL(k_cell_range, dim3((unsigned)div_up(ncells, kBlock)), dim3(kBlock), 0, s, ncells, shift,
                       start, range);
    return hipGetLastError();
}

// ------------------------------------------------------------------ scan ---
// Exclusive prefix sum of n uint32 counts into the n + 1 elements of out, out[n] =
// total.  Three passes: per-block totals, a scan of the block totals, per-block
// scans with offset.  Inside a block: per-thread serial sums, a wave-level
// inclusive scan with lane shuffles, and a scan of the wave totals through LDS.

constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

__device__ inline uint32_t wave_inclusive(uint32_t v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive scan across the block of one value per thread; returns the
// thread's exclusive prefix and the block total.
__device__ inline uint32_t block_exclusive(uint32_t v, uint32_t& total) {
    __shared__ uint32_t wsum[kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    uint32_t inc = wave_inclusive(v);
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) {
        uint32_t x = wsum[w];
        if (w < wid) off += x;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return off + inc - v;
}

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                        uint32_t* __restrict__ partials) {
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) s += in[base + k];
    uint32_t total;
    block_exclusive(s, total);
    if (threadIdx.x == 0) partials[blockIdx.x] = total;
}

// one block scans nb partials in tiles, carrying the running offset
__global__ __launch_bounds__(kBlock) void k_scan_partials(uint32_t* __restrict__ partials, int64_t nb) {
    uint32_t carry = 0;
    for (int64_t base = 0; base < nb; base += kScanTile) {
        int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
        uint32_t v[kScanItems];
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = (i0 + k < nb) ? partials[i0 + k] : 0u;
            s += v[k];
        }
        uint32_t total;
        uint32_t ex = block_exclusive(s, total) + carry;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i0 + k < nb) partials[i0 + k] = ex;
            ex += v[k];
        }
        carry += total;
    }
}

__global__ __launch_bounds__(kBlock) void k_scan_down(const uint32_t* in, uint32_t* out, int64_t n,
                                                      const uint32_t* __restrict__ partials) {
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t total;
    uint32_t ex = block_exclusive(s, total) + partials[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = ex;
        ex += v[k];
    }
    // the last element of the last block closes the prefix sum
    if (base < n && base + kScanItems >= n) out[n] = ex;
}

// The whole scan in one block, tile by tile: one launch instead of three where
// there is little to scan (4096 cells: 2 us instead of 3 x 3).
constexpr int64_t kScanOne = 8 * kScanTile;
__global__ __launch_bounds__(kBlock) void k_scan_one(const uint32_t* in, uint32_t* out, int64_t n) {
    uint32_t carry = 0;
    for (int64_t tile = 0; tile < n; tile += kScanTile) {
        const int64_t base = tile + (int64_t)threadIdx.x * kScanItems;
        uint32_t v[kScanItems];
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = (base + k < n) ? in[base + k] : 0u;
            s += v[k];
        }
        uint32_t total;
        uint32_t ex = block_exclusive(s, total) + carry;   // its barriers order the reads before the writes
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (base + k < n) out[base + k] = ex;
            ex += v[k];
        }
        carry += total;
    }
    if (threadIdx.x == 0) out[n] = carry;
}

size_t scan_partials_bytes(int64_t n) { return (size_t)(div_up(n, kScanTile) + 1) * sizeof(uint32_t); }

hipError_t launch_scan_exclusive(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* partials,
                                 hipStream_t s) {
    if (n <= 0) return hipErrorInvalidValue;
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kBlock), 0, s, in, out, n);
        return hipGetLastError();
    }
    int64_t nb = div_up(n, kScanTile);
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kBlock), 0, s, in, n, partials);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kBlock), 0, s, partials, nb);
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, n, partials);
    return hipGetLastError();
}

// --------------------------------------------------------------- scatter ---

// Cell-centred trilinear albedo of a grid [R][R][R] (z, y, x).
__device__ inline float trilerp_alpha(const float* grid, int R, float px, float py, float pz) {
    uint32_t idx[8];
    float w[8];
    trilerp_corners(R, px, py, pz, idx, w);
    float a = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) a = fmaf(w[c], grid[idx[c]], a);
    return a;
}

__device__ inline void fill_record(const pg_paths& P, int64_t v, VRec& r) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.t[a] = P.dir_in[3 * v + a];
        r.w[a] = P.dir_out[3 * v + a];
        r.we[a] = P.dir_env[3 * v + a];
        r.ls[a] = P.l_sun[3 * v + a];
        r.le[a] = P.l_env[3 * v + a];
        r.lp[a] = P.l_phase[3 * v + a];
    }
    r.alpha = P.albedo_grid ? trilerp_alpha(P.albedo_grid, P.albedo_grid_res, P.pos[3 * v], P.pos[3 * v + 1],
                                            P.pos[3 * v + 2])
                            : P.albedo[v];
    r.pad = 0.0f;
}

__device__ inline void store_record(VRec* dst, const VRec& r) {
    const float4* s4 = reinterpret_cast<const float4*>(&r);
    float4* d4 = reinterpret_cast<float4*>(dst);
#pragma unroll
    for (int k = 0; k < 5; ++k) d4[k] = s4[k];
}

__global__ __launch_bounds__(kBlock) void k_scatter(int64_t N, pg_paths P,
                                                    const uint32_t* __restrict__ cellid,
                                                    const uint32_t* __restrict__ rank,
                                                    const uint32_t* __restrict__ cell_start,
                                                    int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                    uint64_t* __restrict__ qsorted, float4* __restrict__ pts,
                                                    const int32_t* __restrict__ as_given) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const bool given = as_given && *as_given != 0;
    int64_t s = given ? v : (int64_t)cell_start[cellid[v]] + rank[v];
    perm[s] = (int32_t)v;
    inv[v] = (int32_t)s;
    if (!qsorted && !pts) return;
    const uint32_t qx = quant(P.pos[3 * v]), qy = quant(P.pos[3 * v + 1]), qz = quant(P.pos[3 * v + 2]);
    if (qsorted) qsorted[s] = qpack(qx, qy, qz);
    if (pts) pts[s] = make_float4((float)qx, (float)qy, (float)qz, __int_as_float((int32_t)v));   // exact: below 2^24
}

hipError_t launch_scatter(int64_t N, const pg_paths& paths, const uint32_t* cellid,
                          const uint32_t* rank, const uint32_t* cell_start, int32_t* perm, int32_t* inv,
                          uint64_t* qsorted, float4* pts, hipStream_t s, const int32_t* as_given) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, paths, cellid,
                       rank, cell_start, perm, inv, qsorted, pts, as_given);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_pack_records(int64_t N, pg_paths P, VRec* __restrict__ rec,
                                                         int32_t* flag) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    float x = P.pos[3 * v], y = P.pos[3 * v + 1], z = P.pos[3 * v + 2];
    if (!(x >= 0.0f && x <= 1.0f && y >= 0.0f && y <= 1.0f && z >= 0.0f && z <= 1.0f)) set_flag(flag, kFlagPos);
    VRec r;
    fill_record(P, v, r);
    store_record(rec + v, r);
}

// k_quantize_count and k_pack_records in one pass over the vertices: the
// atomics' latency passes behind the copy of the records, one launch less.
__global__ __launch_bounds__(kBlock) void k_count_pack(int64_t N, pg_paths P, int shift, uint32_t* __restrict__ count,
                                                       uint32_t* __restrict__ cellid, uint32_t* __restrict__ rank,
                                                       VRec* __restrict__ rec, int32_t* flag) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    count_vertex(v, P.pos[3 * v], P.pos[3 * v + 1], P.pos[3 * v + 2], shift, count, cellid, rank, flag);
    VRec r;
    fill_record(P, v, r);
    store_record(rec + v, r);
}

hipError_t launch_count_pack(int64_t N, const pg_paths& paths, int shift, uint32_t* count, uint32_t* cellid,
                             uint32_t* rank, VRec* rec, int32_t* flag, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_count_pack, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, paths, shift, count,
                       cellid, rank, rec, flag);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_alpha(int64_t N, pg_paths P, float* __restrict__ alpha) {
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    alpha[v] = P.albedo_grid ? trilerp_alpha(P.albedo_grid, P.albedo_grid_res, P.pos[3 * v], P.pos[3 * v + 1],
                                             P.pos[3 * v + 2])
                             : P.albedo[v];
}

hipError_t launch_alpha(int64_t N, const pg_paths& paths, float* alpha, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_alpha, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, paths, alpha);
    return hipGetLastError();
}

// rec[s] = recp[perm[s]]: the records packed in path order, gathered into the
// sorted order (one 80-byte read and one coalesced 80-byte write per vertex
// instead of scattering them from path order).
__global__ __launch_bounds__(kBlock) void k_gather_records(int64_t N, const int32_t* __restrict__ perm,
                                                           const VRec* __restrict__ recp, VRec* __restrict__ rec) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= N) return;
    const float4* src = reinterpret_cast<const float4*>(recp + perm[s]);
    float4* dst = reinterpret_cast<float4*>(rec + s);
    float4 v[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] = src[k];
#pragma unroll
    for (int k = 0; k < 5; ++k) dst[k] = v[k];
}

hipError_t launch_gather_records(int64_t N, const int32_t* perm, const VRec* recp, VRec* rec, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_records, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, perm, recp, rec);
    return hipGetLastError();
}

hipError_t launch_pack_records(int64_t N, const pg_paths& paths, VRec* rec, int32_t* flag, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_records, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, paths, rec,
                       flag);
    return hipGetLastError();
}

// ------------------------------------------------------------------- kNN ---
// One query per thread, queries in cell (Hilbert) order so that the lanes of a
// wave visit the same cells.  The K-1 best candidates live in registers,
// sorted ascending by (d2, id) and right-aligned in an array of KM slots; the
// KM-(K-1) leading slots hold (0, 0), which no candidate can move past, so the
// current worst is always slot KM-1 and every index is a compile-time
// constant.  Cells are searched in Chebyshev shells; after the shells up to r
// every unvisited vertex is at least `gap` quantisation steps away on some axis,
// so the search stops once the worst kept distance is < gap^2 (a candidate at
// exactly gap could still win on a smaller id).

__device__ inline bool key_less(uint64_t d1, uint32_t o1, uint64_t d2, uint32_t o2) {
    return d1 < d2 || (d1 == d2 && o1 < o2);
}

// Insert (d2, oid) into the sorted, right-aligned list if it beats the worst.
template <int KM>
__device__ __forceinline__ void list_insert(uint64_t (&d)[KM], uint32_t (&o)[KM], uint64_t d2, uint32_t oid) {
    if (key_less(d2, oid, d[KM - 1], o[KM - 1])) {
        d[KM - 1] = d2;
        o[KM - 1] = oid;
#pragma unroll
        for (int p = KM - 1; p > 0; --p) {
            const bool sw = key_less(d[p], o[p], d[p - 1], o[p - 1]);
            const uint64_t td = d[p];
            const uint32_t to = o[p];
            d[p] = sw ? d[p - 1] : d[p];
            o[p] = sw ? o[p - 1] : o[p];
            d[p - 1] = sw ? td : d[p - 1];
            o[p - 1] = sw ? to : o[p - 1];
        }
    }
}

template <int KM>
__device__ __forceinline__ void list_reset(uint64_t (&d)[KM], uint32_t (&o)[KM], int m) {
#pragma unroll
    for (int p = 0; p < KM; ++p) {
        const bool sentinel = p < KM - m;
        d[p] = sentinel ? 0ull : ~0ull;
        o[p] = sentinel ? 0u : ~0u;
    }
}

// Exact search for query s by Chebyshev shells of cells around its own.  A
// cell whose box is farther from q than the current (K-1)-th distance cannot
// contribute and is skipped without reading it (only once the list is full:
// before that the worst key is (inf, inf)); a cell at exactly that distance is
// still read, since a tie may win on id.  Candidates are loaded two at a time.
template <int KM>
__device__ __forceinline__ void shell_search(int64_t s, int shift, int32_t qx, int32_t qy, int32_t qz,
                                             const float4* __restrict__ pts, const uint2* __restrict__ cell_range,
                                             uint64_t (&d)[KM], uint32_t (&o)[KM]) {
    const int G = 1 << (kQBits - shift);
    const int cx = qx >> shift, cy = qy >> shift, cz = qz >> shift;
    const int64_t cs = (int64_t)1 << shift;
    auto offer = [&](const float4& p) {
        const int64_t ex = (int32_t)p.x - qx, ey = (int32_t)p.y - qy, ez = (int32_t)p.z - qz;
        list_insert<KM>(d, o, (uint64_t)(ex * ex + ey * ey + ez * ez), __float_as_uint(p.w));
    };
    for (int r = 0;; ++r) {
        for (int dz = -r; dz <= r; ++dz) {
            const int z = cz + dz;
            if (z < 0 || z >= G) continue;
            const int64_t gz = dz < 0 ? (int64_t)qz - ((int64_t)(z + 1) * cs - 1) : (dz > 0 ? (int64_t)z * cs - qz : 0);
            for (int dy = -r; dy <= r; ++dy) {
                const int y = cy + dy;
                if (y < 0 || y >= G) continue;
                const int64_t gy = dy < 0 ? (int64_t)qy - ((int64_t)(y + 1) * cs - 1) : (dy > 0 ? (int64_t)y * cs - qy : 0);
                const bool face = (dz == -r || dz == r || dy == -r || dy == r);
                const int step = (face || r == 0) ? 1 : 2 * r;
                for (int dx = -r; dx <= r; dx += step) {
                    const int x = cx + dx;
                    if (x < 0 || x >= G) continue;
                    const int64_t gx = dx < 0 ? (int64_t)qx - ((int64_t)(x + 1) * cs - 1) : (dx > 0 ? (int64_t)x * cs - qx : 0);
                    if ((uint64_t)(gx * gx + gy * gy + gz * gz) > d[KM - 1]) continue;   // whole cell too far
                    const uint2 cr = cell_range[((uint32_t)z * (uint32_t)G + (uint32_t)y) * (uint32_t)G + (uint32_t)x];
                    for (uint32_t t = cr.x; t < cr.y; t += 2) {
                        const bool two = t + 1 < cr.y;
                        const float4 p0 = pts[t], p1 = pts[two ? t + 1 : t];
                        if ((int64_t)t != s) offer(p0);
                        if (two && (int64_t)t + 1 != s) offer(p1);
                    }
                }
            }
        }
        // smallest per-axis distance from q to a cell outside the searched cube
        int64_t gap = INT64_MAX;
        const int c3[3] = {cx, cy, cz};
        const int64_t q3[3] = {qx, qy, qz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (c3[a] - r > 0) gap = min(gap, q3[a] - (int64_t)(c3[a] - r) * cs + 1);
            if (c3[a] + r < G - 1) gap = min(gap, (int64_t)(c3[a] + r + 1) * cs - q3[a]);
        }
        if (gap == INT64_MAX) break;                    // the whole grid was searched
        if (d[KM - 1] < (uint64_t)(gap * gap)) break;   // list full and provably final
    }
}

template <int KM>
__device__ __forceinline__ void knn_write(int64_t s, int K, int m, uint32_t self, int64_t N, const int32_t* inv,
                                          const uint64_t (&d)[KM], const uint32_t (&o)[KM], int32_t* col_sorted,
                                          int32_t* col_canon, int64_t* row_ptr) {
    (void)d;
    if (col_sorted) {   // sliced-ELL layout; the padding slots of the row's last quad point at itself
        col_sorted[eidx(s, 0, K)] = (int32_t)s;
#pragma unroll
        for (int p = 0; p < KM; ++p)
            if (p >= KM - m) col_sorted[eidx(s, 1 + p - (KM - m), K)] = inv[o[p]];
        for (int l = K; l < ell_k4(K); ++l) col_sorted[eidx(s, l, K)] = (int32_t)s;
    }
    if (col_canon) {
        int32_t* row = col_canon + (int64_t)self * K;
        row[0] = (int32_t)self;
#pragma unroll
        for (int p = 0; p < KM; ++p)
            if (p >= KM - m) row[1 + p - (KM - m)] = (int32_t)o[p];
    }
    if (row_ptr) {
        row_ptr[self] = (int64_t)self * K;
        if (s == 0) row_ptr[N] = N * (int64_t)K;
    }
}

// ---- fast path: one 64-bit key per candidate --------------------------
// key = (min(d2, sat) << idb) | id, with idb = the bits ids of this scene need
// (N - 1 < 2^idb) and sat = 2^(64 - idb) - 1, orders exactly like (d2, id) as
// long as d2 < sat.  Every scene below 2^25 vertices keeps 39 distance bits
// (no saturation below ~70% of the unit cube); at 2^31 vertices 33 bits
// (~8.8%).  A k-th neighbour that far saturates the key, and that query is
// redone by the exact search.
struct KeyFmt {
    int idb;
    uint64_t sat, idmask;
    double satd;   // sat where it can bind (d2 < 2^42), else larger than any d2
};

inline KeyFmt key_fmt(int64_t N) {
    int idb = 1;
    while (idb < 31 && ((int64_t)1 << idb) < N) ++idb;
    const uint64_t sat = (~0ull) >> idb;
    return KeyFmt{idb, sat, ((uint64_t)1 << idb) - 1, sat < (1ull << 50) ? (double)sat : 1e18};
}

// The exact key of a candidate at (dx, dy, dz) quantisation steps from the
// query.  The differences are whole numbers below 2^21, so the double-precision
// sum of squares is exact, and adding 2^52 leaves it in the mantissa's low bits.
__device__ __forceinline__ uint64_t make_key(float dx, float dy, float dz, uint32_t id, const KeyFmt& f) {
    const double x = dx, y = dy, z = dz;
    const double d2 = fmin(fma(x, x, fma(y, y, z * z)), f.satd);
    const uint64_t u = (uint64_t)__double_as_longlong(d2 + 4503599627370496.0) & 0x000fffffffffffffull;
    return (u << f.idb) | (uint64_t)id;
}

// Insert c into the ascending list (unchanged if c is not below the last key),
// as a merge: slot p keeps its key if c is not below it, takes c if c falls
// between slots p-1 and p, and the key of slot p-1 otherwise.  The comparisons
// against c are independent of each other (a bubble pass would chain them), and
// each slot costs one 64-bit compare and two selects.
template <int KM>
__device__ __forceinline__ void key_insert(uint64_t (&k)[KM], uint64_t c) {
    bool lt[KM];
    uint64_t v[KM];
#pragma unroll
    for (int p = 0; p < KM; ++p) {
        lt[p] = c < k[p];
        // an empty asm hides that v[p] equals k[p]: the selects below then
        // reuse lt[] instead of being rebuilt as min/max with compares of their own
        v[p] = k[p];
        asm("" : "+v"(v[p]));
    }
#pragma unroll
    for (int p = KM - 1; p > 0; --p) k[p] = lt[p] ? (lt[p - 1] ? v[p - 1] : c) : v[p];
    k[0] = lt[0] ? c : v[0];
}

// The search starts from the kKnnWin vertices on either side of the query in
// cell order (the nearer half first), which gives the shells a tight bound to
// prune cells with from the start; the shells then skip that index range, so
// every vertex is offered once.
constexpr int kKnnWin = 16;

// Per-lane scratch of the search, in LDS: cell ranges still to be read, and
// candidates that passed the distance filter (positions in sorted order).
// [entry][lane], so a wave's accesses never conflict.  8 + 8 entries are 6 KB a
// wave, which leaves room for the 6 waves per SIMD that the registers allow:
// 12 + 8 entries (5 waves) took 14.5 ms where these take 13.1 on 20M vertices at
// k = 16, 6 + 8 13.5 ms.
constexpr int kKnnRanges = 8;
constexpr int kKnnPend = 8;
constexpr int kKnnKeep = kKnnPend / 2;
// With lanes to spare (SUB > 1) the LDS a wider range queue takes is free: fewer
// turns, 29 thousand queries (k = 16) 0.107 -> 0.103 ms (30 ranges: from 60 thousand
// queries slower than 8).
template <int SUB>
struct KnnScratch {
    static constexpr int kRanges = SUB > 1 ? 2 * kKnnRanges : kKnnRanges;
    uint2 range[kRanges][kBlock];
    uint32_t pend[kKnnPend][kBlock];
};

// The search is bound by the instructions a wave issues (32 thousand a wave with
// 29% of the lanes active when every lane searched by itself, a dense cloud of 69M
// vertices; now 17 thousand with 90%, a fifth of a wave's cycles waiting for memory),
// and what a wave issues is the union of what its 64 lanes do.  So the lanes stay
// together wherever the work is heavy:
//  * cells are tested at offsets the whole wave shares, in single precision
//    (gap and table index a few operations each), and only queued;
//  * the queued ranges are then read as one flat loop per lane, so a wave
//    takes as many steps as its busiest lane has candidates in all, not the
//    sum over cells of the fullest lane's;
//  * a candidate is first compared in single precision with the current
//    bound, and only those that pass are queued for the sorted list, which
//    the lanes extend together (64-bit keys, exact).  When a lane's queue is
//    full, half of it is taken in; the lanes behind it catch up meanwhile.
// Single-precision values only decide what is looked at again: distances are
// rounded by at most 2^-22 of their value and the bound is raised by 2^-20, so
// nothing that could enter the list is dropped.
// Neighbour lists with the grid build, before and after: 20M vertices (k = 16)
// 17.0 -> 13.1 ms; 64M vertices at the default cells 103 -> 60 ms; 29 thousand
// (k = 8) 0.190 -> 0.070 ms, with four lanes a query (one: 0.115).
//
// SUB > 1 (few queries): a launch that leaves the chip half idle lasts as long as
// one wave's walk, so SUB neighbouring lanes share a query.  All test the same
// cells; each reads every SUB-th candidate of a range into a list of its own.
// After the seeds and after each pass over cells the lists are merged for the
// bound that the group goes on with, and in the end for the result.
template <int KM, int SUB>
struct KnnSearch {
    const float4* __restrict__ pts;
    const uint2* __restrict__ cells;
    KeyFmt f;
    float qx, qy, qz;
    uint32_t lo, nwin;      // seeded index range: [lo, lo + nwin]
    float bound;            // not below the worst kept squared distance; inf until the list is full
    int nr, np;             // queued ranges, pending candidates
    int m, sub;             // keys wanted, lane of the query's group
    uint32_t dense;         // vertices from which a cell is searched before its neighbours are queued
    uint64_t k[KM];
    KnnScratch<SUB>* sc;

    __device__ __forceinline__ float reach(uint64_t worst) const {
        return worst == ~0ull ? INFINITY : (float)(worst >> f.idb) * (1.0f + 0x1p-20f);
    }

    // g = the KM smallest keys of the group's lists (every lane the same).  Of two
    // ascending lists the smaller of g[p] and o[KM - 1 - p] are the KM smallest, up
    // and then down; half-cleaners of a power of two sort them, as if smaller keys
    // that never move stood before them.
    __device__ __forceinline__ void merge_group(uint64_t (&g)[KM]) const {
        constexpr int P = KM <= 1 ? 1 : KM <= 2 ? 2 : KM <= 4 ? 4 : KM <= 8 ? 8 : KM <= 16 ? 16 : KM <= 32 ? 32 : 64;
#pragma unroll
        for (int p = 0; p < KM; ++p) g[p] = k[p];
#pragma unroll
        for (int step = 1; step < SUB; step <<= 1) {
            uint64_t o[KM];
#pragma unroll
            for (int p = 0; p < KM; ++p) o[p] = __shfl_xor((unsigned long long)g[p], step, kWave);
            for (int i = m; i < KM; ++i) {   // without the other's leading zeros
#pragma unroll
                for (int p = 0; p + 1 < KM; ++p) o[p] = o[p + 1];
                o[KM - 1] = ~0ull;
            }
#pragma unroll
            for (int p = 0; p < KM; ++p) g[p] = g[p] < o[KM - 1 - p] ? g[p] : o[KM - 1 - p];
#pragma unroll
            for (int h = P / 2; h > 0; h >>= 1) {
#pragma unroll
                for (int i = P - KM; i + h < P; ++i) {
                    if ((i & h) == 0) {
                        const int a = i - (P - KM), b = a + h;
                        const bool swap = g[b] < g[a];
                        const uint64_t lower = swap ? g[b] : g[a], upper = swap ? g[a] : g[b];
                        g[a] = lower;
                        g[b] = upper;
                    }
                }
            }
        }
    }

    // Reads the queued ranges, one candidate per lane and step, and lets those
    // within the bound into the list.  The one place where the list grows: it is
    // unrolled over registers, and a second copy of it spills.
    __device__ __forceinline__ void drain(bool flush_all) {
        const int tid = threadIdx.x;
        int i = 0;
        uint2 r = make_uint2(0u, ~0u);
        float4 p = make_float4(NAN, 0.f, 0.f, 0.f);   // a lane without a candidate: no distance passes
        if (nr > 0) {
            r = sc->range[0][tid];
            p = pts[r.x];
        }
        for (;;) {
            const float dx = p.x - qx, dy = p.y - qy, dz = p.z - qz;
            const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            const bool take = d2 <= bound && r.x - lo > nwin;
            if (take) sc->pend[np][tid] = r.x;
            np += take ? 1 : 0;
            if ((r.x += SUB) >= r.y) {
                p.x = NAN;
                r.y = ~0u;
                if (++i < nr) r = sc->range[i][tid];
            }
            if (i < nr) p = pts[r.x];   // in flight over the next turn's bookkeeping
            const bool more = __any(i < nr);
            if (__any(np == kKnnPend) || (flush_all && !more)) {
                // no branch of its own per lane: a lane without a candidate offers
                // the largest key, which changes nothing
                const int keep = more ? kKnnKeep : 0;
                do {
                    const bool has = np > 0;
                    np -= has ? 1 : 0;
                    const float4 c = pts[has ? sc->pend[np][tid] : lo];
                    const uint64_t key = make_key(c.x - qx, c.y - qy, c.z - qz, __float_as_uint(c.w), f);
                    key_insert<KM>(k, has ? key : ~0ull);
                } while (__any(np > keep));
                bound = fminf(bound, reach(k[KM - 1]));
            }
            if (!more) break;
        }
        nr = 0;
    }

    __device__ __forceinline__ void queue(uint32_t a, uint32_t e) {
        a += (uint32_t)sub;   // 0 without groups
        if (a < e) sc->range[nr++][threadIdx.x] = make_uint2(a, e);
    }

    __device__ __forceinline__ void run(uint32_t N, uint32_t s, int shift) {
        nr = np = 0;
        bound = INFINITY;
        const uint32_t a1 = s < kKnnWin / 2 ? 0u : s - kKnnWin / 2, e1 = N - s <= kKnnWin / 2 ? N : s + kKnnWin / 2 + 1;
        const uint32_t a2 = s < kKnnWin ? 0u : s - kKnnWin, e2 = N - s <= kKnnWin ? N : s + kKnnWin + 1;
        queue(a1, s);
        queue(s + 1, e1);
        lo = s;
        nwin = 0;
        const int lg = kQBits - shift, G = 1 << lg;
        const int cx = (int)qx >> shift, cy = (int)qy >> shift, cz = (int)qz >> shift;
        const uint32_t cell0 = ((uint32_t)cz << (2 * lg)) + ((uint32_t)cy << lg) + (uint32_t)cx;
        const float cs = (float)(1 << shift);
        // distance to the neighbouring cells on either side of each axis
        const float lx = qx - (float)(cx << shift) + 1.0f, ly = qy - (float)(cy << shift) + 1.0f,
                    lz = qz - (float)(cz << shift) + 1.0f;
        const float hx = cs + 1.0f - lx, hy = cs + 1.0f - ly, hz = cs + 1.0f - lz;
        auto gap1 = [&](int d, float l, float h) {   // to the cells at offset d (uniform) on one axis; exact
            return d == 0 ? 0.0f : (d < 0 ? l + (float)(-d - 1) * cs : h + (float)(d - 1) * cs);
        };
        // Passes over the cells at Chebyshev distance (rin, rout] from the
        // query's own: first the 27 around it (where a lane's own cell is populous,
        // that one alone, and then the 26), after that one shell a pass.  (iz, iy,
        // ix): the next cells to test, the same for the whole wave, rows nearest
        // first.  Each turn drains what is queued, then tests cells until the queue
        // may be full or the pass is through.
        bool live = true;
        int rin = -1, rout = -1, iz = 0, iy = 0, ix = 0;
        int stage = 0;           // 0, 1: the nearer and farther seeds, 2: cells
        bool pass_end = true;
        for (;;) {
            drain(pass_end);
            if (SUB > 1 && pass_end && stage > 0) {
                uint64_t g[KM];
                merge_group(g);
                bound = fminf(bound, reach(g[KM - 1]));
            }
            if (pass_end) {
                if (stage == 0) {
                    queue(a2, a1);
                    queue(e1, e2);
                } else if (stage == 1) {
                    lo = a2;
                    nwin = e2 - 1 - a2;
                    const uint2 own = cells[cell0];
                    rout = __any(own.y - own.x > dense) ? 0 : 1;
                    pass_end = false;
                } else {
                    // the nearest unvisited cell on any axis: every unvisited vertex is at least `gap` steps away
                    float gap = INFINITY;
                    const float rc = (float)rout * cs;
                    if (cx - rout > 0) gap = fminf(gap, lx + rc);
                    if (cx + rout < G - 1) gap = fminf(gap, hx + rc);
                    if (cy - rout > 0) gap = fminf(gap, ly + rc);
                    if (cy + rout < G - 1) gap = fminf(gap, hy + rc);
                    if (cz - rout > 0) gap = fminf(gap, lz + rc);
                    if (cz + rout < G - 1) gap = fminf(gap, hz + rc);
                    live = live && gap < INFINITY && !(bound < gap * gap * (1.0f - 0x1p-22f));
                    if (!__any(live)) break;
                    rin = rout++;
                    pass_end = false;
                }
                ++stage;
                iz = iy = ix = 0;
            }
            while (!pass_end && !__any(nr > KnnScratch<SUB>::kRanges - 4)) {
                const int dz = zigzag(iz), dy = zigzag(iy);
                const float gz = gap1(dz, lz, hz), gzz = gz * gz;
                const bool okz = live && (uint32_t)(cz + dz) < (uint32_t)G && gzz <= bound;
                const float gy = gap1(dy, ly, hy), gyz = fmaf(gy, gy, gzz);
                const bool oky = okz && (uint32_t)(cy + dy) < (uint32_t)G && gyz <= bound;
                bool row_end = !__any(oky);
                if (!row_end) {
                    // a row through the cube already read has two parts
                    const bool holed = abs(dz) <= rin && abs(dy) <= rin;
                    const int n1 = holed ? rout - rin : 2 * rout + 1, n = holed ? 2 * n1 : n1;
                    const int row = (dz << (2 * lg)) + (dy << lg);
                    uint2 cr[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {   // up to four lookups in flight
                        const int i = ix + u, dx = i < n1 ? i - rout : rin + 1 + i - n1;
                        cr[u] = make_uint2(0u, 0u);
                        if (i < n) {
                            const float gx = gap1(dx, lx, hx);
                            if (oky && (uint32_t)(cx + dx) < (uint32_t)G && fmaf(gx, gx, gyz) <= bound)
                                cr[u] = cells[cell0 + (uint32_t)(row + dx)];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) queue(cr[u].x, cr[u].y);
                    ix += 4;
                    row_end = ix >= n;
                }
                if (row_end) {
                    ix = 0;
                    if (++iy > 2 * rout || !__any(okz)) {
                        iy = 0;
                        if (++iz > 2 * rout) pass_end = true;
                    }
                }
            }
        }
    }

    // 0, -1, 1, -2, 2, ...
    static __device__ __forceinline__ int zigzag(int i) { return (i & 1) ? -((i + 1) >> 1) : (i >> 1); }
};

// SUB: lanes a query, a power of two.
// WPE: the minimum waves per SIMD the compiler must fit the search in: 6 for
// lists of up to 16 keys (80 registers, three words spilled at 16 keys, nothing
// below; 7 and 8 spill and are 2% and 13% slower at k = 16, 5 is 4% slower);
// longer lists take no bound.
template <int KM, int WPE, int SUB>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(WPE))) void k_knn(
    int64_t N, int K, int shift, const float4* __restrict__ pts, const int32_t* __restrict__ inv,
    const uint2* __restrict__ cell_range, int32_t* __restrict__ col_sorted, int32_t* __restrict__ col_canon,
    int64_t* __restrict__ row_ptr, uint32_t* __restrict__ redo, uint32_t* __restrict__ nredo, const KeyFmt f,
    uint32_t dense) {
    __shared__ KnnScratch<SUB> scratch;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t s = (tile * kBlock + threadIdx.x) / SUB;
    if (s >= N) return;
    const int m = K - 1;
    const float4 q = pts[s];
    const uint32_t self = __float_as_uint(q.w);
    KnnSearch<KM, SUB> ks;
    ks.m = m;
    ks.sub = SUB > 1 ? (int)(threadIdx.x % SUB) : 0;
    ks.pts = pts;
    ks.cells = cell_range;
    ks.f = f;
    ks.dense = dense;
    ks.sc = &scratch;
    ks.qx = q.x;
    ks.qy = q.y;
    ks.qz = q.z;
#pragma unroll
    for (int p = 0; p < KM; ++p) ks.k[p] = p < KM - m ? 0ull : ~0ull;
    if (m > 0) ks.run((uint32_t)N, (uint32_t)s, shift);
    if (SUB > 1) {
        uint64_t g[KM];
        ks.merge_group(g);
#pragma unroll
        for (int p = 0; p < KM; ++p) ks.k[p] = g[p];
        if (ks.sub != 0) return;   // the lists are all the same: the group's first lane writes
    }
    const bool sat = m > 0 && (ks.k[KM - 1] >> f.idb) >= f.sat;   // a kept distance saturated: redo exactly
    const uint32_t slot = wave_append(nredo, sat);
    if (sat) {
        redo[slot] = (uint32_t)s;
        return;
    }
    if (col_sorted) {   // sliced-ELL layout; the padding slots of the row's last quad point at itself
        col_sorted[eidx(s, 0, K)] = (int32_t)s;
#pragma unroll
        for (int p = 0; p < KM; ++p)
            if (p >= KM - m) col_sorted[eidx(s, 1 + p - (KM - m), K)] = inv[(uint32_t)(ks.k[p] & f.idmask)];
        for (int l = K; l < ell_k4(K); ++l) col_sorted[eidx(s, l, K)] = (int32_t)s;
    }
    if (col_canon) {
        int32_t* row = col_canon + (int64_t)self * K;
        row[0] = (int32_t)self;
#pragma unroll
        for (int p = 0; p < KM; ++p)
            if (p >= KM - m) row[1 + p - (KM - m)] = (int32_t)(ks.k[p] & f.idmask);
    }
    if (row_ptr) {
        row_ptr[self] = (int64_t)self * K;
        if (s == 0) row_ptr[N] = N * (int64_t)K;
    }
}

// Exact (d2, id) search for the queries the fast path handed over.
template <int KM>
__global__ __launch_bounds__(kBlock) void k_knn_exact(int64_t N, int K, int shift, const float4* __restrict__ pts,
                                                      const int32_t* __restrict__ inv,
                                                      const uint2* __restrict__ cell_range,
                                                      int32_t* __restrict__ col_sorted,
                                                      int32_t* __restrict__ col_canon,
                                                      int64_t* __restrict__ row_ptr,
                                                      const uint32_t* __restrict__ redo,
                                                      const uint32_t* __restrict__ nredo) {
    const uint32_t n = *nredo;
    const int m = K - 1;
    for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += gridDim.x * blockDim.x) {
        const int64_t s = redo[idx];
        const float4 q = pts[s];
        uint64_t d[KM];
        uint32_t o[KM];
        list_reset<KM>(d, o, m);
        shell_search<KM>(s, shift, (int32_t)q.x, (int32_t)q.y, (int32_t)q.z, pts, cell_range, d, o);
        knn_write<KM>(s, K, m, __float_as_uint(q.w), N, inv, d, o, col_sorted, col_canon, row_ptr);
    }
}

// Every query handed to the exact search (PG_FLAG_EXACT_KNN).
__global__ __launch_bounds__(kBlock) void k_redo_all(int64_t N, uint32_t* __restrict__ redo,
                                                     uint32_t* __restrict__ nredo) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) redo[i] = (uint32_t)i;
    if (i == 0) *nredo = (uint32_t)N;
}

hipError_t launch_knn(int64_t N, int K, int shift, const float4* pts, const int32_t* inv,
                      const uint2* cell_range, int32_t* col_sorted, int32_t* col_canon,
                      int64_t* row_ptr, uint32_t* redo, uint32_t* nredo, bool exact_only, hipStream_t s) {
    if (N == 0) return hipSuccess;
    const int m = K - 1;
    const KeyFmt f = key_fmt(N);
    // up to 2^22 vertices a key holds any distance in the cube: no query is redone
    const bool redone = exact_only || f.sat <= 3ull * kQMax * kQMax;
    if (redone) {
        hipError_t e = launch_fill(nredo, sizeof(uint32_t), s);
        if (e != hipSuccess) return e;
    }
    // Cells are queued by the bound of the moment, which the seeds leave loose where a
    // cell holds many vertices: its neighbours were then read to the end although the
    // cell itself rules them out.  A pass more for it pays where the launch is bound by
    // its instructions (1M vertices of deviation 0.01: k = 2 0.73 -> 0.19 s, k = 16 0.36
    // -> 0.27 s; deviation 0.1, k = 16: 3.8 -> 3.4 ms; on a plane 1.6 -> 1.1 ms; even
    // clouds the same), not where few waves wait for their slowest (3 thousand
    // vertices of deviation 0.01, k = 18: 0.69 and 1.2 ms).
    const uint32_t dense = N * K > int64_t(1) << 19 ? 64u : ~0u;
    auto launch = [&](auto km, auto sub) {
        constexpr int KM = decltype(km)::value, SUB = decltype(sub)::value;
        constexpr int WPE = KM <= 16 && SUB == 1 ? 6 : 1;
        if (exact_only)
            hipLaunchKernelGGL(k_redo_all, dim3((unsigned)div_up(N, kBlock)), dim3(kBlock), 0, s, N, redo, nredo);
        else
            hipLaunchKernelGGL((k_knn<KM, WPE, SUB>), dim3((unsigned)div_up(N * SUB, kBlock)), dim3(kBlock), 0, s, N, K,
                               shift, pts, inv, cell_range, col_sorted, col_canon, row_ptr, redo, nredo, f, dense);
        if (redone)
            hipLaunchKernelGGL(k_knn_exact<KM>, dim3(256), dim3(kBlock), 0, s, N, K, shift, pts, inv, cell_range,
                               col_sorted, col_canon, row_ptr, (const uint32_t*)redo, (const uint32_t*)nredo);
    };
    // The fewer queries, the more lanes to each: a small launch lasts as long as its
    // slowest wave, a large one as long as its instructions, of which groups take
    // more.  Lists with the grid build, 1 / 2 / 4 / 8 lanes a query:
    //   N = 3 thousand, k = 16    0.229  0.145  0.098  0.073 ms   (N K = 2^15.6)
    //       10 thousand, 8        0.155  0.104  0.094  0.093      (2^16.3)
    //       29 thousand, 16       0.146  0.113  0.106  0.127      (2^18.8)
    //       60 thousand, 16       0.243  0.224  0.252  0.283      (2^19.9)
    //       120 thousand, 16      0.273  0.247  0.310  0.370      (2^20.9)
    //       240 thousand, 16      0.514  0.503  0.633  0.749      (2^21.9)
    //       480 thousand, 8       0.438  0.457  0.538  0.741      (2^21.9)
    // Lists longer than 16 keys stay with one lane: merging needs two in registers.
    auto go = [&](auto km) {
        constexpr int KM = decltype(km)::value;
        const int64_t work = N * K;
        if constexpr (KM <= 16) {
            if (work <= int64_t(1) << 16) return launch(km, std::integral_constant<int, 8>{});
            if (work <= int64_t(1) << 19) return launch(km, std::integral_constant<int, 4>{});
            if (work <= int64_t(1) << 21) return launch(km, std::integral_constant<int, 2>{});
        }
        return launch(km, std::integral_constant<int, 1>{});
    };
    // k = 8..17 get a list of exactly K-1 keys: a sentinel slot costs its
    // compare and selects in every insertion
    switch (m) {
        case 7: go(std::integral_constant<int, 7>{}); break;
        case 8: go(std::integral_constant<int, 8>{}); break;
        case 9: go(std::integral_constant<int, 9>{}); break;
        case 10: go(std::integral_constant<int, 10>{}); break;
        case 11: go(std::integral_constant<int, 11>{}); break;
        case 12: go(std::integral_constant<int, 12>{}); break;
        case 13: go(std::integral_constant<int, 13>{}); break;
        case 14: go(std::integral_constant<int, 14>{}); break;
        case 15: go(std::integral_constant<int, 15>{}); break;
        case 16: go(std::integral_constant<int, 16>{}); break;
        default:
            if (m < 7) go(std::integral_constant<int, 8>{});
            else if (m <= 32) go(std::integral_constant<int, 32>{});
            else go(std::integral_constant<int, 64>{});
    }
    return hipGetLastError();
}

}  // namespace pg
