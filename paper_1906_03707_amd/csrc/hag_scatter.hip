// Transposed pass of max without device-wide atomics: gradients are sorted into blocks of winners, and every block is added up in LDS.
#include "hag_device_common.hpp"

namespace hag {

// gx[argmax[v, f], f] += gy[v, f].  An atomic add in memory is one request of 64 bytes at the memory side whoever issues it, about 17 of them per ns here:
// 16.8 M elements (131072 nodes, d = 128) took 990 us for 0.2 GB of inputs and results.  Three launches instead:
//   max_bin_kernel: a workgroup takes 512 rows of up to 32 columns (128 contiguous bytes a row), sorts its elements by the block of 512 nodes their winner is
//     in (rank by LDS atomics on a histogram, a scan, a pass through LDS) and writes them as runs, one per block: 4 bytes of value and 2 of place in the block,
//     in a segment of its own, with the beginnings of the runs beside it.  No counting pass, no global counters.
//   max_split_kernel: how many elements a block has.  One with more than kFoldElems is cut by tiles into parts for several workgroups (a hub may be the
//     winner of a third of all rows), whose sums meet in rows of gx that are cleared here.
//   max_fold_kernel: a workgroup takes a block of 512 nodes and the same columns, walks that block's run of every segment, adds into 64 KB of LDS and writes
//     its rows of gx whole (so nothing else is cleared beforehand).  Runs average 16384 / blocks elements: 64 at 131072 nodes; a wavefront asks for four at
//     once, and several wavefronts share a long one.
// 131072 nodes, d = 128, winners anywhere: 809 us with atomics, 163 in blocks (int32 634 and 114: LDS adds 32-bit integers faster than floats); winners of a
//     graph with communities 990 and 165; one node winning everything 3160 and 313; 232965 nodes, d = 16: 185 and 60.
// From 2^20 elements: 16384 x 64 55 us with atomics and 46 in blocks, 65536 x 16 55 and 34, but 8192 x 64 30 and 43, 16384 x 36 33 and 34 (three launches, and few
//     workgroups).  Up to 2^21 nodes: the histogram is 16 KB of LDS then (2000000 x 64: 6517 and 2518 us).
// Few columns of many nodes stay with the atomics: a block's workgroup looks up its run in the table of every tile (tiles x blocks entries), and the runs of 512 rows hold an element or
//     two.  us, atomics / blocks, winners anywhere: 4 columns of 262145 nodes 56 / 49, 524288 106 / 99, 700000 140 / 158, 1000003 198 / 243, 2000000 391 / 651; 8 of 1000003 390 / 281,
//     1500000 582 / 513, 2000000 774 / 796; 12 of 2000000 1157 / 897.  Atomics of integers are a fifth faster: 4 of 262145 44 / 49, 1000003 155 / 239; 8 of 1000003 307 / 281, 1500000 456 / 508,
//     2000000 606 / 791; 12 of 1500000 681 / 566.  blocks_us below is those with the table's lookups at 50 ps each.
// 32 columns: wider tiles would make the blocks of a 64 KB accumulator shorter and the runs with them; narrower ones read less than a cache line.
// Every element is added once; the order inside a run and between runs is not fixed, as it was not with the atomics.
constexpr int kBinRows = 512, kBinNodes = 512, kBinCols = 32, kBinThreads = 1024, kBinElems = kBinRows * kBinCols, kBinQuads = kBinElems / 4 / kBinThreads;

constexpr uint32_t kFoldElems = 1 << 16;   // elements per workgroup of the fold (four times what a block has on average at 131072 nodes)
constexpr int kFoldExtra = 1024;           // workgroups for further parts; a part holds more elements where these would not do

struct BinShape { int64_t tiles, blocks, chunks, cols, pitch; };   // cols: columns of a chunk (a multiple of 4); pitch: entries of a segment's table of run beginnings
static BinShape bin_shape(int64_t n, int64_t d) {
    BinShape b;
    b.tiles = (n + kBinRows - 1) / kBinRows;
    b.blocks = (n + kBinNodes - 1) / kBinNodes;
    b.chunks = (d + kBinCols - 1) / kBinCols;
    b.cols = (d / 4 + b.chunks - 1) / b.chunks * 4;
    b.pitch = (b.blocks + 2) & ~(int64_t)1;
    return b;
}

static size_t align_256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t max_scatter_bytes(int64_t n, int64_t d, hag_dtype_t dt) {
    if (n <= 0 || n > kBinMaxNodes || n * d < kBinMinElements) return 0;
    const BinShape b = bin_shape(n, d);
    const double elements = (double)n * (double)d, blocks_us = 33. + 50e-6 * (double)b.tiles * (double)b.blocks * (double)b.chunks + 8e-6 * elements;
    if (blocks_us > 5. + (dt == HAG_F32 ? 48e-6 : 38e-6) * elements) return 0;
    const size_t segments = (size_t)(b.tiles * b.chunks), elems = segments * (size_t)(kBinRows * b.cols);
    return align_256(elems * 4) + align_256(elems * 2) + align_256(segments * (size_t)b.pitch * 2) + align_256((size_t)(b.blocks * b.chunks) * 4) +
           align_256((kFoldExtra * 2 + 2) * 4);
}

template <typename T>
__global__ __launch_bounds__(kBinThreads) void max_bin_kernel(const T *__restrict__ gy, const int32_t *__restrict__ argmax, int32_t n, int32_t d, int32_t cols,
                                                              int32_t blocks, int32_t pitch, T *__restrict__ vals, uint16_t *__restrict__ keys,
                                                              uint16_t *__restrict__ begins, uint32_t *__restrict__ extra) {
    using V = typename V4<T>::type;
    __shared__ __align__(16) T sval[kBinElems];
    __shared__ __align__(16) uint16_t skey[kBinElems];
    __shared__ uint32_t hist[kBinMaxNodes / kBinNodes + 4];   // counts, then beginnings
    __shared__ uint32_t wave_sum[kBinThreads / kWave + 1];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int quads = cols / 4, col0 = blockIdx.y * cols;
    const int64_t row0 = (int64_t)blockIdx.x * kBinRows;
    const int rows = (int)min((int64_t)kBinRows, (int64_t)n - row0), mine = min(quads, (d - col0) / 4);
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *extra = 0;   // (counted up by the next launch)
    for (int b = tid; b < blocks; b += kBinThreads) hist[b] = 0;
    __syncthreads();
    int4 who[kBinQuads];
    V val[kBinQuads];
    uint32_t rank[kBinQuads][4];
#pragma unroll
    for (int k = 0; k < kBinQuads; ++k) {
        const int i = tid + k * kBinThreads, r = i / quads, q = i % quads;
        who[k] = make_int4(-1, -1, -1, -1);
        val[k] = V{};
        if (r < rows && q < mine) {
            const size_t at = (size_t)(row0 + r) * d + col0 + 4 * q;
            who[k] = ld4(argmax + at);
            val[k] = ld4(gy + at);
        }
    }
#pragma unroll
    for (int k = 0; k < kBinQuads; ++k) {
        int *w = reinterpret_cast<int *>(&who[k]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            rank[k][e] = 0;
            if ((uint32_t)w[e] < (uint32_t)n) rank[k][e] = atomicAdd(&hist[w[e] / kBinNodes], 1u);
        }
    }
    __syncthreads();
    {
        // exclusive scan of the counts, in place: every thread takes `per` neighbouring blocks
        const int per = (blocks + kBinThreads - 1) / kBinThreads;
        uint32_t sum = 0;
        for (int j = 0; j < per; ++j)
            if (tid * per + j < blocks) sum += hist[tid * per + j];
        uint32_t upto = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t v = __shfl_up(upto, off);
            if (lane >= off) upto += v;
        }
        if (lane == kWave - 1) wave_sum[wave] = upto;
        __syncthreads();
        uint32_t at = upto - sum;
        for (int w = 0; w < wave; ++w) at += wave_sum[w];
        for (int j = 0; j < per; ++j)
            if (tid * per + j < blocks) { const uint32_t c = hist[tid * per + j]; hist[tid * per + j] = at; at += c; }
        if (tid == kBinThreads - 1) hist[blocks] = at;     // (this thread's prefix ends at the total, whatever blocks it had)
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kBinQuads; ++k) {
        const int *w = reinterpret_cast<const int *>(&who[k]);
        const T *v = reinterpret_cast<const T *>(&val[k]);
        const int q = (tid + k * kBinThreads) % quads;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if ((uint32_t)w[e] < (uint32_t)n) {
                const uint32_t at = hist[w[e] / kBinNodes] + rank[k][e];
                sval[at] = v[e];
                skey[at] = (uint16_t)((w[e] % kBinNodes) * kBinCols + 4 * q + e);
            }
    }
    __syncthreads();
    const int64_t segment = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int total = (int)hist[blocks];
    T *out_v = vals + (size_t)segment * kBinRows * cols;
    uint16_t *out_k = keys + (size_t)segment * kBinRows * cols;
    // (the last vector may hold elements beyond the total: the segment has room for them and nobody reads them)
    for (int i = tid * 4; i < total; i += kBinThreads * 4) st4(out_v + i, ld4(sval + i));
    for (int i = tid * 8; i < total; i += kBinThreads * 8) *reinterpret_cast<int4 *>(out_k + i) = *reinterpret_cast<const int4 *>(skey + i);
    uint16_t *out_b = begins + (size_t)segment * pitch;
    for (int b = tid; b <= blocks; b += kBinThreads) out_b[b] = (uint16_t)hist[b];
}

__device__ __forceinline__ void lds_accumulate(float *p, float v) { __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void lds_accumulate(int32_t *p, int32_t v) {   // wraps modulo 2^32
    __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(p), (uint32_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// the number of parts a block's elements are added up in: part p takes the tiles [tiles * p / parts, tiles * (p + 1) / parts)
__device__ __forceinline__ int fold_parts(uint32_t total, uint32_t per_part, int tiles) {
    return (int)min(max(total / per_part, 1u), (uint32_t)tiles);
}

// totals[chunk][block], and for every part beyond a block's first an entry {chunk * blocks + block, part}.  64 blocks per workgroup, its wavefronts share the tiles.
template <typename T>
__global__ __launch_bounds__(kBinThreads) void max_split_kernel(const uint16_t *__restrict__ begins, int32_t n, int32_t d, int32_t cols, int32_t tiles, int32_t blocks,
                                                                int32_t pitch, uint32_t per_part, uint32_t *__restrict__ totals, uint32_t *__restrict__ extra,
                                                                T *__restrict__ gx) {
    using V = typename V4<T>::type;
    __shared__ uint32_t sums[kBinThreads / kWave][kWave];
    __shared__ int parts_of[kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, block = blockIdx.x * kWave + lane;
    uint32_t sum = 0;
    if (block < blocks) {
        constexpr int kAsk = 8, kStep = kBinThreads / kWave;
        for (int tile = wave; tile < tiles; tile += kAsk * kStep) {
            uint32_t from[kAsk], to[kAsk];
#pragma unroll
            for (int k = 0; k < kAsk; ++k) {
                const uint16_t *b = begins + ((size_t)blockIdx.y * tiles + min(tile + k * kStep, tiles - 1)) * pitch + block;
                from[k] = b[0];
                to[k] = b[1];
            }
#pragma unroll
            for (int k = 0; k < kAsk; ++k) sum += tile + k * kStep < tiles ? to[k] - from[k] : 0;
        }
    }
    sums[wave][lane] = sum;
    __syncthreads();
    if (wave == 0) {
        for (int w = 1; w < kBinThreads / kWave; ++w) sum += sums[w][lane];
        const int parts = block < blocks ? fold_parts(sum, per_part, tiles) : 1;
        parts_of[lane] = parts;
        if (block < blocks) totals[(size_t)blockIdx.y * blocks + block] = sum;
        if (parts > 1) {
            // (per_part is such that the further parts of all blocks together are no more than kFoldExtra)
            const uint32_t at = atomicAdd(extra, (uint32_t)(parts - 1));
            for (int p = 1; p < parts && at + p - 1 < (uint32_t)kFoldExtra; ++p) {
                extra[2 + 2 * (at + p - 1)] = (uint32_t)(blockIdx.y * blocks + block);
                extra[3 + 2 * (at + p - 1)] = (uint32_t)p;
            }
        }
    }
    __syncthreads();
    const int quads = cols / 4, col0 = blockIdx.y * cols, mine = min(quads, (d - col0) / 4);
    for (int k = 0; k < kWave; ++k) {
        if (parts_of[k] <= 1) continue;
        const int64_t u0 = (int64_t)(blockIdx.x * kWave + k) * kBinNodes;
        for (int i = threadIdx.x; i < kBinNodes * quads; i += kBinThreads)
            if (u0 + i / quads < n && i % quads < mine) st4(gx + (size_t)(u0 + i / quads) * d + col0 + 4 * (i % quads), V{});
    }
}

__device__ __forceinline__ void device_accumulate(float *p, float v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void device_accumulate(int32_t *p, int32_t v) { atomicAdd(p, v); }

// Workgroups [0, blocks * chunks): the first part of a block; the others: the entries of max_split_kernel.
template <typename T>
__global__ __launch_bounds__(kBinThreads) void max_fold_kernel(const T *__restrict__ vals, const uint16_t *__restrict__ keys, const uint16_t *__restrict__ begins,
                                                               const uint32_t *__restrict__ totals, const uint32_t *__restrict__ extra, int32_t n, int32_t d,
                                                               int32_t cols, int32_t tiles, int32_t blocks, int32_t chunks, int32_t pitch, uint32_t per_part,
                                                               T *__restrict__ gx) {
    using V = typename V4<T>::type;
    __shared__ __align__(16) T acc[kBinNodes * kBinCols];
    constexpr int kWaves = kBinThreads / kWave, kAsk = 4;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    int which = blockIdx.x, part = 0;
    if (which >= blocks * chunks) {
        const uint32_t e = which - blocks * chunks;
        if (e >= *extra) return;
        which = (int)extra[2 + 2 * e];
        part = (int)extra[3 + 2 * e];
    }
    const int chunk = which / blocks, block = which % blocks;
    const uint32_t total = totals[which];
    const int parts = fold_parts(total, per_part, tiles), tile0 = (int)((int64_t)tiles * part / parts), tile1 = (int)((int64_t)tiles * (part + 1) / parts);
    // wavefronts that share a run: as many as it has pieces of 64, and so that none is left without a tile
    int share = 1;
    while (share < kWaves && (total / tiles > (uint32_t)(kWave * share) || (tile1 - tile0) * share < kWaves)) share *= 2;
    const int sub = wave % share, step = kWaves / share;
    for (int i = tid * 4; i < kBinNodes * kBinCols; i += kBinThreads * 4) st4(acc + i, V{});
    __syncthreads();
    const size_t first_segment = (size_t)chunk * tiles, per_segment = (size_t)kBinRows * cols;
    for (int base = tile0 + wave / share; base < tile1; base += step * kWave) {
        const int tile = base + step * lane;               // this lane knows the run of that tile
        int lo = 0, hi = 0;
        if (tile < tile1) {
            const uint16_t *b = begins + (first_segment + tile) * pitch + block;
            lo = b[0]; hi = b[1];
        }
        const int known = min(kWave, (tile1 - base + step - 1) / step);
        for (int i = 0; i < known; i += kAsk) {
            int from[kAsk], to[kAsk];
            T v[kAsk];
            uint32_t key[kAsk];
#pragma unroll
            for (int k = 0; k < kAsk; ++k) {
                const int j = min(i + k, kWave - 1);
                from[k] = __builtin_amdgcn_readlane(lo, j) + sub * kWave;
                to[k] = i + k < known ? __builtin_amdgcn_readlane(hi, j) : 0;
                const size_t at = (first_segment + base + step * (i + k)) * per_segment + from[k] + lane;
                if (from[k] + lane < to[k]) { v[k] = vals[at]; key[k] = keys[at]; }
            }
#pragma unroll
            for (int k = 0; k < kAsk; ++k)
                if (from[k] + lane < to[k]) lds_accumulate(&acc[key[k]], v[k]);
#pragma unroll
            for (int k = 0; k < kAsk; ++k)
                for (int e = from[k] + share * kWave + lane; e < to[k]; e += share * kWave) {
                    const size_t at = (first_segment + base + step * (i + k)) * per_segment + e;
                    lds_accumulate(&acc[keys[at]], vals[at]);
                }
        }
    }
    __syncthreads();
    const int quads = cols / 4, col0 = chunk * cols, mine = min(quads, (d - col0) / 4);
    const int64_t u0 = (int64_t)block * kBinNodes;
    if (parts > 1) {
        for (int i = tid; i < kBinNodes * kBinCols; i += kBinThreads) {
            const int r = i / kBinCols, c = i % kBinCols;
            const T v = acc[i];
            if (u0 + r < n && c < 4 * mine && v != T(0)) device_accumulate(gx + (size_t)(u0 + r) * d + col0 + c, v);
        }
        return;
    }
    for (int i = tid; i < kBinNodes * quads; i += kBinThreads) {
        const int r = i / quads, q = i % quads;
        if (u0 + r < n && q < mine) st4(gx + (size_t)(u0 + r) * d + col0 + 4 * q, ld4(acc + r * kBinCols + 4 * q));
    }
}

template <typename T>
int launch_max_scatter(int64_t n, int64_t d, const T *gy, const int32_t *argmax, T *gx, void *ws, hipStream_t s) {
    const BinShape b = bin_shape(n, d);
    const size_t segments = (size_t)(b.tiles * b.chunks), elems = segments * (size_t)(kBinRows * b.cols);
    T *vals = (T *)ws;
    uint16_t *keys = (uint16_t *)((char *)ws + align_256(elems * 4)), *begins = (uint16_t *)((char *)keys + align_256(elems * 2));
    uint32_t *totals = (uint32_t *)((char *)begins + align_256(segments * (size_t)b.pitch * 2));
    uint32_t *extra = (uint32_t *)((char *)totals + align_256((size_t)(b.blocks * b.chunks) * 4));
    const uint32_t per_part = std::max<uint32_t>(kFoldElems, (uint32_t)((uint64_t)(n * d) / kFoldExtra + 1));
    const uint64_t main_groups = (uint64_t)(b.blocks * b.chunks);
    if (main_groups + kFoldExtra > 0x7fffffffULL) { set_error("launch too large"); return HAG_EINVAL; }
    hipLaunchKernelGGL((max_bin_kernel<T>), dim3((unsigned)b.tiles, (unsigned)b.chunks), dim3(kBinThreads), 0, s, gy, argmax, (int32_t)n, (int32_t)d,
                       (int32_t)b.cols, (int32_t)b.blocks, (int32_t)b.pitch, vals, keys, begins, extra);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL((max_split_kernel<T>), dim3((unsigned)((b.blocks + kWave - 1) / kWave), (unsigned)b.chunks), dim3(kBinThreads), 0, s, begins, (int32_t)n,
                       (int32_t)d, (int32_t)b.cols, (int32_t)b.tiles, (int32_t)b.blocks, (int32_t)b.pitch, per_part, totals, extra, gx);
    HIP_TRY(hipGetLastError());
    const uint64_t more = std::min<uint64_t>(kFoldExtra, (uint64_t)(n * d) / per_part);
    hipLaunchKernelGGL((max_fold_kernel<T>), dim3((unsigned)(main_groups + more)), dim3(kBinThreads), 0, s, vals, keys, begins, totals, extra, (int32_t)n,
                       (int32_t)d, (int32_t)b.cols, (int32_t)b.tiles, (int32_t)b.blocks, (int32_t)b.chunks, (int32_t)b.pitch, per_part, gx);
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}
template int launch_max_scatter<float>(int64_t, int64_t, const float *, const int32_t *, float *, void *, hipStream_t);
template int launch_max_scatter<int32_t>(int64_t, int64_t, const int32_t *, const int32_t *, int32_t *, void *, hipStream_t);

}  // namespace hag
