// Batches of small graphs as small dense products, f32 features.
#include "hag_device_common.hpp"

namespace hag {

typedef __bf16 dense_b8_t __attribute__((ext_vector_type(8)));
typedef float dense_f4_t __attribute__((ext_vector_type(4)));
typedef unsigned int dense_u4_t __attribute__((ext_vector_type(4)));

// y = A x for one component, A its adjacency matrix as bits (what a HAG aggregates for a node is exactly the node's neighbour set,
// so the bits serve the HAG and the plain graph alike).  The product runs on the matrix cores: an fp32 feature is cut
// into three bf16 pieces of eight significant bits each, which add up to it exactly, and a bit becomes the bf16 number 2 or 0, so every
// product is exact and the sums are rounded where an fp32 sum is; the factor 2 (one bit to move instead of seven to
// set) comes off at the end.
//
// One wavefront per (component, 16 * VEC feature columns, up to MT * 16 output rows), no LDS, no barrier.  v_mfma_f32_16x16x32_bf16 takes its
// second operand as 8 consecutive k (nodes) of one column per lane; column c of the product t of VEC is feature VEC * c + t, so that a lane loads
// VEC consecutive floats and 16 lanes a contiguous row, and the results of a lane are VEC consecutive floats of the output row.  VEC is 4, or 2 and
// 1 for matrices of up to 32 and 16 columns, which would leave most lanes without a column (d = 4, density 0.1: 56 us with VEC 4, lists 41 us).
// Graphs up to kDenseMaxNodes nodes: the matrix and vector instructions of a wavefront (about 0.1 nv^2 + 10 nv cycles of a compute unit
// per 64 columns) stay below the time its rows take from and to HBM (about 60 nv), whatever the number of edges; lists of ids cost about two
// cycles per edge and column block, plus a barrier per stage.  Measured, 5000 graphs of 74 nodes, d = 64, forward and transposed pass
// together: 75 us repeated alone, 89 us on new features (4.3 TB/s of features in and results out, a copy runs at 5.2) at any density; lists repeated alone 160 us
// at density 0.9 and about what the products take at 0.05.  Few, large and sparse graphs are better served by the lists: 100 of 250 nodes, mean degree 5: 35 against 22 us
// (which form runs is decided in hag_cost.cpp).
//
// A feature is multiplied by 2^48 first, which takes even the last bit of a subnormal into the range of bf16 and is exact.  Features that the pieces
// cannot hold then (infinities, NaN, |x| above 2^70) would also reach rows they are no neighbour of (0 * inf); a wavefront that has loaded one redoes
// its rows by adding the neighbours one by one.
constexpr float kDenseScale = 0x1p48f;
__device__ __forceinline__ void dense_split2(float a, float b, uint32_t &p0, uint32_t &p1, uint32_t &p2) {
    // cut, not rounded: no piece can overflow, and the three still hold all 24 bits
    uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    p0 = __builtin_amdgcn_perm(ub, ua, 0x07060302);
    a -= __uint_as_float(ua & 0xffff0000u); b -= __uint_as_float(ub & 0xffff0000u);
    ua = __float_as_uint(a); ub = __float_as_uint(b);
    p1 = __builtin_amdgcn_perm(ub, ua, 0x07060302);
    a -= __uint_as_float(ua & 0xffff0000u); b -= __uint_as_float(ub & 0xffff0000u);
    p2 = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302);
}

template <int VEC> struct DenseVec;
template <> struct DenseVec<1> { typedef float type; };
template <> struct DenseVec<2> { typedef float2 type; };
template <> struct DenseVec<4> { typedef float4 type; };

template <int VEC, int ROLE>
__global__ __launch_bounds__(kBlock, 2) void dense_kernel(DenseArgs A) {
    constexpr int MT = kDenseTiles;
    const int lane = threadIdx.x & (kWave - 1), n = lane & 15, q4 = lane >> 4;
    const int64_t task = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const int per = A.m_chunks * A.f_chunks;
    if (task >= (int64_t)A.count * per) return;
    const int c = (int)(task / per), rest = (int)(task % per), mc = rest / A.f_chunks, fc = rest % A.f_chunks;
    const int4 meta = *reinterpret_cast<const int4 *>(A.meta + 4 * (size_t)c);   // first node, nodes, first word of the bits, -
    const int v0 = meta.x, nv = meta.y;
    const uint32_t *bits = A.bits + (uint32_t)meta.z;
    const int tiles = (nv + 15) / 16, kw = (nv + 31) / 32;
    const int t0 = tiles * mc / A.m_chunks, nt = tiles * (mc + 1) / A.m_chunks - t0;   // at most MT
    if (nt <= 0) return;
    const int f = fc * 16 * VEC + VEC * n;
    const bool col_ok = f < A.d;
    const float *in = A.in + (size_t)v0 * A.d + (col_ok ? f : 0);
    dense_f4_t acc[MT][VEC];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[m][t] = dense_f4_t{0.f, 0.f, 0.f, 0.f};
    uint32_t largest = 0;                                  // of the scaled magnitudes
    typedef typename DenseVec<VEC>::type vec_t;
    union Vec { vec_t v; float e[VEC]; };
    auto load = [&](int k) { Vec u; u.v = *reinterpret_cast<const vec_t *>(in + (size_t)k * A.d); return u; };
    Vec x[8];
    uint32_t word[MT];
    auto request = [&](int s) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = 32 * s + 8 * q4 + i;
#pragma unroll
            for (int t = 0; t < VEC; ++t) x[i].e[t] = 0.f;
            if (k < nv && col_ok) x[i] = load(k);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int row = (t0 + m) * 16 + n;
            word[m] = m < nt && row < nv ? bits[row * kw + s] : 0;
        }
    };
    request(0);
    for (int s = 0; s < kw; ++s) {
        Vec v[8];
        dense_u4_t a[MT];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = x[i];
        if (A.scale_in) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = 32 * s + 8 * q4 + i;
                const float scale = A.scale_in[v0 + (k < nv ? k : 0)];
#pragma unroll
                for (int t = 0; t < VEC; ++t) v[i].e[t] *= scale;
            }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const uint32_t b = (word[m] >> (8 * q4)) & 0xffu, e = b | (b << 15);   // bit 2 i below bit 2 i + 1 of the next half word
#pragma unroll
            for (int i = 0; i < 4; ++i) a[m][i] = (e << (14 - 2 * i)) & 0x40004000u;
        }
        if (s + 1 < kw) request(s + 1);
#pragma unroll
        for (int t = 0; t < VEC; ++t) {
            dense_u4_t p[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float lo = kDenseScale * v[2 * i].e[t], hi = kDenseScale * v[2 * i + 1].e[t];
                const uint32_t ul = __float_as_uint(lo) & 0x7fffffffu, uh = __float_as_uint(hi) & 0x7fffffffu;
                largest = max(largest, max(ul, uh));
                uint32_t p0, p1, p2;
                dense_split2(lo, hi, p0, p1, p2);
                p[0][i] = p0; p[1][i] = p1; p[2][i] = p2;
            }
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if (m >= nt) continue;
                const dense_b8_t w = __builtin_bit_cast(dense_b8_t, a[m]);
#pragma unroll
                for (int k = 2; k >= 0; --k)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, __builtin_bit_cast(dense_b8_t, p[k]), acc[m][t], 0, 0, 0);
            }
        }
    }
    const bool plain = __any(largest > 0x7a800000u);       // 2^118: 256 twice as large stay finite
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if (m >= nt) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = (t0 + m) * 16 + 4 * q4 + r;
            if (row >= nv || !col_ok) continue;
            Vec y;
#pragma unroll
            for (int t = 0; t < VEC; ++t) y.e[t] = 0.5f / kDenseScale * acc[m][t][r];
            if (plain) {
#pragma unroll
                for (int t = 0; t < VEC; ++t) y.e[t] = 0.f;
                for (int k = 0; k < nv; ++k) {
                    if (!((bits[row * kw + k / 32] >> (k & 31)) & 1)) continue;
                    const Vec u = load(k);
                    const float scale = A.scale_in ? A.scale_in[v0 + k] : 1.f;
#pragma unroll
                    for (int t = 0; t < VEC; ++t) y.e[t] += u.e[t] * scale;
                }
            }
            if (A.add_self) {
                const Vec own = load(row);
                const float scale = A.scale_in ? A.scale_in[v0 + row] : 1.f;
#pragma unroll
                for (int t = 0; t < VEC; ++t) y.e[t] += own.e[t] * scale;
            }
            if (A.scale_out) {
                const float scale = A.scale_out[v0 + row];
#pragma unroll
                for (int t = 0; t < VEC; ++t) y.e[t] *= scale;
            }
            *reinterpret_cast<vec_t *>(A.out + (size_t)(v0 + row) * A.d + f) = y.v;
        }
    }
}

template <int VEC>
static int launch_dense_vec(DenseArgs a, int role, hipStream_t s) {
    a.f_chunks = (a.d + 16 * VEC - 1) / (16 * VEC);
    const int64_t tasks = (int64_t)a.count * a.m_chunks * a.f_chunks, blocks = (tasks + kBlock / kWave - 1) / (kBlock / kWave);
    if (blocks <= 0) return HAG_OK;
    if (blocks > 0x7fffffffLL) { set_error("launch too large"); return HAG_EINVAL; }
    const dim3 grid((unsigned)blocks), block(kBlock);
    switch (role) {
        case 0: hipLaunchKernelGGL((dense_kernel<VEC, 0>), grid, block, 0, s, a); break;
        case 1: hipLaunchKernelGGL((dense_kernel<VEC, 1>), grid, block, 0, s, a); break;
        case 2: hipLaunchKernelGGL((dense_kernel<VEC, 2>), grid, block, 0, s, a); break;
        default: hipLaunchKernelGGL((dense_kernel<VEC, 3>), grid, block, 0, s, a); break;
    }
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

int launch_dense(DenseArgs a, int role, int max_nodes, hipStream_t s) {
    a.m_chunks = dense_row_chunks(max_nodes);
    switch (dense_vec(a.d)) {
        case 1: return launch_dense_vec<1>(a, role, s);
        case 2: return launch_dense_vec<2>(a, role, s);
        default: return launch_dense_vec<4>(a, role, s);
    }
}

// The tiles of a list set: 128 rows of the output against the sources that at least five of them name, the same products as above with a gathered operand.  A list entry costs a
// gather one row read, mostly out of L2; here a source's row is read once per tile, whatever the number of rows that name it.  Graphs with communities have half of
// their entries in such (tile, source) pairs, twelve to a pair on average.  What bounds it are the instructions: vector instructions issue 69 % of the time and the matrix cores are busy
// 34 % of it, one after the other (131072 nodes, d = 128: 0.8 GB of L2 requests, 0.28 GB of fills and 0.13 GB of writes in 162 us).  A pair costs about as much as three or four list
// entries, and pairs of three (212 us for 64 k steps instead of 121 for 33 k) gain nothing over the lists.  Whole forward sums, lists / tiles and rest, us: 131072 nodes, 26 M edges, d = 64 331 / 305, 128 634 / 569, 512 2696 / 2245; 65536 nodes, 8.4 M edges, d = 256 409 / 373,
// 512 826 / 746, but 64 119 / 146, 16 58 / 78 (where the line lies: tiles_us in hag_cost.cpp).
// A wavefront takes a unit, at most 24 steps of 32 sources of a tile, and 16 * VEC columns; tiles of more steps are added up by the fold, like cut rows.  Shorter units cost more partial
// rows than they gain, longer ones leave the smaller graphs waiting for the last of them (steps 16 / 24 / 32: 131072 nodes, d = 128, 595 / 569 / 560 us; 65536 nodes, d = 256, 388 / 373 / 383).
// The matrix cores cut what they add to the size of the largest operand, always in one direction: sums carried along in the accumulator were too small by 6e-9 to 1e-8 on average, with an error
// against 64 bits of 5.7e-8 on features of one sign, where the same sum as a plain gather had 5.2e-8 one after the other and has 4.2e-8 (131072 nodes, d = 128).  Every step therefore begins at
// zero, the largest pieces (exact unless their sizes differ by more than 2^11 or so) apart from the others (whose cut bits are 2^-8 of theirs), and joins the running sum in rounded additions:
// 4.8e-8 (normal features 1.17e-7 -> 9.4e-8, a gather 9.4e-8) with no bias left, for 4 % of the pass, which units of 24 steps in place of 16 give back.  One chain from zero for all three pieces took
// half of that, but left normal features with a bias of 3e-8.
// Four wavefronts sharing a tile's steps through LDS took 261 us where this takes 212: most tiles are a few steps long.
template <int VEC>
__global__ __launch_bounds__(kBlock, 2) void tile_kernel(TileArgs A) {
    constexpr int MT = kTileRows / 16;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), n = lane & 15, q4 = lane >> 4;
    const int xcd = blockIdx.x % kPartitions, at = blockIdx.x / kPartitions * (kBlock / kWave) + wave, fc = at % A.f_chunks;
    const int which = A.range[xcd] + at / A.f_chunks;
    if (which >= A.range[xcd + 1]) return;
    const Tiles::Unit unit = A.units[which];
    const int s0 = unit.first, s1 = unit.last;
    const int f = fc * 16 * VEC + VEC * n;
    const bool col_ok = f < A.d;
    const int from = col_ok ? f : 0;
    dense_f4_t acc[MT][VEC];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[m][t] = dense_f4_t{0.f, 0.f, 0.f, 0.f};
    uint32_t largest = 0;                                  // of the scaled magnitudes
    typedef typename DenseVec<VEC>::type vec_t;
    union Vec { vec_t v; float e[VEC]; };
    auto load = [&](int id) { Vec u; u.v = *reinterpret_cast<const vec_t *>(A.in + ((size_t)id * A.d + from)); return u; };
    int ids = 0;                                           // lane l: source l % 32 of the step after next
    Vec x[8];
    uint2 bits = make_uint2(0, 0);                         // of the next step: byte m, bit i: source 8 * (l / 16) + i for row 16 m + l % 16
    auto request_bits = [&](int s) { bits = *reinterpret_cast<const uint2 *>(A.bits + ((size_t)s * kTileRows + 2 * lane)); };
    auto request_ids = [&](int s) { ids = A.ids[(size_t)s * kTileStep + (lane & 31)]; };
    auto request_rows = [&](int i0, int i1) {
#pragma unroll
        for (int i = i0; i < i1; ++i) x[i] = load(__shfl(ids, 8 * q4 + i));
    };
    if (s0 < s1) {
        request_ids(s0);
        request_bits(s0);
        request_rows(0, 8);
        request_ids(min(s0 + 1, s1 - 1));
    }
    for (int s = s0; s < s1; ++s) {
        dense_u4_t p[VEC][3];
#pragma unroll
        for (int t = 0; t < VEC; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float lo = kDenseScale * x[2 * i].e[t], hi = kDenseScale * x[2 * i + 1].e[t];
                const uint32_t ul = __float_as_uint(lo) & 0x7fffffffu, uh = __float_as_uint(hi) & 0x7fffffffu;
                largest = max(largest, max(ul, uh));
                uint32_t p0, p1, p2;
                dense_split2(lo, hi, p0, p1, p2);
                p[t][0][i] = p0; p[t][1][i] = p1; p[t][2][i] = p2;
            }
        const uint2 now = bits;
        if (s + 1 < s1) {
            request_bits(s + 1);
            request_rows(0, 8);
            request_ids(min(s + 2, s1 - 1));
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if (VEC == 4) __builtin_amdgcn_sched_barrier(0);   // (one row tile at a time: registers are short)
            const uint32_t b = ((m < 4 ? now.x : now.y) >> (8 * (m % 4))) & 0xffu, e = b | (b << 15);   // bit 2 i below bit 2 i + 1 of the next half word
            dense_u4_t a;
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = (e << (14 - 2 * i)) & 0x40004000u;
            // a step's sums begin at zero, of the largest pieces and of the others, and join the running sum in rounded additions
#pragma unroll
            for (int t0 = 0; t0 < VEC; t0 += 2) {
                constexpr int TN = VEC < 2 ? VEC : 2;
                dense_f4_t sum[TN][2];
#pragma unroll
                for (int k = 2; k >= 0; --k)
#pragma unroll
                    for (int t = 0; t < TN; ++t)
                        sum[t][k == 0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dense_b8_t, a), __builtin_bit_cast(dense_b8_t, p[t0 + t][k]),
                                                                                 k == 1 ? sum[t][0] : dense_f4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                for (int t = 0; t < TN; ++t) acc[m][t0 + t] += sum[t][0] + sum[t][1];
            }
        }
    }
    // 2^118 as in the dense kernel, and room for sums of 2^19 sources: otherwise this wavefront's sources are added one by one
    const bool plain = __any(largest > 0x71000000u);
    int again = threadIdx.x;                               // (what the loop above does not need is derived again: registers are short)
    asm volatile("" : "+v"(again));
    const int q4_out = (again >> 4) & 3, f_out = fc * 16 * VEC + VEC * (again & 15);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int t = 0; t < VEC; ++t) acc[m][t][r] *= 0.5f / kDenseScale;
            if (plain) {
                Vec y;
#pragma unroll
                for (int t = 0; t < VEC; ++t) y.e[t] = 0.f;
                for (int s = s0; s < s1; ++s)
                    for (int k = 0; k < kTileStep; ++k) {
                        const uint32_t w = A.bits[(size_t)s * kTileRows + 2 * (k / 8 * 16 + 4 * q4_out + r) + m / 4];
                        if (!((w >> (8 * (m % 4) + k % 8)) & 1)) continue;
                        const Vec z = load(A.ids[(size_t)s * kTileStep + k]);
#pragma unroll
                        for (int t = 0; t < VEC; ++t) y.e[t] += z.e[t];
                    }
#pragma unroll
                for (int t = 0; t < VEC; ++t) acc[m][t][r] = y.e[t];
            }
        }
    if (f_out >= A.d) return;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * m + 4 * q4_out + r, node = A.rows[(size_t)unit.tile * kTileRows + row];
            if (node < 0) continue;
            float *out = unit.slot < 0 ? A.out + (size_t)node * A.d : A.part + ((size_t)unit.slot + (size_t)row * unit.parts) * A.d;
            Vec y;
#pragma unroll
            for (int t = 0; t < VEC; ++t) y.e[t] = acc[m][t][r];
            if (A.self && unit.slot < 0) {
                Vec own;
                own.v = *reinterpret_cast<const vec_t *>(A.self + (size_t)node * A.d + f_out);
                const float scale = A.self_scale ? A.self_scale[node] : 1.f;
#pragma unroll
                for (int t = 0; t < VEC; ++t) y.e[t] += own.e[t] * scale;
            }
            *reinterpret_cast<vec_t *>(out + f_out) = y.v;
        }
}

int launch_tiles(TileArgs a, hipStream_t s) {
    const int vec = dense_vec(a.d);
    a.f_chunks = (a.d + 16 * vec - 1) / (16 * vec);
    const int64_t per = kBlock / kWave, blocks = ((int64_t)a.longest_range * a.f_chunks + per - 1) / per * kPartitions;
    if (blocks <= 0) return HAG_OK;
    if (blocks > 0x7fffffffLL) { set_error("launch too large"); return HAG_EINVAL; }
    const dim3 grid((unsigned)blocks), block(kBlock);
    switch (vec) {
        case 1: hipLaunchKernelGGL(tile_kernel<1>, grid, block, 0, s, a); break;
        case 2: hipLaunchKernelGGL(tile_kernel<2>, grid, block, 0, s, a); break;
        default: hipLaunchKernelGGL(tile_kernel<4>, grid, block, 0, s, a); break;
    }
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

}  // namespace hag
