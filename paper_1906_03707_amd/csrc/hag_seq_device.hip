// Device path for a SEQUENTIAL Aggregate (Section 3.1): an LSTM aggregator over ordered neighbour
// lists, run over a prefix HAG found by hag_seq_search (or over the plain lists).
//
// A prefix HAG turns the lists into a forest of states: the state after the one-element prefix (u)
// has no predecessor, an aggregation node w = (v1, v2) is "the state of v1, then x[v2]" (Equation 2:
// cover(w) = (cover(v1), cover(v2))), and every v continues from the state of its list's head
// through the rest of its list (Algorithm 2: aggregation nodes first, then the nodes of V).  The
// forest is cut into PATHS: every state hands its running (h, c) on to one continuation (its
// largest subtree, or one node's private remainder) without a trip through memory, and is written
// to memory only if something else needs it (another path starts there, or it is some a_v).  A path
// that starts from a written state is one level above the path that wrote it; paths run 64 per workgroup, each step a
// matrix product on the matrix cores.  The half of the gates that depends on the input row only, W_ih x + b, is computed once
// per node (a node occurs in many lists); a step adds to it
//     gates^T [4H, paths] += W_hh [4H, H] . H^T [H, paths],
// with fp32 operands cut into two fp16 pieces.  The rows of W_hh are ordered so that a lane ends up holding all four gates
// of its hidden units for its path and the cell's element-wise part runs in registers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "hag_device_common.hpp"

struct hag_seq {
    int64_t n = 0, e = 0, n_merges = 0, n_states = 0;
    std::vector<int32_t> final_state; // per node: state row holding a_v, -1 for an empty list, -2: written by its path
    // paths, level by level, longest first within a level: 4 per path, (state row it starts from or -1,
    // first step, steps, node whose a_v its last h is or -1); per step the input row and the state row the
    // step's (h, c) is written to (-1: not needed outside the path)
    std::vector<int32_t> paths, step_x, step_out;
    std::vector<int64_t> level_ptr;   // paths of level l: [level_ptr[l], level_ptr[l+1])
    std::vector<int64_t> tile_ptr;    // tiles of 64 paths of level l: [tile_ptr[l], tile_ptr[l+1]) (a tile never mixes levels)
    // The same paths in the order of the one-launch pass: grouped by the DEPTH of the state they start from (the
    // number of evaluations behind it; 0 for the zero state), longest first within a group.  A path that writes a
    // state starts from a shallower one, so here too a path depends only on earlier groups; and the order follows
    // the time at which start states become available, which keeps tiles from waiting.
    std::vector<int32_t> paths_by_depth;
    std::vector<int64_t> depth_ptr, depth_tile_ptr;
    int64_t longest = 0;
    int64_t n_empty = 0, n_from_state = 0;   // nodes with an empty list; nodes whose a_v is a state that no path of their own ends in
    bool one_launch = true;           // HAG_SEQ_ONE_LAUNCH (default 1): all levels in one launch, paths waiting for the states they start from
    int32_t spin_limit = 1 << 21;     // HAG_SPIN_LIMIT: polls (about half a microsecond apart) after which such a wait gives up
    bool wait_unreachable = false;    // tests only: flags are never set, so every wait gives up
    int32_t *d_final = nullptr, *d_paths = nullptr, *d_step_out = nullptr;   // d_paths: padded to whole tiles per level
    int32_t *d_paths_by_depth = nullptr;                    // likewise per depth group
    // for the backward pass: per step where its h_{t-1} lives (>= 0: that step's tape row, -1: the zero state,
    // <= -2: state row -(value) - 2); all three in the order of the input row that the steps read: the steps, their step_prev, the
    // place of the input row among the used ones
    std::vector<int32_t> xt_idx, xt_prev, xt_seg;
    std::vector<int32_t> used, step_g;   // the nodes that occur in a list, ascending; per step the place of its input row among them
    std::vector<int32_t> pending_init;   // per state: the paths that start from it
    int32_t *d_xt_idx = nullptr, *d_xt_prev = nullptr, *d_xt_seg = nullptr, *d_pending_init = nullptr;
    int32_t *d_used = nullptr, *d_step_g = nullptr;
    int64_t resident_reverse[3] = {0, 0, 0};   // reverse kernel variants: hidden up to 32, 64, 128
    int64_t resident[3] = {0, 0, 0}, resident_tape[3] = {0, 0, 0};   // forward kernel variants, without and with the tape: workgroups the device holds at once (set by hag_seq_upload)
    int32_t *d_gave_up = nullptr;     // set by a wait that gave up; read and cleared by hag_seq_check
    int device = -1;
};

namespace hag {

constexpr int kSeqJobs = 64;      // paths per tile
constexpr int kSeqMaxK = 256;     // D + H at most

typedef float seq_acc_t __attribute__((ext_vector_type(16)));
typedef __bf16 seq_b8_t __attribute__((ext_vector_type(8)));
typedef _Float16 seq_h8_t __attribute__((ext_vector_type(8)));
typedef _Float16 seq_h2_t __attribute__((ext_vector_type(2)));
typedef __bf16 seq_b2_t __attribute__((ext_vector_type(2)));
typedef float seq_f2_t __attribute__((ext_vector_type(2)));
typedef unsigned int seq_u2_t __attribute__((ext_vector_type(2)));

// An fp32 number as the sum of three bf16 numbers: 8 + 8 + 8 significant bits hold the 24 of an fp32 exactly, so a product
// of two such sums loses only the terms mid * lo, lo * mid and lo * lo, about 2^-26 of the product and of either sign
// (round to nearest at every cut), which is below the rounding of the fp32 accumulator.  Two numbers at a time,
// packed as the low and the high half of each word.
// Numbers above kSeqSplitMost have no first piece, and those below 2^-109 no whole third one (bf16 ends at 2^-133): whoever cuts numbers without a
// bound keeps to this range, the lower end for the largest of those that are added up.
constexpr float kSeqSplitMost = 0x1.fep127f, kSeqSplitLeast = 0x1p-100f;
__device__ __forceinline__ void seq_split2(float a, float b, uint32_t (&p)[3]) {
#pragma clang fp contract(off)   // the pieces are those of the rounded number, however it was computed
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const seq_f2_t v = {a, b};
        p[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, seq_b2_t));
        if (k < 2) { a -= __uint_as_float(p[k] << 16); b -= __uint_as_float(p[k] & 0xffff0000u); }
    }
}

// The operands of the recurrent product in the forward pass as two fp16 numbers each, 11 + 11 significant bits: what is cut off is 2^-23 of a number at
// most, 2^-25 on average and of either sign, about what one fp32 addition rounds, and a product needs three matrix instructions
// instead of six.  Both operands fit fp16's range because both are bounded: |h| <= 1 is multiplied by 2^15 and the weights of a gate row by the power of two
// that brings the largest to [2^14, 2^15), so what the second piece of a small number rounds off (2^-25, the subnormal numbers of fp16) is
// 2^-40 of that.  A smaller h or weight than 2^-17 of the largest loses bits, which the others hide: the gate functions leave errors of a few 2^-25 in h, and the row's
// largest weight hands them on.  Where output gates let only e^-k through and weights of 0.3 e^k make up for it, the error of the result is that of three bf16 pieces up to k = 16
// (8 units: 8.4e-6 and 7.8e-6, from the rounding of such a gate's own pre-activation); with weights of 2e7 and 1e9 (k = 18 and 22) it is 3e-5 and 2e-3 (bf16 pieces 8e-6 and 6e-5).
constexpr float kSeqHScale = 32768.f;
constexpr int kSeqHScaleExp = 15;
constexpr float kSeqXMost = 0x1p60f;   // see seq_input_gates_kernel
__device__ __forceinline__ void seq_halves2(float a, float b, uint32_t (&p)[2]) {   // two numbers, packed as the low and the high half of each word
#pragma clang fp contract(off)
    const seq_f2_t v = {a, b};
    const seq_h2_t hi = __builtin_convertvector(v, seq_h2_t);
    const seq_f2_t r = {fmaf((float)hi.x, -1.f, a), fmaf((float)hi.y, -1.f, b)};   // exact; one mixed-precision instruction each
    p[0] = __builtin_bit_cast(uint32_t, hi);
    p[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, seq_h2_t));
}

// The same where small numbers beside large ones count too, as in the backward pass: the second piece times 2^11, which makes it as large as the first one, so that of numbers
// up to 2^15 it rounds off 2^-36 instead of 2^-25.  The products with a second piece are summed first and multiplied by 2^-11 before those of the first pieces join them.
constexpr float kSeqLow = 2048.f;
__device__ __forceinline__ void seq_halves2_low(float a, float b, uint32_t (&p)[2]) {
#pragma clang fp contract(off)
    const seq_f2_t v = {a, b};
    const seq_h2_t hi = __builtin_convertvector(v, seq_h2_t);
    const seq_f2_t r = {fmaf((float)hi.x, -kSeqLow, a * kSeqLow), fmaf((float)hi.y, -kSeqLow, b * kSeqLow)};   // exact
    p[0] = __builtin_bit_cast(uint32_t, hi);
    p[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, seq_h2_t));
}

constexpr float kSeqHLeast = 0x1p-26f;   // the smallest h that keeps all its bits so: its second piece rounds off 2^-51

// Weights in the forms the kernels read, from the usual layout (w_ih [4H, D], w_hh [4H, H], b [4H], gate-major rows: input,
// forget, cell, output gate).  Pre-activations are kept multiplied by a power of two of their gate row (see seq_halves2):
//   wx: W_ih for the product over input rows, fp32, times the rows' factors too, [gate tile][dp / 8 groups of four k-steps][lane][4]; lane l supplies
//       column l % 32 of the tile (gate row tile * 32 + l % 32 in (unit, gate) order) and k = 2 * step + l / 32;
//   wq: W_hh for the recurrent product times the rows' factors, two fp16 pieces, [gate tile][ks steps of 16][piece][lane][8]; lane l supplies row
//       l % 32 of the tile, k = 16 * step + 8 * (l / 32) + 0..7.  Row 8 m + 4 p + gate of a tile is that gate of hidden unit
//       8 * tile + 4 p + m, so that lane l of the product ends up with all gates of four CONSECUTIVE units;
//   bp: in (unit, gate) order, the bias times the factor; what turns a pre-activation into the exponent of its gate function, -log2(e) over the row's factor, twice that for the cell gate,
//       whose tanh is a function of 2 z; the factor itself, negative where the row is too large to be multiplied: W_ih and the bias then stay as they are.
// One workgroup per unit.  The "state is written" counters of the pass start at zero, and a_v of the nodes with an empty list is zero (final_state NULL: there are none).
__global__ __launch_bounds__(256) void seq_pack_kernel(const float *__restrict__ w_ih, const float *__restrict__ w_hh,
                                                      const float *__restrict__ b, float *__restrict__ wx,
                                                      uint16_t *__restrict__ wq, float *__restrict__ bp, int d, int dp,
                                                      int hidden, int ks, int32_t *__restrict__ flags, int64_t n_flags,
                                                      const int32_t *__restrict__ final_state, float *__restrict__ a_out, int64_t n) {
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
    for (int64_t f = first; f < n_flags; f += stride) flags[f] = 0;
    if (final_state) {                                     // 64 nodes per wavefront, as in seq_output_kernel
        const int lane = threadIdx.x & 63;
        for (int64_t base = first - lane; base < n; base += stride)
            for (unsigned long long left = __ballot(base + lane < n && final_state[base + lane < n ? base + lane : 0] == -1); left; left &= left - 1)
                for (int u = lane; u < hidden; u += 64) a_out[(base + __builtin_ctzll(left)) * hidden + u] = 0.f;
    }
    const int unit = blockIdx.x, gate = threadIdx.x >> 6, lane = threadIdx.x & 63;   // a wavefront per gate row
    if (unit >= hidden) return;
    const float *row = w_hh + (size_t)(gate * hidden + unit) * hidden;
    float v[2];                                            // (hidden is 128 at most)
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = lane + 64 * i < hidden ? row[lane + 64 * i] : 0.f;
    float most = fmaxf(fabsf(v[0]), fabsf(v[1]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = fmaxf(most, __shfl_xor(most, off));
    // (weights below 2^-26 are not brought up all the way: what they lose is 2^-66, and pre-activations up to 2^72 have a place in fp32)
    const int up = most < INFINITY ? min(15 - __builtin_amdgcn_frexp_expf(most), 40) : 0;
    const float by = __builtin_ldexpf(1.f, up);
    const int r = 4 * unit + gate, tile = unit >> 3, in_tile = 8 * (unit & 3) + 4 * ((unit >> 2) & 1) + gate;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = lane + 64 * i;
        if (k >= 16 * ks) continue;
        uint32_t p[2];
        seq_halves2(v[i] * by, 0.f, p);
        uint16_t *out = wq + (size_t)(tile * ks + (k >> 4)) * 1024 + (in_tile + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
        out[0] = (uint16_t)(p[0] & 0xffffu);
        out[512] = (uint16_t)(p[1] & 0xffffu);
    }
    // a row of usual size leaves the sums of seq_input_gates_kernel within 2^126 for features below kSeqXMost
    const float *row_x = w_ih + (size_t)(gate * hidden + unit) * d;
    float all = lane == 0 ? fabsf(b[gate * hidden + unit]) : 0.f;
    for (int k = lane; k < d; k += 64) all += fabsf(row_x[k]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) all += __shfl_xor(all, off);
    const float factor = __builtin_ldexpf(1.f, up + kSeqHScaleExp);
    const bool large = !(all * factor < 0x1p126f / kSeqXMost);
    const float with_h = large ? 1.f : factor;
    for (int k = lane; k < dp; k += 64)
        wx[(size_t)(r >> 5) * 32 * dp + (k >> 3) * 256 + ((r & 31) + 32 * (k & 1)) * 4 + ((k >> 1) & 3)] = k < d ? row_x[k] * with_h : 0.f;
    if (lane == 0) {
        bp[r] = b[gate * hidden + unit] * with_h;
        bp[4 * hidden + r] = __builtin_ldexpf(gate == 2 ? -2.f * 1.44269504f : -1.44269504f, -up - kSeqHScaleExp);
        bp[8 * hidden + r] = large ? -factor : factor;
    }
}

// The input half of the gates, once per node that occurs in a list instead of once per cell that reads it:
//     gx[i] = (b + W_ih x[used[i]]) times the row's factor   ([n_used, 4H], (unit, gate) order),
// 64 nodes per workgroup against all gate rows, fp32 matrix-core products, nodes as rows so that a store instruction writes
// 128 contiguous bytes of two rows.  On the lists of the benchmark every row serves 6 to 16 cells; the sums start from the
// bias and take the columns in order, as a product over (x, h) in one piece would.
// Features above kSeqXMost and rows marked by seq_pack_kernel would overflow with the factor in the weights (two terms of opposite signs then make NaN): their sums are
// taken without it, in all of fp32's range, and multiplied afterwards.  What that would bring beyond 2^127 stays there, where the gate functions have long reached their
// limits (it is 2^72 without the factor) and the recurrent half, 2^37 at most, does not count.
template <bool LARGE>
__device__ __forceinline__ void seq_input_gates_tile(const float *xl, const float4 *wq, int zs, int dp, float bias, float factor, seq_acc_t (&acc)[2]) {
    const float down = LARGE && factor > 0.f ? 1.f / factor : 1.f;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[g][r] = LARGE ? bias * down : bias;
    float4 wa = wq[0];
    for (int q = 0; q < dp / 8; ++q) {
        const float4 wn = wq[(q + 1 < dp / 8 ? q + 1 : q) * 64];
        const float w4[4] = {wa.x, wa.y, wa.z, wa.w};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int g = 0; g < 2; ++g)
                acc[g] = __builtin_amdgcn_mfma_f32_32x32x2f32(xl[g * 32 * zs + 2 * (4 * q + r)], LARGE ? w4[r] * down : w4[r], acc[g], 0, 0, 0);
        wa = wn;
    }
    if constexpr (LARGE) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float z = acc[g][r] * fabsf(factor);
                acc[g][r] = fabsf(z) > 0x1p127f ? copysignf(0x1p127f, z) : z;   // (NaN stays)
            }
    }
}
__global__ __launch_bounds__(256, 3) void seq_input_gates_kernel(const float *__restrict__ x, const int32_t *__restrict__ used, int64_t n_used,
                                                             const float *__restrict__ wx, const float *__restrict__ bp,
                                                             float *__restrict__ gx, int d, int dp, int hidden) {
    extern __shared__ float xs[];                          // [64][dp + 2]: rows 2 banks apart
    __shared__ int32_t large_at;                           // the last block of nodes with a large feature
    const int zs = dp + 2, n_tiles = hidden / 8, rows4 = 4 * hidden;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t blocks = (n_used + 63) / 64;
    if (threadIdx.x == 0) large_at = -1;
    __syncthreads();
    for (int64_t bt = blockIdx.x; bt < blocks; bt += gridDim.x) {
        {
            const int row = threadIdx.x >> 2;
            const int64_t at = bt * 64 + row;
            const int u = at < n_used ? used[at] : -1;
            float most = 0.f;
            for (int k = (threadIdx.x & 3) * 4; k < dp; k += 16) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (u >= 0 && k < d) v = *reinterpret_cast<const float4 *>(x + (size_t)u * d + k);
                *reinterpret_cast<float2 *>(&xs[row * zs + k]) = make_float2(v.x, v.y);
                *reinterpret_cast<float2 *>(&xs[row * zs + k + 2]) = make_float2(v.z, v.w);
                most = fmaxf(fmaxf(most, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
            }
            if (most > kSeqXMost) large_at = (int32_t)bt;
        }
        __syncthreads();
        const bool large = large_at == (int32_t)bt;
        for (int tile = wave; tile < n_tiles; tile += 4) {
            const float bias = bp[tile * 32 + (lane & 31)], factor = bp[8 * hidden + tile * 32 + (lane & 31)];
            seq_acc_t acc[2];
            const float4 *wq = reinterpret_cast<const float4 *>(wx) + (size_t)tile * (dp / 8) * 64 + lane;
            const float *xl = &xs[(lane & 31) * zs + (lane >> 5)];
            if (large || __any(factor < 0.f)) seq_input_gates_tile<true>(xl, wq, zs, dp, bias, factor, acc);
            else seq_input_gates_tile<false>(xl, wq, zs, dp, bias, factor, acc);
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t at = bt * 64 + g * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
                    if (at < n_used) gx[(size_t)at * rows4 + tile * 32 + (lane & 31)] = acc[g][r];
                }
        }
        __syncthreads();
    }
}

// Gate functions on the hardware's exp2 and reciprocal: absolute error of a few 1e-7 on outputs in (0, 1) and
// (-1, 1), against ~150 instructions per hidden unit for the library versions, which made the element-wise
// part as long as the matrix products.
// Of a pre-activation times a factor, with `by` = -log2(e) over that factor (tanh: of 2 z).
__device__ __forceinline__ float seq_sigmoid(float z, float by) { return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(z * by)); }
__device__ __forceinline__ float seq_tanh(float z, float by) {
    const float e = __builtin_amdgcn_exp2f(fabsf(z) * by);   // in (0, 1]: no overflow, no cancellation in 1 + e
    return copysignf((1.f - e) * __builtin_amdgcn_rcpf(1.f + e), z);
}
// seq_sigmoid(z, by) * seq_tanh(x, by_x); the denominators' product is infinite only where the first factor is 0, and so is the result
__device__ __forceinline__ float seq_sigmoid_tanh(float z, float by, float x, float by_x) {
    const float e = __builtin_amdgcn_exp2f(fabsf(x) * by_x);
    return copysignf((1.f - e) * __builtin_amdgcn_rcpf((1.f + __builtin_amdgcn_exp2f(z * by)) * (1.f + e)), x);
}
__device__ __forceinline__ float seq_tanh(float z) { return seq_tanh(z, -2.f * 1.44269504f); }

struct SeqChainArgs {
    const int32_t *chains;   // paths, 4 per path, in tiles of 64 (padded with empty paths), longest first within a level
    int64_t n_path_tiles;
    int32_t *flags;          // per state row: the wavefronts that have written their part of it (NULL: every start state was written by an earlier launch)
    int32_t *gave_up;        // set by a wait that gives up
    int32_t spin_limit;      // polls of a flag before giving up
    int32_t publish;         // 0 in a test of the time-out: no flag is ever set
    const int32_t *step_g;   // per step: row of gx
    const int32_t *step_out; // per step: state row to write, or -1
    const float *gx;         // the input half of the gates, [n_used, 4H] in (unit, gate) order
    const uint16_t *wq;      // W_hh in fp16 pieces, see seq_pack_kernel
    const float *unscale;    // per gate row in (unit, gate) order, see seq_pack_kernel
    float *h, *c;            // [n_states, H]: read where a path starts (written by a lower level), written where a step says so
    float *a_out;            // [n, H]
    float *tape_g, *tape_c, *tape_h;   // training: per step the activated gates [H][4], the new c [H] and the new h [H] (NULL: inference)
    int32_t hidden;
};

// State rows that another workgroup of the same launch reads, possibly on another XCD: device-scope accesses,
// which are written through to, and read from, the level all XCDs share instead of a private cache; eight bytes
// at a time (the widest access that has a device-scope form).
__device__ __forceinline__ float4 seq_ld4_device(const float *p) {
    const unsigned long long a = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long b = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float4(__uint_as_float((unsigned)a), __uint_as_float((unsigned)(a >> 32)), __uint_as_float((unsigned)b), __uint_as_float((unsigned)(b >> 32)));
}
__device__ __forceinline__ void seq_st4_device(float *p, float4 v) {
    const unsigned long long a = (unsigned long long)__float_as_uint(v.x) | ((unsigned long long)__float_as_uint(v.y) << 32);
    const unsigned long long b = (unsigned long long)__float_as_uint(v.z) | ((unsigned long long)__float_as_uint(v.w) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p) + 1, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Hides a value's origin from the optimiser, so that what is derived from it is computed where it is used
// instead of being held in a register across the products.
__device__ __forceinline__ int seq_opaque(int v) { asm volatile("" : "+v"(v)); return v; }

// The 128 bytes that one path has of a gate tile (eight units, four gates) are held by lanes l and l + 32, four float4 each (unit
// 4 * (l / 32) + m).  Moved to memory as they are, an instruction would touch 16 or 32 bytes of 64 or 32 rows, which a streaming
// kernel moves at 2.9 TB/s here; exchanged between the rows of 16 lanes first, it touches 64 bytes of 16 paths (5.0 TB/s).  After
// seq_to_pieces lane l holds, of path l % 16 in v[0] and v[1] and of path 16 + l % 16 in v[2] and v[3], unit piece(l) and unit 4 + piece(l).
// All 64 lanes take part.
__device__ __forceinline__ int seq_piece(int lane) { return ((lane >> 5) & 1) | (((lane >> 4) & 1) << 1); }
__device__ __forceinline__ void seq_swap32(float &a, float &b) {
    const seq_u2_t v = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(v.x); b = __uint_as_float(v.y);
}
__device__ __forceinline__ void seq_swap16(float &a, float &b) {
    const seq_u2_t v = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(v.x); b = __uint_as_float(v.y);
}
// v: sixteen values, (m, gate); V is indexable (an array or an accumulator)
template <typename V>
__device__ __forceinline__ void seq_to_pieces(V &v, float4 (&p)[4]) {
    float r[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) r[e] = v[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        seq_swap32(r[e], r[4 + e]);           // -> units {0, 1} and {4, 5}
        seq_swap32(r[8 + e], r[12 + e]);      // -> units {2, 3} and {6, 7}
        seq_swap16(r[e], r[8 + e]);
        seq_swap16(r[4 + e], r[12 + e]);
    }
    p[0] = make_float4(r[0], r[1], r[2], r[3]);
    p[1] = make_float4(r[4], r[5], r[6], r[7]);
    p[2] = make_float4(r[8], r[9], r[10], r[11]);
    p[3] = make_float4(r[12], r[13], r[14], r[15]);
}
// the reverse, in place: v holds the float4 p[0], p[1], ... as seq_to_pieces leaves them
template <typename V>
__device__ __forceinline__ void seq_from_pieces(V &v) {
    float r[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) r[e] = v[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        seq_swap16(r[e], r[8 + e]);
        seq_swap16(r[4 + e], r[12 + e]);
        seq_swap32(r[e], r[4 + e]);
        seq_swap32(r[8 + e], r[12 + e]);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = r[e];
}

// Paths of one level, or of all.  A workgroup takes tiles of 64 paths and walks ALL their steps; the running states never leave
// the compute unit: c in registers, h in LDS as the operand of the next step's product.  A step reads one row of gx per path
// (the accumulators start from it), multiplies W_hh with the 64 h rows, runs the element-wise part on the result in
// registers and writes the new h to the other of two LDS buffers, so that a step has one barrier.  Paths are sorted by length, so
// the paths of a tile end within a step or two of each other; a path that has ended keeps quiet while the others finish.
//
// The product runs in fp16 pieces (seq_halves2): three v_mfma_f32_32x32x16_f16 per 16 columns, 96 cycles (bf16 pieces 192, fp32 instructions 512).
// Bound by what it issues, products and element-wise part one after the other: vector instructions 65 % of the time, matrix cores 22 % (64 units; with the tape 50 and 17 % at
// 3.3 TB/s, 128 units with the tape 38 and 19 % at 4.3 TB/s).  So sigmoid times tanh takes one reciprocal, and of 64 units no gates go to the tape.
// Measured: inference over 370 k nodes (hidden = d = 64, prefix HAG with 3.35 M cells) 723 us (bf16 pieces 877); the same with the tape, this kernel alone, 0.96 ms (1.49
// with the gates on it); 0.85 M cells of 128 units with the tape 1.01 ms.  Error of the result against 64 bits 1.9e-7 (bf16 pieces 2.1e-7).
// A gate tile is 32 gate rows = 8 hidden units; lane l of the product holds, for path l % 32 of its half of the tile, the four
// gates of units 8 * tile + 4 * (l / 32) + 0..3.
//   HMAX 64 (hidden 33..64): 8 wavefronts, wavefront w holds gate tile w in registers and takes both halves of the paths;
//   HMAX 32: wavefront w holds gate tile w % 4 and takes half w / 4;
//   HMAX 128: 16 wavefronts, wavefront w holds half of gate tile w in registers (a whole tile would be 64 of the 128 there are at four wavefronts per SIMD) and streams
//   the rest (2 KB per 16 columns) from the L2 cache once per step for both halves of the paths.  The weights in registers come first: the streamed ones, which
//   queue behind the tape's stores, arrive meanwhile (9 % faster than with all of the tile streamed).
template <int HMAX, bool TAPE>
__global__ __launch_bounds__(HMAX == 128 ? 1024 : 512, 4) void seq_chain_kernel(SeqChainArgs A) {
    constexpr bool BIG = HMAX == 128, WIDE = HMAX >= 64, C_LDS = HMAX == 64 || TAPE, GATES = TAPE && HMAX != 64;   // (of 64 units the backward pass computes the gates again)
    constexpr int KS = HMAX / 16, ZS = HMAX + 8, JG = WIDE ? 2 : 1;
    __shared__ __align__(16) uint16_t z[2][2][kSeqJobs][ZS];   // h of every path in fp16 pieces: this step's and the next step's
    __shared__ __align__(16) float hs[TAPE ? kSeqJobs : 1][HMAX + 4];   // the step's h as it is, for the tape
    // c: in registers, except where those are too short or the tape takes it from here (rows 4 banks apart: conflict-free 16-byte accesses)
    __shared__ __align__(16) float cs[C_LDS ? kSeqJobs : 1][HMAX + 4];
    __shared__ int32_t sdesc[kSeqJobs * 4];
    __shared__ int32_t spend[2][kSeqJobs];                 // per path: the state row that a step wrote, to be announced a step later
    __shared__ float4 sby[BIG ? HMAX : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
    const int hidden = A.hidden, n_tiles = hidden / 8, ks = BIG ? (hidden + 15) / 16 : KS;
    const int tile = WIDE ? wave : (wave & 3), group0 = WIDE ? 0 : (wave >> 2);
    const bool on = tile < n_tiles;                        // wavefronts beyond the hidden size only keep the barriers
    constexpr int KR = BIG ? 4 : KS;                       // steps of 16 columns whose weights stay in registers (above 64 units there are five at least)
    seq_h8_t wreg[KR][2];
    const seq_h8_t *wl = reinterpret_cast<const seq_h8_t *>(A.wq) + (size_t)tile * ks * 2 * 64 + lane;
    // what turns a lane's pre-activations into exponents, per unit (input, forget, cell, output gate): in registers where there are enough
    float4 by_reg[BIG ? 1 : 4];
    if constexpr (BIG) { if ((int)threadIdx.x < hidden) sby[threadIdx.x] = reinterpret_cast<const float4 *>(A.unscale)[threadIdx.x]; }   // (read behind the barriers of a tile)
    if (on) {
        if constexpr (!BIG) {
#pragma unroll
            for (int m = 0; m < 4; ++m) by_reg[m] = reinterpret_cast<const float4 *>(A.unscale)[tile * 8 + half * 4 + m];
        }
#pragma unroll
        for (int s = 0; s < KR; ++s)
#pragma unroll
            for (int p = 0; p < 2; ++p) wreg[s][p] = wl[(s * 2 + p) * 64];
    }
    // columns from `hidden` on stay zero in both buffers
    for (int i = threadIdx.x; i < (int)(sizeof(z) / 4); i += blockDim.x) reinterpret_cast<uint32_t *>(&z[0][0][0][0])[i] = 0;
    for (int64_t ct = blockIdx.x; ct < A.n_path_tiles; ct += gridDim.x) {
        {
            const int tid = seq_opaque(threadIdx.x);
            if (tid < kSeqJobs * 4) sdesc[tid] = A.chains[ct * (kSeqJobs * 4) + tid];
        }
        __syncthreads();
        if (A.flags) {
            // All levels in one launch: wait until the states this tile's paths start from are written.  They
            // belong to tiles with a smaller index, which this or another resident workgroup finishes without
            // waiting for this one, so the wait ends; it is bounded all the same, and a time-out is recorded.
            const int tid = seq_opaque(threadIdx.x);
            if (tid < kSeqJobs) {
                const int start = sdesc[tid * 4];
                if (start >= 0) {
                    bool ready = false;
                    for (int spin = 0; spin < A.spin_limit; ++spin) {
                        if (__hip_atomic_load(A.flags + start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= n_tiles) { ready = true; break; }
                        // once any wait of the pass has given up its output is void: the others do not sit theirs out
                        if (__hip_atomic_load(A.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
                        __builtin_amdgcn_s_sleep(16);
                    }
                    if (!ready) __hip_atomic_store(A.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            __syncthreads();
            // the awaited rows are read with device-scope loads, which do not look into a private cache, so no
            // cache is invalidated here; the fence keeps those loads behind the polls
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
        const int steps = sdesc[2];                        // the tile's first path is its longest
        int row[JG], keep[JG];                             // (begin and length are read from LDS where they are needed: registers are short)
        float4 creg[C_LDS ? 1 : JG];
        seq_acc_t acc[JG];
        auto load_gates = [&](int g) {                     // the accumulators of the next step start from these rows of gx (row -1: the path has ended); the pieces are put in place by seq_from_pieces when they are used, so that nothing waits for them here
            const seq_u2_t rows = __builtin_amdgcn_permlane16_swap((unsigned)row[g], (unsigned)row[g], false, false);   // of paths l % 16 and 16 + l % 16
            const int l = seq_opaque(threadIdx.x) & 63;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int r = (int)(q ? rows.y : rows.x);
                if (r >= 0) {
                    const float *p = A.gx + ((size_t)r * hidden + tile * 8 + seq_piece(l)) * 4;
                    const float4 v = *reinterpret_cast<const float4 *>(p), w = *reinterpret_cast<const float4 *>(p + 16);
                    acc[g][8 * q] = v.x; acc[g][8 * q + 1] = v.y; acc[g][8 * q + 2] = v.z; acc[g][8 * q + 3] = v.w;
                    acc[g][8 * q + 4] = w.x; acc[g][8 * q + 5] = w.y; acc[g][8 * q + 6] = w.z; acc[g][8 * q + 7] = w.w;
                }
            }
        };
        auto put_h = [&](int buf, int j, int unit0, const float (&h)[4]) {
            uint32_t a[2], b[2];
            seq_halves2(h[0] * kSeqHScale, h[1] * kSeqHScale, a);
            seq_halves2(h[2] * kSeqHScale, h[3] * kSeqHScale, b);
#pragma unroll
            for (int p = 0; p < 2; ++p) *reinterpret_cast<uint2 *>(&z[buf][p][j][unit0]) = make_uint2(a[p], b[p]);
        };
#pragma unroll
        for (int g = 0; g < JG; ++g) {
            const int l = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (l >> 5) * 4, j = (group0 + g) * 32 + (l & 31), start = sdesc[j * 4];
            const int beg = sdesc[j * 4 + 1], len = on ? sdesc[j * 4 + 2] : 0;   // (the path's row of gx for the next step is asked for a step ahead)
            row[g] = -1; keep[g] = -1;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][r] = 0.f;
            if (len > 0) {
                row[g] = A.step_g[beg];
                keep[g] = A.step_out[beg];
                float h[4] = {0.f, 0.f, 0.f, 0.f};
                float4 cv = make_float4(0.f, 0.f, 0.f, 0.f);
                if (start >= 0) {
                    const size_t o = (size_t)start * hidden + unit0;
                    const float4 hv = A.flags ? seq_ld4_device(A.h + o) : *reinterpret_cast<const float4 *>(A.h + o);
                    cv = A.flags ? seq_ld4_device(A.c + o) : *reinterpret_cast<const float4 *>(A.c + o);
                    h[0] = hv.x; h[1] = hv.y; h[2] = hv.z; h[3] = hv.w;
                }
                if constexpr (C_LDS) *reinterpret_cast<float4 *>(&cs[j][unit0]) = cv;
                else creg[g] = cv;
                put_h(0, j, unit0, h);
            }
            if (on) load_gates(g);
            row[g] = len > 1 ? A.step_g[beg + 1] : -1;
        }
        {
            const int tid = seq_opaque(threadIdx.x);
            if (tid < 2 * kSeqJobs) (&spend[0][0])[tid] = -1;
        }
        __syncthreads();
        // counts this wavefront off for the states it wrote a step ago: their stores are older than the rows of gx that the
        // product just used, so they have long completed
        auto publish = [&](int par) {
            if (!A.flags) return;
            int pend[JG];
            bool any = false;
#pragma unroll
            for (int g = 0; g < JG; ++g) { pend[g] = spend[par][(group0 + g) * 32 + (lane & 31)]; any |= pend[g] >= 0; }
            if (!__any(any)) return;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int g = 0; g < JG; ++g)
                if (pend[g] >= 0 && half == 0 && A.publish) __hip_atomic_fetch_add(A.flags + pend[g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        auto product = [&](int cur, int g, seq_acc_t &a, const seq_h8_t (&w)[2], int s) {
            seq_h8_t zb[2];
#pragma unroll
            for (int p = 0; p < 2; ++p)
                zb[p] = *reinterpret_cast<const seq_h8_t *>(&z[cur][p][(group0 + g) * 32 + (lane & 31)][16 * s + 8 * half]);
            a = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[1], zb[0], a, 0, 0, 0);
            a = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[0], zb[1], a, 0, 0, 0);
            a = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[0], zb[0], a, 0, 0, 0);
        };
        for (int t = 0; t < steps; ++t) {
            const int cur = t & 1;
            if (on) {
                if constexpr (BIG) {
                    // the others are requested first, two steps at a time, and arrive while the products of those in registers run
                    seq_h8_t wa[2][2];
                    auto load_w = [&](int i, int s) {
                        s = s < ks ? s : ks - 1;
#pragma unroll
                        for (int p = 0; p < 2; ++p) wa[i][p] = wl[(s * 2 + p) * 64];
                    };
                    load_w(0, KR);
                    load_w(1, KR + 1);
#pragma unroll
                    for (int g = 0; g < JG; ++g) seq_from_pieces(acc[g]);
#pragma unroll
                    for (int s = 0; s < KR; ++s)
#pragma unroll
                        for (int g = 0; g < JG; ++g) product(cur, g, acc[g], wreg[s], s);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int s = KR; s < 8; s += 2) {
                        if (s >= ks) break;
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            if (s + i < ks) {
#pragma unroll
                                for (int g = 0; g < JG; ++g) product(cur, g, acc[g], wa[i], s + i);
                            }
                            if (s + 2 < 8) load_w(i, s + 2 + i);
                        }
                    }
                }
#pragma unroll
                for (int g = 0; g < JG; ++g) {
                    if constexpr (!BIG) {
                        seq_from_pieces(acc[g]);
#pragma unroll
                        for (int s = 0; s < KS; ++s) product(cur, g, acc[g], wreg[s], s);
                    }
                    if (g == 0) publish(cur ^ 1);
                    const int l = seq_opaque(threadIdx.x) & 63, half = l >> 5, unit0 = tile * 8 + half * 4, j = (group0 + g) * 32 + (l & 31);
                    const int beg = sdesc[j * 4 + 1], len = sdesc[j * 4 + 2];
                    if (A.flags && half == 0) spend[cur][j] = t < len ? keep[g] : -1;
                    if (t < len) {
                        float4 cv;
                        if constexpr (C_LDS) cv = *reinterpret_cast<const float4 *>(&cs[j][unit0]);
                        else cv = creg[g];
                        float h[4], c[4] = {cv.x, cv.y, cv.z, cv.w};
#pragma unroll
                        for (int m = 0; m < 4; ++m) {
                            float4 by;
                            if constexpr (BIG) by = sby[unit0 + m];
                            else by = by_reg[m];
                            const float gf = seq_sigmoid(acc[g][4 * m + 1], by.y);
                            if constexpr (HMAX == 64) {
                                // sigmoid times tanh with one reciprocal of both denominators: the reciprocal is a quarter of a gate function's time
                                c[m] = fmaf(gf, c[m], seq_sigmoid_tanh(acc[g][4 * m], by.x, acc[g][4 * m + 2], by.z));   // (spelled out: one rounding, the same in every copy of this code)
                                h[m] = seq_sigmoid_tanh(acc[g][4 * m + 3], by.w, c[m], -2.f * 1.44269504f);
                            } else {
                                const float gi = seq_sigmoid(acc[g][4 * m], by.x), gg = seq_tanh(acc[g][4 * m + 2], by.z), go = seq_sigmoid(acc[g][4 * m + 3], by.w);
                                c[m] = fmaf(gf, c[m], gi * gg);
                                h[m] = go * seq_tanh(c[m]);
                                if constexpr (GATES) { acc[g][4 * m] = gi; acc[g][4 * m + 1] = gf; acc[g][4 * m + 2] = gg; acc[g][4 * m + 3] = go; }
                            }
                        }
                        put_h(cur ^ 1, j, unit0, h);
                        const float4 h4 = make_float4(h[0], h[1], h[2], h[3]), c4 = make_float4(c[0], c[1], c[2], c[3]);
                        if constexpr (C_LDS) *reinterpret_cast<float4 *>(&cs[j][unit0]) = c4;
                        else creg[g] = c4;
                        if constexpr (TAPE) *reinterpret_cast<float4 *>(&hs[j][unit0]) = h4;
                        // (gates, c and h leave for the tape further down, in larger pieces)
                        if (keep[g] >= 0) {                // a state that another path starts from, or some a_v
                            const size_t o = (size_t)keep[g] * hidden + unit0;
                            if (A.flags) {
                                seq_st4_device(A.h + o, h4);
                                seq_st4_device(A.c + o, c4);
                            } else {
                                *reinterpret_cast<float4 *>(A.h + o) = h4;
                                *reinterpret_cast<float4 *>(A.c + o) = c4;
                            }
                        }
                        if (t + 1 == len) {
                            // a_v = the last h of the path, where the path ends a node's list
                            const int node = sdesc[j * 4 + 3];
                            if (node >= 0) *reinterpret_cast<float4 *>(A.a_out + (size_t)node * hidden + unit0) = h4;
                            row[g] = -1;
                        } else {
                            keep[g] = A.step_out[beg + t + 1];
                        }
                    }
                    if constexpr (GATES) {
                        // the activated gates, for the backward pass, indexed by the step
                        float4 v[4];
                        seq_to_pieces(acc[g], v);
                        const int l = seq_opaque(threadIdx.x) & 63;
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const int jj = (group0 + g) * 32 + 16 * q + (l & 15);
                            if (t < sdesc[jj * 4 + 2]) {
                                float *p = A.tape_g + ((size_t)(sdesc[jj * 4 + 1] + t) * hidden + tile * 8 + seq_piece(l)) * 4;
                                st4_stream(p, v[2 * q]);   // (streaming stores: nothing reads the tape before the backward pass)
                                st4_stream(p + 16, v[2 * q + 1]);
                            }
                        }
                    }
                    load_gates(g);
                    if (t + 2 < len) row[g] = A.step_g[beg + t + 2];
                }
            }
            __syncthreads();                               // the h rows of the next step are complete, this step's have been read
            if constexpr (TAPE) {
                // h and c of the step as whole rows.  A wavefront holds 32 bytes of
                // c per path: written from there, they left as 64-byte requests that were half empty (6.8 GB instead of 5.9 at 3.35 M cells of 64
                // units: 2.18 ms, now 1.59; 0.85 M cells of 128: 1.33 and 1.19).
                const int tid = seq_opaque(threadIdx.x), j = tid / (HMAX / 8), part = tid % (HMAX / 8);
                if (j < kSeqJobs && t < sdesc[j * 4 + 2]) {
                    const size_t cell = (size_t)(sdesc[j * 4 + 1] + t) * hidden;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int u = part * 4 + i * (HMAX / 2);
                        if (u >= hidden) continue;
                        st4_stream(A.tape_h + cell + u, *reinterpret_cast<const float4 *>(&hs[j][u]));
                        st4_stream(A.tape_c + cell + u, *reinterpret_cast<const float4 *>(&cs[j][u]));
                    }
                }
                __syncthreads();                           // the rows of h and c have been read
            }
        }
        if (on) publish((steps - 1) & 1);
        __syncthreads();
    }
}

// a_v of the nodes whose whole list is a shared prefix: that state's h.  Most nodes are written by their path, so a
// wavefront looks at 64 nodes at once and moves rows only for those that are left (one thread per element took 40 us for 370 k nodes).
__global__ __launch_bounds__(256) void seq_output_kernel(const int32_t *__restrict__ final_state, const float *__restrict__ h,
                                                        float *__restrict__ out, int64_t n, int hidden) {
    const int lane = threadIdx.x & 63;
    const int64_t base = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
    const int state = base + lane < n ? final_state[base + lane] : -2;
    for (unsigned long long left = __ballot(state >= 0); left; left &= left - 1) {
        const int b = __builtin_ctzll(left), s = __builtin_amdgcn_readlane(state, b);
        for (int u = lane; u < hidden; u += 64) out[(size_t)(base + b) * hidden + u] = h[(size_t)s * hidden + u];
    }
}


// ---------------------------------------------------------------------------------------------------------
// Backward pass (backpropagation through time along the same paths, last step first).  For the cell of a step,
// with the gradients dh, dc of its outputs:  t = tanh(c'),  d_o = dh t,  dc += dh o (1 - t^2),
//   dG = d(pre-activations) = (dc g i(1-i),  dc c f(1-f),  dc i (1-g^2),  d_o o(1-o)),   dc_prev = dc f,
//   dh_prev = W_hh^T dG,   dW_hh += dG h_prev^T;
// what depends on the input row x[u] goes through the sum of dG over the steps that read it, once per node:
//   s[u] = sum of dG,   g_x[u] = W_ih^T s[u],   dW_ih = sum over u of s[u] x[u]^T,   db = sum over u of s[u].
// A state that other paths start from (or that is some a_v) collects their gradients in its row of gh / gc; levels
// run last to first, so a path finds those rows complete when it reaches the step that wrote the state.

struct SeqRevArgs {
    const int32_t *paths;    // this level's paths in tiles of 64
    int64_t n_path_tiles;
    const int32_t *step_out;
    const uint16_t *wqt;     // W_hh^T in fp16 pieces, in the order the matrix instructions consume it, see seq_backward_start_kernel
    const int32_t *wqt_unscale; // per hidden unit, likewise
    float *tape_g;           // out: the gradients of every step's pre-activations; in, but for 40 to 64 units: its activated gates
    const float *tape_c, *tape_h;   // c' and h of every step
    const float *h_state, *c_state; // rows of the kept states
    // for 40 to 64 units, what the forward pass computed the gates from (see SeqChainArgs)
    const int32_t *step_g;
    const float *gx;
    const uint16_t *wq;
    const float *unscale;
    const float *g_a;        // [n, H]
    float *gh, *gc;          // [n_states, H]
    // all levels in one launch (NULL: one launch per level): per kept state the number of paths that start from it
    // and have not sent their gradients yet; tiles are taken last first
    int32_t *pending;
    int32_t *gave_up;
    int32_t spin_limit, reversed;
    int32_t publish;         // 0 in a test of the time-out: no path is ever counted off
    int32_t hidden;
};


// the largest of sixteen lanes, in all of them
__device__ __forceinline__ float seq_max16(float v) {
#define HAG_SEQ_ROR(n) v = fmaxf(v, __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x120 + n, 0xf, 0xf, false)))
    HAG_SEQ_ROR(8); HAG_SEQ_ROR(4); HAG_SEQ_ROR(2); HAG_SEQ_ROR(1);
#undef HAG_SEQ_ROR
    return v;
}
// The power of two that brings numbers of size `most` to [2^14, 2^15), as its exponent: as far up as fp16's range allows, so that what the second piece
// of a number rounds off (see seq_halves2_low) is 2^-51 of the largest.  Infinities and NaN stay what they are; beside an infinity the factor is 1 and numbers above 65504
// become infinite too, in sums that are not finite anyway.
__device__ __forceinline__ int seq_up(float most) { return most < INFINITY ? min(15 - __builtin_amdgcn_frexp_expf(most), 125) : 0; }
// Sums of products of two such operands are put right in two steps, neither of which leaves fp32's range: by 2^(-kSeqBack - up) of the gradients' power, which is at
// least 2^-149 and leaves up to 512 terms of the largest gradient's size, and by the exponent kSeqBack - up of the weights'.
// Between the two steps gradients are 2^9 times smaller than in the end: of those below 2^-115 last bits go (gradients of 1e-36: errors of up to 1.1e-6).
constexpr int kSeqBack = 24;

// What the backward pass starts from, in one launch: cleared gradient rows of the kept states, cleared g_x where some node is in no list
// (n_g_x > 0), the pending counts of a one-launch pass (n_states > 0) and the weights of the products, from the usual layout.
//   wqt: W_hh^T in two fp16 pieces (seq_halves2_low), the weights of an output unit (a column of W_hh) brought to a common size by a power of two (seq_up); unscale: per output
//       unit the exponent that undoes it, see kSeqBack;
//     hidden <= 64: [gate tile][m_tiles of 32 hidden units][2 steps of 16][piece][lane][8]; lane l supplies output unit 32 * mt + l % 32, and as k
//       value e = 8 * step + i = 4 m + gate the gate row of unit 8 * tile + 4 * (l / 32) + m: the order in which the lanes hold dG;
//     hidden > 64: [m_tiles][4H / 16 steps][piece][lane][8]; lane l supplies unit 32 * mt + l % 32, k = 16 * step + 8 * (l / 32) + i the gate
//       row in (unit, gate) order;
//   wxt: W_ih^T for g_x: [d tiles of 32 columns][4H / 8 groups of four k-steps][lane][4]; lane l supplies column 32 * tile + l % 32,
//       k-step q the gate rows 2 q + l / 32.
// The first 32 * m_tiles workgroups (there are at least as many) cut one column of W_hh each.
__global__ __launch_bounds__(256) void seq_backward_start_kernel(const float *__restrict__ w_ih, const float *__restrict__ w_hh,
                                                                uint16_t *__restrict__ wqt, int32_t *__restrict__ unscale, float *__restrict__ wxt, int d, int hidden,
                                                                float *__restrict__ state_grads, int64_t n_state_grads, float *__restrict__ g_x,
                                                                int64_t n_g_x, const int32_t *__restrict__ pending_init,
                                                                int32_t *__restrict__ pending, int64_t n_states) {
    __shared__ float largest[4];
    const int m_tiles = (hidden + 31) / 32, d_tiles = (d + 31) / 32, rows = 4 * hidden;
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
    for (int64_t i = first; i < n_state_grads; i += stride) state_grads[i] = 0.f;
    for (int64_t i = first; i < n_g_x; i += stride) g_x[i] = 0.f;
    for (int64_t i = first; i < n_states; i += stride) pending[i] = pending_init[i];
    for (int64_t i = first; i < (int64_t)d_tiles * 32 * rows; i += stride) {
        const int tile = (int)(i / (32 * rows)), rest = (int)(i % (32 * rows)), q = rest / 256, lane = (rest % 256) / 4;
        const int r = 2 * (4 * q + (rest & 3)) + (lane >> 5), z = tile * 32 + (lane & 31);
        wxt[i] = z < d ? w_ih[(size_t)((r & 3) * hidden + (r >> 2)) * d + z] : 0.f;
    }
    const int z = blockIdx.x, mt = z >> 5;
    if (z >= 32 * m_tiles) return;
    float v[2], most = 0.f;                                // row r = threadIdx.x + 256 i of the column, in (unit, gate) order (4H is 512 at most)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = threadIdx.x + 256 * i;
        v[i] = z < hidden && r < rows ? w_hh[(size_t)((r & 3) * hidden + (r >> 2)) * hidden + z] : 0.f;
        most = fmaxf(most, fabsf(v[i]));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = fmaxf(most, __shfl_xor(most, off));
    if ((threadIdx.x & 63) == 0) largest[threadIdx.x >> 6] = most;
    __syncthreads();
    const int up = seq_up(fmaxf(fmaxf(largest[0], largest[1]), fmaxf(largest[2], largest[3])));
    const float by = __builtin_ldexpf(1.f, up);
    if (threadIdx.x == 0 && z < hidden) unscale[z] = kSeqBack - up;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = threadIdx.x + 256 * i;
        if (r >= rows) continue;
        uint32_t p[2];
        seq_halves2_low(v[i] * by, 0.f, p);
        size_t at;
        if (hidden <= 64) {
            const int unit = r >> 2, e = 4 * (unit & 3) + (r & 3);
            at = ((size_t)(((unit >> 3) * m_tiles + mt) * 2 + (e >> 3)) * 2 * 64 + (z & 31) + 32 * ((unit >> 2) & 1)) * 8 + (e & 7);
        } else {
            at = ((size_t)(mt * (rows / 16) + (r >> 4)) * 2 * 64 + (z & 31) + 32 * ((r >> 3) & 1)) * 8 + (r & 7);
        }
        wqt[at] = (uint16_t)(p[0] & 0xffffu);
        wqt[at + 512] = (uint16_t)(p[1] & 0xffffu);
    }
}

// a_v that is a shared state's h (the node's whole list is a shared prefix): its gradient goes to the state's row.  64 nodes per wavefront, as in
// seq_output_kernel.
__global__ __launch_bounds__(256) void seq_final_grad_kernel(const int32_t *__restrict__ final_state, const float *__restrict__ g_a,
                                                            float *gh, int64_t n, int hidden) {
    const int lane = threadIdx.x & 63;
    const int64_t base = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
    const int state = base + lane < n ? final_state[base + lane] : -2;
    for (unsigned long long left = __ballot(state >= 0); left; left &= left - 1) {
        const int b = __builtin_ctzll(left), s = __builtin_amdgcn_readlane(state, b);
        for (int u = lane; u < hidden; u += 64)
            __hip_atomic_fetch_add(gh + (size_t)s * hidden + u, g_a[(size_t)(base + b) * hidden + u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Waits (bounded) until everything that continues from a kept state has sent its gradients.  One launch for all levels: the paths
// that start from the state belong to tiles taken before this one, which never wait for it, so the count reaches zero.
__device__ __forceinline__ void seq_wait_pending(const SeqRevArgs &A, int keep) {
    bool ready = false;
    for (int spin = 0; spin < A.spin_limit; ++spin) {
        if (__hip_atomic_load(A.pending + keep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= 0) { ready = true; break; }
        if (__hip_atomic_load(A.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
        __builtin_amdgcn_s_sleep(16);
    }
    if (!ready) __hip_atomic_store(A.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");       // the sums are then read with device-scope loads
}

constexpr int kSeqRevJobs = 32;   // paths per workgroup of the reverse kernels above 32 hidden units: half a tile

// Hidden sizes up to 32.  Lanes and wavefronts are those of the forward kernel: a lane holds (path, four units of
// gate tile w), their running dh and dc and, per step, the sixteen dG.  The k index of dh_prev = W_hh^T dG can be taken in any order, so the
// dG are the product's operand where they are, in the registers of the lane that made them: wavefront w multiplies the 32 gate
// rows of its own tile and leaves its part of dh_prev for all units in LDS; after a barrier every lane adds the parts
// for its own units, in a fixed order.  The operands are two fp16 pieces each (seq_halves2_low): gradients have no bound, so the
// largest of a path's 32 gate rows in the tile says what power of two brings them into fp16's range (seq_up), and whoever adds the parts multiplies by what undoes it.
// The matrix cores cut what they add up, always downwards, and the gradients of hundreds of thousands of cells are added in the end: the factor's
// sign alternates over paths, tiles and steps, so that half of the parts are cut upwards.  (Error of g_w_hh and g_b against 64 bits over 0.4 M cells of 32 units: 9e-7 and
// 1.7e-6 with one sign, 2.9e-7 and 2.3e-7 so, 4.3e-7 and 2.7e-7 with fp32 instructions; the same where gradients go with the parity of the paths.)
// The tape of the next step is requested before the product, without conditions (1 to 4 % of training steps of 90 to 470 us).
__global__ __launch_bounds__(512, 4) void seq_reverse_narrow_kernel(SeqRevArgs A) {
    constexpr int HMAX = 32, NT = 4, RS = HMAX + 4, RJ = kSeqJobs;
    __shared__ __align__(16) float red[NT][RJ][RS];
    __shared__ __align__(16) int32_t sun[HMAX];            // the units' exponents
    __shared__ int32_t sdesc[RJ * 4];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hidden = A.hidden, n_tiles = hidden / 8, tile = wave & 3, group = wave >> 2;
    const bool on = tile < n_tiles;
    seq_h8_t wt[2][2];                                     // [step][piece]
#pragma unroll
    for (int k = 0; k < 4; ++k)
        wt[k >> 1][k & 1] = on ? reinterpret_cast<const seq_h8_t *>(A.wqt)[((size_t)tile * 4 + k) * 64 + (threadIdx.x & 63)] : seq_h8_t{};
    if ((int)threadIdx.x < hidden) sun[threadIdx.x] = A.wqt_unscale[threadIdx.x];   // (read behind the barriers of a tile)
    for (int64_t ci = blockIdx.x; ci < A.n_path_tiles; ci += gridDim.x) {
        const int64_t ct = A.reversed ? A.n_path_tiles - 1 - ci : ci;
        {
            const int tid = seq_opaque(threadIdx.x);
            if (tid < RJ * 4) sdesc[tid] = A.paths[ct * (RJ * 4) + tid];
        }
        __syncthreads();
        const int steps = __builtin_amdgcn_readfirstlane(sdesc[2]);
        float dh[4] = {0.f, 0.f, 0.f, 0.f}, dc[4] = {0.f, 0.f, 0.f, 0.f};
        float gates[16];                                   // requested a step ahead, in pieces (see seq_to_pieces)
        float4 c_now = make_float4(0.f, 0.f, 0.f, 0.f), c_prev;   // c_prev is the next step's c_now
        int keep;
        // The tape of step t.  No load hangs on a condition, or the compiler waits for each before the next: a path without such a step reads its first cell, and
        // c before a first step from the zero state is cleared where it is used.
        auto load_step = [&](int t) {
            const int l = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (l >> 5) * 4;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int jj = group * 32 + 16 * q + (l & 15);
                const float *p = A.tape_g + ((size_t)(sdesc[jj * 4 + 1] + (t >= 0 && t < sdesc[jj * 4 + 2] ? t : 0)) * hidden + tile * 8 + seq_piece(l)) * 4;
                const float4 v = *reinterpret_cast<const float4 *>(p), w = *reinterpret_cast<const float4 *>(p + 16);
                gates[8 * q] = v.x; gates[8 * q + 1] = v.y; gates[8 * q + 2] = v.z; gates[8 * q + 3] = v.w;
                gates[8 * q + 4] = w.x; gates[8 * q + 5] = w.y; gates[8 * q + 6] = w.z; gates[8 * q + 7] = w.w;
            }
            const int j = group * 32 + (l & 31), start = sdesc[j * 4], beg = sdesc[j * 4 + 1], len = sdesc[j * 4 + 2];
            const bool inner = t > 0 && t < len, from_state = t == 0 && len > 0 && start >= 0;
            keep = A.step_out[beg + (t >= 0 && t < len ? t : 0)];
            c_prev = *reinterpret_cast<const float4 *>((from_state ? A.c_state : A.tape_c) + (size_t)(from_state ? start : inner ? beg + t - 1 : beg) * hidden + unit0);
        };
        auto sum_parts = [&](int j) {
            const int unit0 = tile * 8 + ((seq_opaque(threadIdx.x) >> 5) & 1) * 4;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int w = 0; w < NT; ++w) {
                const int from = w < n_tiles ? w : 0;      // (no branch, so that the reads go out together; what is not finite in tile 0 makes the sum so anyway)
                const float4 q = *reinterpret_cast<const float4 *>(&red[from][j][unit0]);
                const float by = w < n_tiles ? red[from][j][HMAX] : 0.f;
                v.x = fmaf(q.x, by, v.x); v.y = fmaf(q.y, by, v.y); v.z = fmaf(q.z, by, v.z); v.w = fmaf(q.w, by, v.w);
            }
            const int4 un4 = *reinterpret_cast<const int4 *>(&sun[unit0]);
            dh[0] = __builtin_ldexpf(v.x, un4.x); dh[1] = __builtin_ldexpf(v.y, un4.y); dh[2] = __builtin_ldexpf(v.z, un4.z); dh[3] = __builtin_ldexpf(v.w, un4.w);
        };
        if (on) {
            const int lane = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (lane >> 5) * 4;
            const int j = group * 32 + (lane & 31), len = sdesc[j * 4 + 2], node = sdesc[j * 4 + 3];
            if (node >= 0) {
                const float4 v = *reinterpret_cast<const float4 *>(A.g_a + (size_t)node * hidden + unit0);
                dh[0] = v.x; dh[1] = v.y; dh[2] = v.z; dh[3] = v.w;
            }
            if (len > 0) c_now = *reinterpret_cast<const float4 *>(A.tape_c + ((size_t)sdesc[j * 4 + 1] + len - 1) * hidden + unit0);
            load_step(steps - 1);
            for (int t = steps - 1; t >= 0; --t) {
                const int lane = seq_opaque(threadIdx.x) & 63, half = lane >> 5, unit0 = tile * 8 + half * 4;
                const int j = group * 32 + (lane & 31), len = sdesc[j * 4 + 2];
                float dg[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) dg[e] = 0.f;
                seq_from_pieces(gates);
                if (t == 0 && sdesc[j * 4] < 0) c_prev = make_float4(0.f, 0.f, 0.f, 0.f);
                if (t < len) {
                    if (t + 1 < len) sum_parts(j);         // dh_prev of the step before is this step's dh
                    if (keep >= 0) {                       // what the other users of this state sent back
                        if (A.pending) seq_wait_pending(A, keep);
                        const size_t o = (size_t)keep * hidden + unit0;
                        const float4 a = A.pending ? seq_ld4_device(A.gh + o) : *reinterpret_cast<const float4 *>(A.gh + o);
                        const float4 b = A.pending ? seq_ld4_device(A.gc + o) : *reinterpret_cast<const float4 *>(A.gc + o);
                        dh[0] += a.x; dh[1] += a.y; dh[2] += a.z; dh[3] += a.w;
                        dc[0] += b.x; dc[1] += b.y; dc[2] += b.z; dc[3] += b.w;
                    }
                    const float cn[4] = {c_now.x, c_now.y, c_now.z, c_now.w}, cp[4] = {c_prev.x, c_prev.y, c_prev.z, c_prev.w};
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const float4 g4 = make_float4(gates[4 * m], gates[4 * m + 1], gates[4 * m + 2], gates[4 * m + 3]);   // i, f, g, o
                        const float tc = seq_tanh(cn[m]);
                        const float d_o = dh[m] * tc;
                        const float dcc = dc[m] + dh[m] * g4.w * (1.f - tc * tc);
                        dg[4 * m] = dcc * g4.z * g4.x * (1.f - g4.x);
                        dg[4 * m + 1] = dcc * cp[m] * g4.y * (1.f - g4.y);
                        dg[4 * m + 2] = dcc * g4.x * (1.f - g4.z * g4.z);
                        dg[4 * m + 3] = d_o * g4.w * (1.f - g4.w);
                        dc[m] = dcc * g4.y;
                    }
                    c_now = c_prev;
                }
                load_step(t - 1);
                // dG replaces the gates on the tape
                float4 v[4];
                seq_to_pieces(dg, v);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int jj = group * 32 + 16 * q + (lane & 15);
                    if (t < sdesc[jj * 4 + 2]) {
                        float *p = A.tape_g + ((size_t)(sdesc[jj * 4 + 1] + t) * hidden + tile * 8 + seq_piece(lane)) * 4;
                        *reinterpret_cast<float4 *>(p) = v[2 * q];
                        *reinterpret_cast<float4 *>(p + 16) = v[2 * q + 1];
                    }
                }
                __syncthreads();                           // every lane has read the parts of the step before
                float most = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) most = fmaxf(most, fabsf(dg[e]));
                const seq_u2_t both = __builtin_amdgcn_permlane32_swap(__float_as_uint(most), __float_as_uint(most), false, false);
                const int up = seq_up(fmaxf(__uint_as_float(both.x), __uint_as_float(both.y)));   // of the path's 32 gate rows
                const float one = (tile + j + t) & 1 ? -1.f : 1.f, by = __builtin_ldexpf(one, up);
                if (half == 0) red[tile][j][HMAX] = __builtin_ldexpf(one, -kSeqBack - up);
                seq_h8_t zb[2][2];                         // [step][piece]
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    uint32_t p[4][2];
#pragma unroll
                    for (int i = 0; i < 4; ++i) seq_halves2_low(dg[8 * k + 2 * i] * by, dg[8 * k + 2 * i + 1] * by, p[i]);
#pragma unroll
                    for (int i = 0; i < 2; ++i) zb[k][i] = __builtin_bit_cast(seq_h8_t, make_uint4(p[0][i], p[1][i], p[2][i], p[3][i]));
                }
                seq_acc_t acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wt[k][1], zb[k][0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wt[k][0], zb[k][1], acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] *= 1.f / kSeqLow;
#pragma unroll
                for (int k = 0; k < 2; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wt[k][0], zb[k][0], acc, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(&red[tile][j][8 * q + 4 * half]) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
                __syncthreads();                           // the parts of dh_prev are complete
            }
        } else {                                           // wavefronts beyond the hidden size only keep the barriers
            for (int t = steps - 1; t >= 0; --t) {
                __syncthreads();
                __syncthreads();
            }
        }
        // What is left: the gradient of the state the path started from, as rows in LDS first, so that one atomic instruction
        // covers a row of 256 contiguous bytes (issued by the lanes that hold the values, four bytes of each of 64 rows per
        // instruction, they took most of the kernel's time: the memory side does about 17 such requests per ns).
        if (__any(sdesc[(seq_opaque(threadIdx.x) & 63) * 4] >= 0)) {   // (the same for every wavefront)
            const int lane = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (lane >> 5) * 4, own = group * 32 + (lane & 31);
            if (on) sum_parts(own);
            __syncthreads();
            if (on) {
                *reinterpret_cast<float4 *>(&red[0][own][unit0]) = make_float4(dh[0], dh[1], dh[2], dh[3]);
                *reinterpret_cast<float4 *>(&red[1][own][unit0]) = make_float4(dc[0], dc[1], dc[2], dc[3]);
            }
            __syncthreads();
            for (int j = wave; j < RJ; j += 8) {
                const int start = sdesc[j * 4];
                if (start < 0) continue;                   // (the same for the whole wavefront; an empty path starts nowhere)
                if (lane < hidden) {
                    __hip_atomic_fetch_add(A.gh + (size_t)start * hidden + lane, red[0][j][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_add(A.gc + (size_t)start * hidden + lane, red[1][j][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (A.pending) {
                // once the wavefront has seen its atomics complete, its paths are counted off
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                const int start = lane < RJ / 8 ? sdesc[(wave + 8 * lane) * 4] : -1;
                if (start >= 0 && A.publish) __hip_atomic_fetch_sub(A.pending + start, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
    }
}

// Hidden sizes from 40 to 64: the products and their operands of the kernel above, 32 paths per workgroup, and the gates computed again instead of
// read from the tape.
// Sixteen wavefronts in two roles, because one wavefront's registers do not hold both W_hh and W_hh^T, and weights streamed from the cache between the tape's
// loads would wait for those (loads return in order: a quarter slower):
//   wavefronts 8..15 run ahead: they load h and c of the tape and the rows of gx, multiply W_hh with h in the forward pass's pieces and leave the gates of the
//     next step in LDS, and c of this one; they are the only ones that wait for loads.  (The sum begins at zero and gx joins it last, where the forward pass begins with gx: the
//     gates differ by a rounding from those that made c.);
//   wavefronts 0..7 go back through the steps, wavefront w for gate tile w, out of LDS, and write dG.
// A step has two barriers, and the loads of a step are requested two steps ahead, across half tiles too.  What bounds it: reads out of LDS, vector instructions (61 % of the time),
// products (16 %) and barriers, one after the other; 3.2 TB/s.
// Why from 40 to 64: training steps with the gates on the tape and so, us: 370 k nodes, prefix HAG, 64 units 4600 and 4030; 74 k nodes in lists of 16, prefix HAG, 1302 and 1115
// (40 units), 1654 and 1480 (64); 50 k nodes in lists of up to 8, 438 and 394, 566 and 525; 2 k nodes 148 and 143, 186 and 177; only lists of one and two entries lose, 514 and 547,
// 744 and 775 (200 k nodes), too little to keep both forms.  Up to 32 units the products and the lockstep take longer than the gates' bytes (steps of 90 to 290 us: 4 %
// slower), and above 64 the two forms of the weights fit no wavefronts' registers.
__global__ __launch_bounds__(1024, 4) void seq_reverse_kernel(SeqRevArgs A) {
    constexpr int HMAX = 64, MT = 2, NT = 8, RS = HMAX + 4, RJ = kSeqRevJobs, KS = 4, ZS = HMAX + 8;
    constexpr int PT = 512 / RJ;                           // threads that stage the h and c of one path, four columns each
    __shared__ __align__(16) float red[NT][RJ][RS], sfac[RJ][NT + 4];   // the parts of dh_prev, and what each is multiplied by
    __shared__ __align__(16) uint16_t z[2][2][RJ][ZS];     // the h that a step began with, in fp16 pieces: of the next step and of the one after it
    __shared__ __align__(16) float cs[2][RJ][RS];          // the c that a step began with: of this step and of the next one
    __shared__ float4 gates[8][4][64];                     // of the next step, as the lanes hold them
    __shared__ int32_t skeep[2][RJ];                       // the state row that a step wrote, or -1
    __shared__ __align__(16) int32_t sun[HMAX];            // the units' exponents
    __shared__ float4 sby[HMAX];                           // the factors of the forward pass's pre-activations, per unit those of its gates
    __shared__ int32_t sdesc_of[2][4][RJ];                 // of a path: start state, first step, steps, node; of this half tile and of the next one
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), worker = wave & 7;
    const bool ahead = wave >= 8;
    const int hidden = A.hidden, n_tiles = hidden / 8, tile = worker;
    const bool on = tile < n_tiles;                        // (wavefronts beyond the hidden size only keep the barriers, and stage h)
    seq_h8_t wr[KS * 2];                                   // W_hh [step][piece], or W_hh^T [output tile][step][piece]
#pragma unroll
    for (int k = 0; k < KS * 2; ++k) {
        const seq_h8_t *from = ahead ? reinterpret_cast<const seq_h8_t *>(A.wq) + ((size_t)tile * KS * 2 + k) * 64
                                     : reinterpret_cast<const seq_h8_t *>(A.wqt) + ((size_t)tile * MT * 4 + k) * 64;
        wr[k] = on ? from[threadIdx.x & 63] : seq_h8_t{};
    }
    if ((int)threadIdx.x < hidden) { sun[threadIdx.x] = A.wqt_unscale[threadIdx.x]; sby[threadIdx.x] = reinterpret_cast<const float4 *>(A.unscale)[threadIdx.x]; }   // (read behind the barriers of a tile)
    for (int i = threadIdx.x; i < (int)(sizeof(z) / 4); i += 1024) reinterpret_cast<uint32_t *>(&z[0][0][0][0])[i] = 0;   // columns from `hidden` on stay zero
    if (threadIdx.x < RJ * (NT + 4)) (&sfac[0][0])[threadIdx.x] = 0.f;
    const int64_t n_parts = A.n_path_tiles * (kSeqJobs / RJ);
    const int32_t (*sdesc)[RJ] = sdesc_of[0];              // of this half tile
    // The words of half tile number i; past the end those of the last one (nothing uses what is loaded for them).
    auto word_of = [&](int64_t i, int w) {
        i = i < n_parts ? i : n_parts - 1;
        return A.paths[(A.reversed ? n_parts - 1 - i : i) * (RJ * 4) + w];
    };
    {
        const int tid = seq_opaque(threadIdx.x);
        if (tid < RJ * 4) sdesc_of[0][tid & 3][tid >> 2] = word_of(blockIdx.x, tid);
    }
    __syncthreads();
    // The two roles take the same half tiles and keep the same barriers: two before the first step, two per step, two after the last if a path of the half tile started from a state.
    auto hands_back = [&] { return __any(sdesc[0][seq_opaque(threadIdx.x) & 31] >= 0) != 0; };   // (the same for every wavefront)
    if (ahead) {
        // What the wavefronts that run ahead hold for their next steps.  Loads return in order and the compiler counts them, so none hangs on a condition: where a
        // path has no such step its first cell is read.
        float4 h_next, c_next;
        int row, keep_next;                                // row: of gx
        bool zero_next;
        auto load_row = [&](int t) {
            const int j = seq_opaque(threadIdx.x) & 31;
            row = A.step_g[sdesc[1][j] + (t >= 0 && t < sdesc[2][j] ? t : 0)];
        };
        auto load_begun = [&](int t) {                     // four columns of the h and c that step t of a path began with, and the state row that it wrote
            const int tid = seq_opaque(threadIdx.x) - 512, j = tid / PT, u = tid % PT * 4, start = sdesc[0][j], beg = sdesc[1][j], len = sdesc[2][j];
            const bool inner = t > 0 && t < len, first = t == 0 && len > 0 && start >= 0;
            const size_t at = (size_t)(inner ? beg + t - 1 : first ? start : beg) * hidden + (u < hidden ? u : 0);
            h_next = *reinterpret_cast<const float4 *>((first ? A.h_state : A.tape_h) + at);
            c_next = *reinterpret_cast<const float4 *>((first ? A.c_state : A.tape_c) + at);
            keep_next = A.step_out[beg + (t >= 0 && t < len ? t : 0)];
            zero_next = u >= hidden || !(inner || first);
        };
        int owed = -1;                                     // the start state of a path whose gradients this lane has still to count off
        auto count_off = [&] {                             // once the wavefront has seen its atomics complete
            if (!A.pending) return;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (owed >= 0 && A.publish) __hip_atomic_fetch_sub(A.pending + owed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            owed = -1;
        };
        float gx[16];                                      // in pieces (see seq_to_pieces)
        seq_acc_t pre;
        float4 c_held = make_float4(0.f, 0.f, 0.f, 0.f);
        int keep_held = -1;
        auto load_gx = [&] {                               // of the step whose row is at hand
            const seq_u2_t rows = __builtin_amdgcn_permlane16_swap((unsigned)row, (unsigned)row, false, false);   // of paths l % 16 and 16 + l % 16
            const int l = seq_opaque(threadIdx.x) & 63;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float *p = A.gx + ((size_t)(q ? rows.y : rows.x) * hidden + tile * 8 + seq_piece(l)) * 4;
                const float4 v = *reinterpret_cast<const float4 *>(p), w = *reinterpret_cast<const float4 *>(p + 16);
                gx[8 * q] = v.x; gx[8 * q + 1] = v.y; gx[8 * q + 2] = v.z; gx[8 * q + 3] = v.w;
                gx[8 * q + 4] = w.x; gx[8 * q + 5] = w.y; gx[8 * q + 6] = w.z; gx[8 * q + 7] = w.w;
            }
        };
        auto stage = [&](int t) {                          // h of step t, c of the step before (which is processed one step later than its gates are computed)
            const int tid = seq_opaque(threadIdx.x) - 512, j = tid / PT, u = tid % PT * 4;
            const float4 h = zero_next ? make_float4(0.f, 0.f, 0.f, 0.f) : h_next;
            uint32_t a[2], b[2];
            seq_halves2(h.x * kSeqHScale, h.y * kSeqHScale, a);
            seq_halves2(h.z * kSeqHScale, h.w * kSeqHScale, b);
#pragma unroll
            for (int p = 0; p < 2; ++p) *reinterpret_cast<uint2 *>(&z[t & 1][p][j][u]) = make_uint2(a[p], b[p]);   // (columns beyond `hidden`: zero)
            *reinterpret_cast<float4 *>(&cs[(t + 1) & 1][j][u]) = c_held;
            if (u == 0) skeep[(t + 1) & 1][j] = keep_held;
            c_held = zero_next ? make_float4(0.f, 0.f, 0.f, 0.f) : c_next;
            keep_held = keep_next;
        };
        auto product = [&](int t) {                        // the recurrent half of the gates
            const int l = seq_opaque(threadIdx.x) & 63;
#pragma unroll
            for (int r = 0; r < 16; ++r) pre[r] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                seq_h8_t zb[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) zb[p] = *reinterpret_cast<const seq_h8_t *>(&z[t & 1][p][l & 31][16 * s + 8 * (l >> 5)]);
                pre = __builtin_amdgcn_mfma_f32_32x32x16_f16(wr[2 * s + 1], zb[0], pre, 0, 0, 0);
                pre = __builtin_amdgcn_mfma_f32_32x32x16_f16(wr[2 * s], zb[1], pre, 0, 0, 0);
                pre = __builtin_amdgcn_mfma_f32_32x32x16_f16(wr[2 * s], zb[0], pre, 0, 0, 0);
            }
        };
        auto put_gates = [&] {
            const int l = seq_opaque(threadIdx.x) & 63;
            seq_from_pieces(gx);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const float4 by = sby[tile * 8 + (l >> 5) * 4 + m];
                gates[worker][m][l] = make_float4(seq_sigmoid(pre[4 * m] + gx[4 * m], by.x), seq_sigmoid(pre[4 * m + 1] + gx[4 * m + 1], by.y),
                                                  seq_tanh(pre[4 * m + 2] + gx[4 * m + 2], by.z), seq_sigmoid(pre[4 * m + 3] + gx[4 * m + 3], by.w));   // i, f, g, o
            }
        };
        load_row(sdesc[2][0] - 1);
        load_begun(sdesc[2][0] - 1);
        for (int64_t ci = blockIdx.x, nth = 0; ci < n_parts; ci += gridDim.x, ++nth) {
            sdesc = sdesc_of[nth & 1];
            const int steps = __builtin_amdgcn_readfirstlane(sdesc[2][0]);   // (none where a half of a tile holds nothing but padding)
            const int word = word_of(ci + gridDim.x, seq_opaque(threadIdx.x) & (RJ * 4 - 1));   // of the next half tile
            load_gx();
            load_row(steps - 2);
            stage(steps - 1);
            load_begun(steps - 2);
            __syncthreads();
            if (on) product(steps - 1);                    // (in the order of the loop, so that the counts of loads agree)
            stage(steps - 2);
            count_off();                                   // of the half tile before: a state that this one waits for may be among them
            {
                const int tid = seq_opaque(threadIdx.x) - 512;
                if (tid < RJ * 4) sdesc_of[~nth & 1][tid & 3][tid >> 2] = word;
            }
            load_begun(steps - 3);
            if (on) {
                put_gates();
                load_gx();
                load_row(steps - 3);
                __syncthreads();                           // the gates of the last step are complete, and the h rows of the one before
                for (int t = steps - 1; t >= 0; --t) {
                    product(t - 1);
                    stage(t - 2);
                    load_begun(t - 3);
                    __syncthreads();                       // the gates of step t have been read
                    put_gates();
                    load_gx();
                    load_row(t - 3);
                    __syncthreads();
                }
            } else {
                __syncthreads();
                for (int t = steps - 1; t >= 0; --t) {
                    stage(t - 2);
                    load_begun(t - 3);
                    __syncthreads();
                    __syncthreads();
                }
            }
            // (the next half tile's first loads go out before this one's last gradients)
            sdesc = sdesc_of[~nth & 1];
            load_row(sdesc[2][0] - 1);
            load_begun(sdesc[2][0] - 1);
            sdesc = sdesc_of[nth & 1];
            if (hands_back()) {
                // What is left: the gradient of the state the path started from, as rows in LDS first, so that one atomic instruction
                // covers a row of 256 contiguous bytes (issued by the lanes that hold the values, four bytes of each of 64 rows per
                // instruction, they took most of the kernel's time: the memory side does about 17 such requests per ns).  Counted off in the next
                // half tile, where this wavefront has waited for later loads anyway.
                const int lane = seq_opaque(threadIdx.x) & 63;
                __syncthreads();
                __syncthreads();
                for (int j = worker; j < RJ; j += 8) {
                    const int start = sdesc[0][j];
                    if (start < 0) continue;               // (the same for the whole wavefront; an empty path starts nowhere)
                    if (lane < hidden) {
                        __hip_atomic_fetch_add(A.gh + (size_t)start * hidden + lane, red[0][j][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_fetch_add(A.gc + (size_t)start * hidden + lane, red[1][j][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
                owed = lane < RJ / 8 ? sdesc[0][worker + 8 * lane] : -1;
            }
        }
        count_off();
    } else {
        for (int64_t ci = blockIdx.x, nth = 0; ci < n_parts; ci += gridDim.x, ++nth) {
            sdesc = sdesc_of[nth & 1];
            const int steps = __builtin_amdgcn_readfirstlane(sdesc[2][0]);   // (none where a half of a tile holds nothing but padding)
            float dh[4] = {0.f, 0.f, 0.f, 0.f}, dc[4] = {0.f, 0.f, 0.f, 0.f};
            auto sum_parts = [&](int j) {
                const int unit0 = tile * 8 + ((seq_opaque(threadIdx.x) >> 5) & 1) * 4;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                const float4 f0 = *reinterpret_cast<const float4 *>(&sfac[j][0]), f1 = *reinterpret_cast<const float4 *>(&sfac[j][4]);   // (zero of tiles that do not exist)
                const float by[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
#pragma unroll
                for (int w = 0; w < NT; ++w) {
                    const float4 q = *reinterpret_cast<const float4 *>(&red[w < n_tiles ? w : 0][j][unit0]);   // (no branch, so that the reads go out together; what is not finite in tile 0 makes the sum so anyway)
                    v.x = fmaf(q.x, by[w], v.x); v.y = fmaf(q.y, by[w], v.y); v.z = fmaf(q.z, by[w], v.z); v.w = fmaf(q.w, by[w], v.w);
                }
                const int4 un4 = *reinterpret_cast<const int4 *>(&sun[unit0]);
                dh[0] = __builtin_ldexpf(v.x, un4.x); dh[1] = __builtin_ldexpf(v.y, un4.y); dh[2] = __builtin_ldexpf(v.z, un4.z); dh[3] = __builtin_ldexpf(v.w, un4.w);
            };
            float4 c_now = make_float4(0.f, 0.f, 0.f, 0.f);
            if (on) {
                const int lane = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (lane >> 5) * 4;
                const int j = lane & 31, len = sdesc[2][j], node = sdesc[3][j];
                if (node >= 0) {
                    const float4 v = *reinterpret_cast<const float4 *>(A.g_a + (size_t)node * hidden + unit0);
                    dh[0] = v.x; dh[1] = v.y; dh[2] = v.z; dh[3] = v.w;
                }
                if (len > 0) c_now = *reinterpret_cast<const float4 *>(A.tape_c + ((size_t)sdesc[1][j] + len - 1) * hidden + unit0);
            }
            __syncthreads();
            __syncthreads();                               // the gates of the last step are complete
            // (waited for here, or the compiler waits for everything outstanding, the stores of dG too, in every step)
            asm volatile("" : "+v"(c_now.x), "+v"(c_now.y), "+v"(c_now.z), "+v"(c_now.w), "+v"(dh[0]), "+v"(dh[1]), "+v"(dh[2]), "+v"(dh[3]));
            for (int t = steps - 1; t >= 0; --t) {
                float dg[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) dg[e] = 0.f;
                if (on) {
                    const int lane = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (lane >> 5) * 4;
                    const int j = lane & 31, len = sdesc[2][j];
                    if (t < len) {
                        if (t + 1 < len) sum_parts(j);     // dh_prev of the step before is this step's dh
                        const int keep = skeep[t & 1][j];
                        if (keep >= 0) {                   // what the other users of this state sent back
                            if (A.pending) seq_wait_pending(A, keep);
                            const size_t o = (size_t)keep * hidden + unit0;
                            const float4 a = A.pending ? seq_ld4_device(A.gh + o) : *reinterpret_cast<const float4 *>(A.gh + o);
                            const float4 b = A.pending ? seq_ld4_device(A.gc + o) : *reinterpret_cast<const float4 *>(A.gc + o);
                            dh[0] += a.x; dh[1] += a.y; dh[2] += a.z; dh[3] += a.w;
                            dc[0] += b.x; dc[1] += b.y; dc[2] += b.z; dc[3] += b.w;
                        }
                        const float4 c_prev = *reinterpret_cast<const float4 *>(&cs[t & 1][j][unit0]);
                        const float cn[4] = {c_now.x, c_now.y, c_now.z, c_now.w}, cp[4] = {c_prev.x, c_prev.y, c_prev.z, c_prev.w};
#pragma unroll
                        for (int m = 0; m < 4; ++m) {
                            const float4 g4 = gates[worker][m][lane];   // i, f, g, o
                            const float tc = seq_tanh(cn[m]);
                            const float d_o = dh[m] * tc;
                            const float dcc = dc[m] + dh[m] * g4.w * (1.f - tc * tc);
                            dg[4 * m] = dcc * g4.z * g4.x * (1.f - g4.x);
                            dg[4 * m + 1] = dcc * cp[m] * g4.y * (1.f - g4.y);
                            dg[4 * m + 2] = dcc * g4.x * (1.f - g4.z * g4.z);
                            dg[4 * m + 3] = d_o * g4.w * (1.f - g4.w);
                            dc[m] = dcc * g4.y;
                        }
                        c_now = c_prev;
                    }
                    float4 v[4];
                    seq_to_pieces(dg, v);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int jj = 16 * q + (lane & 15);
                        if (t < sdesc[2][jj]) {
                            float *p = A.tape_g + ((size_t)(sdesc[1][jj] + t) * hidden + tile * 8 + seq_piece(lane)) * 4;
                            *reinterpret_cast<float4 *>(p) = v[2 * q];
                            *reinterpret_cast<float4 *>(p + 16) = v[2 * q + 1];
                        }
                    }
                }
                __syncthreads();                           // every lane has read the parts of the step before
                if (on) {
                    const int l = seq_opaque(threadIdx.x) & 63, half = l >> 5, j = (l & 31);
                    float most = 0.f;
#pragma unroll
                    for (int e = 0; e < 16; ++e) most = fmaxf(most, fabsf(dg[e]));
                    const seq_u2_t both = __builtin_amdgcn_permlane32_swap(__float_as_uint(most), __float_as_uint(most), false, false);
                    const int up = seq_up(fmaxf(__uint_as_float(both.x), __uint_as_float(both.y)));   // of the path's 32 gate rows
                    const float one = (tile + j + t) & 1 ? -1.f : 1.f, by = __builtin_ldexpf(one, up);
                    if (half == 0) sfac[j][tile] = __builtin_ldexpf(one, -kSeqBack - up);
                    seq_h8_t zb[2][2];                     // [step][piece]
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        uint32_t p[4][2];
#pragma unroll
                        for (int i = 0; i < 4; ++i) seq_halves2_low(dg[8 * k + 2 * i] * by, dg[8 * k + 2 * i + 1] * by, p[i]);
#pragma unroll
                        for (int i = 0; i < 2; ++i) zb[k][i] = __builtin_bit_cast(seq_h8_t, make_uint4(p[0][i], p[1][i], p[2][i], p[3][i]));
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        seq_acc_t acc;
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wr[(mt * 2 + k) * 2 + 1], zb[k][0], acc, 0, 0, 0);
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wr[(mt * 2 + k) * 2], zb[k][1], acc, 0, 0, 0);
                        }
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] *= 1.f / kSeqLow;
#pragma unroll
                        for (int k = 0; k < 2; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wr[(mt * 2 + k) * 2], zb[k][0], acc, 0, 0, 0);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<float4 *>(&red[tile][j][mt * 32 + 8 * q + 4 * half]) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
                    }
                }
                __syncthreads();                           // the parts of dh_prev and the gates of the next step are complete
            }
            if (hands_back()) {
                const int lane = seq_opaque(threadIdx.x) & 63, unit0 = tile * 8 + (lane >> 5) * 4, j = lane & 31;
                if (on) sum_parts(j);
                __syncthreads();
                if (on) {
                    *reinterpret_cast<float4 *>(&red[0][j][unit0]) = make_float4(dh[0], dh[1], dh[2], dh[3]);
                    *reinterpret_cast<float4 *>(&red[1][j][unit0]) = make_float4(dc[0], dc[1], dc[2], dc[3]);
                }
                __syncthreads();
            }
        }
    }
}

// Hidden sizes from 72 to 128.  A workgroup takes half a tile, 32 paths: dG is staged as rows of 4 * 128 + 8 pieces in LDS (66 KB), so that two workgroups share
// a compute unit and one's loads, stores and element-wise part run beside the other's products (a third faster than 64 paths and 131 KB).
// Sixteen threads per path run the element-wise part; every wavefront multiplies one 32-unit tile of W_hh^T, streamed from the L2 cache, with one half
// of the gate rows, and the two parts are added by whoever reads dh_prev.  Operands in two fp16 pieces as in the kernels above, a path's gradients with one factor
// for all gate rows.  No load hangs on a condition (it would be waited for before the next), and the weights come four steps ahead of the products.
// 0.85 M cells of 128 units: 0.95 ms (4.5 TB/s; vector instructions 42 % of the time, matrix cores 19 %); 1.77 with fp32 products, 1.27 with fp16 pieces and loads that waited for
// one another.  Error of the training step's results against 64 bits 5.1e-7 (fp32 products 6.7e-7).
__global__ __launch_bounds__(512, 4) void seq_reverse_wide_kernel(SeqRevArgs A) {
    constexpr int ZS = 4 * 128 + 8, IT = 8, TP = 16;       // units per thread, threads per path; rows 4 banks apart
    // per path: the pre-activation gradients of the current step in fp16 pieces (the product's operand), then, in the row of the first pieces, the two parts
    // of the product's result dh_prev; the running dh and dc themselves stay in the registers of the path's sixteen threads
    __shared__ __align__(16) uint16_t z[2][kSeqRevJobs][ZS];
    __shared__ int32_t sun[128];                           // the units' exponents
    auto row_of = [&](int j) { return reinterpret_cast<float *>(&z[0][j][0]); };   // 256 floats (and four of padding)
    __shared__ int32_t sdesc[kSeqRevJobs * 4];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hidden = A.hidden, n_rt = (hidden + 31) / 32;          // 3 or 4 row tiles of the product
    // element-wise phases: 16 threads per path, all in one wavefront (their places are derived again in every phase: registers are short)
    const int64_t n_halves = A.n_path_tiles * (kSeqJobs / kSeqRevJobs);
    if ((int)threadIdx.x < hidden) sun[threadIdx.x] = A.wqt_unscale[threadIdx.x];   // (read behind the barriers of a tile)
    for (int64_t ci = blockIdx.x; ci < n_halves; ci += gridDim.x) {
        const int64_t ct = A.reversed ? n_halves - 1 - ci : ci;
        {
            const int tid = seq_opaque(threadIdx.x);
            if (tid < kSeqRevJobs * 4) sdesc[tid] = A.paths[ct * (kSeqRevJobs * 4) + tid];
        }
        __syncthreads();
        const int steps = __builtin_amdgcn_readfirstlane(sdesc[2]);   // the first path is the longest
        // unit 16 * it + part: the sixteen threads of a path move 256 contiguous bytes of its gates per instruction
        float dcv[IT];
        float back = 1.f;                                  // with the unit's factor, what the product's result is multiplied by
        // the tape of a step is requested while the product of the one after it runs
        float4 gates[IT];
        float c_now[IT], c_prev[IT];                       // c_prev is the next step's c_now
        int keep = -1;
        // (no load hangs on a condition, or the compiler waits for each before the next: a path without a step t reads its first cell, a thread without a unit one
        // that it has; c before a first step from the zero state is cleared where it is used)
        auto load_step = [&](int t) {
            const int tid = seq_opaque(threadIdx.x), sj = tid / TP, part = tid % TP, start = sdesc[sj * 4], beg = sdesc[sj * 4 + 1], len = sdesc[sj * 4 + 2];
            const size_t cell = (size_t)beg + (t >= 0 && t < len ? t : 0);
            const bool inner = t > 0 && t < len, from_state = t == 0 && len > 0 && start >= 0;
            keep = A.step_out[cell];
            const float *g = A.tape_g + cell * hidden * 4, *before = (from_state ? A.c_state : A.tape_c) + (size_t)(from_state ? start : inner ? cell - 1 : cell) * hidden;
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int u = TP * it + part < hidden ? TP * it + part : part;
                gates[it] = *reinterpret_cast<const float4 *>(g + u * 4);
                c_prev[it] = before[u];
            }
        };
        {
            const int tid = seq_opaque(threadIdx.x), sj = tid / TP, part = tid % TP, beg = sdesc[sj * 4 + 1], len = sdesc[sj * 4 + 2], node = sdesc[sj * 4 + 3];
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int u = TP * it + part;
                // (dh lives in the path's row, as the sum of two parts, so that it takes no registers during the products)
                row_of(sj)[u] = node >= 0 && u < hidden ? A.g_a[(size_t)node * hidden + u] : 0.f;
                row_of(sj)[128 + u] = 0.f;
                dcv[it] = 0.f;
                c_now[it] = len > 0 && u < hidden ? A.tape_c[((size_t)beg + len - 1) * hidden + u] : 0.f;
            }
            load_step(steps - 1);
        }
        for (int t = steps - 1; t >= 0; --t) {
            const int tid = seq_opaque(threadIdx.x), sj = tid / TP, part = tid % TP, from = sdesc[sj * 4], len = sdesc[sj * 4 + 2];
            if (t < len) {
                const size_t cell = (size_t)sdesc[sj * 4 + 1] + t;
                if (A.pending && keep >= 0) seq_wait_pending(A, keep);
                // the product of the step before left the parts of dh_prev of this path in its row: this step's dh.  Only this path's own
                // lanes touch the row between the barriers, and they read all of it before any of them overwrites it below: one
                // wavefront, whose LDS accesses take effect in program order, and the fence keeps the compiler to that order.
                float dhv[IT];
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const int u = TP * it + part;
                    const float sum = row_of(sj)[u] + row_of(sj)[128 + u];
                    dhv[it] = t + 1 < len && u < hidden ? __builtin_ldexpf(sum * back, sun[u]) : sum;   // (before the first step: g_a as it is)
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (keep >= 0) {                           // what the other users of this state sent back
#pragma unroll
                    for (int it = 0; it < IT; ++it) {
                        const int u = TP * it + part;
                        if (u >= hidden) continue;
                        const float *h = A.gh + (size_t)keep * hidden + u, *c = A.gc + (size_t)keep * hidden + u;
                        dhv[it] += A.pending ? __hip_atomic_load(h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *h;
                        dcv[it] += A.pending ? __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *c;
                    }
                }
                float most = 0.f;
                float *out = A.tape_g + (cell * hidden + part) * 4;
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const float4 g4 = gates[it];           // i, f, g, o
                    if (t == 0 && from < 0) c_prev[it] = 0.f;
                    const float tc = seq_tanh(c_now[it]);
                    const float d_o = dhv[it] * tc;
                    const float dcc = dcv[it] + dhv[it] * g4.w * (1.f - tc * tc);
                    const float4 dg = make_float4(dcc * g4.z * g4.x * (1.f - g4.x), dcc * c_prev[it] * g4.y * (1.f - g4.y),
                                                  dcc * g4.x * (1.f - g4.z * g4.z), d_o * g4.w * (1.f - g4.w));
                    dcv[it] = dcc * g4.y;
                    c_now[it] = c_prev[it];
                    gates[it] = dg;
                    if (TP * it + part >= hidden) continue;
                    *reinterpret_cast<float4 *>(out + TP * it * 4) = dg;   // kept for the weight gradients
                    most = fmaxf(fmaxf(most, fmaxf(fabsf(dg.x), fabsf(dg.y))), fmaxf(fabsf(dg.z), fabsf(dg.w)));
                }
                __builtin_amdgcn_sched_barrier(0);         // (registers are short)
                most = seq_max16(most);                    // of the path's gate rows
                const int up = seq_up(most);
                const float one = (sj + t) & 1 ? -1.f : 1.f, by = __builtin_ldexpf(one, up);
                back = __builtin_ldexpf(one, -kSeqBack - up);
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const int u = TP * it + part;
                    if (u >= hidden) continue;
                    uint32_t a[2], b[2];
                    seq_halves2_low(gates[it].x * by, gates[it].y * by, a);
                    seq_halves2_low(gates[it].z * by, gates[it].w * by, b);
#pragma unroll
                    for (int p = 0; p < 2; ++p) *reinterpret_cast<uint2 *>(&z[p][sj][u * 4]) = make_uint2(a[p], b[p]);
                }
            }
            __syncthreads();
            // dh_prev^T [units, paths] = W_hh^T . dG^T [4H, paths], the gate rows in two halves
            const int lane = seq_opaque(threadIdx.x) & 63;
            seq_acc_t acc, low;                            // low: the products with a second piece, 2^11 times as large
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = low[r] = 0.f;
            const bool has_pair = wave < 2 * n_rt;
            const int rt = wave % n_rt, half = wave / n_rt;
            // The weights are requested four steps of sixteen gate rows ahead: a step is 96 cycles of products, an access of the L2 cache several hundred.
            constexpr int AHEAD = 4;
            seq_h8_t w[AHEAD][2];
            const int s0 = half * (hidden / 8), s1 = s0 + hidden / 8;   // (hidden is a multiple of 8, 72 at least)
            const seq_h8_t *wq = reinterpret_cast<const seq_h8_t *>(A.wqt) + (size_t)rt * (hidden / 4) * 2 * 64 + lane;
            auto load_w = [&](int i, int s) {
                s = s < s1 ? s : s1 - 1;
#pragma unroll
                for (int p = 0; p < 2; ++p) w[i][p] = wq[(s * 2 + p) * 64];
            };
            auto dg_piece = [&](int p, int s) { return *reinterpret_cast<const seq_h8_t *>(&z[p][lane & 31][16 * s + 8 * (lane >> 5)]); };
            auto step_low = [&](int i, int s, const seq_h8_t &z0) {
                low = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[i][1], z0, low, 0, 0, 0);
                low = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[i][0], dg_piece(1, s), low, 0, 0, 0);
            };
            int s = s0;
            if (has_pair) {
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) load_w(i, s + i);
#pragma unroll 1
                for (; s + AHEAD < s1; s += AHEAD) {
#pragma unroll
                    for (int i = 0; i < AHEAD; ++i) {
                        const seq_h8_t z0 = dg_piece(0, s + i);
                        step_low(i, s + i, z0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[i][0], z0, acc, 0, 0, 0);
                        load_w(i, s + AHEAD + i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // (one accumulator from here on, and below one piece of the weights: the tape needs the registers)
#pragma unroll
                for (int r = 0; r < 16; ++r) low[r] = fmaf(acc[r], kSeqLow, low[r]);
#pragma unroll
                for (int i = 0; i < AHEAD; ++i)
                    if (s + i < s1) step_low(i, s + i, dg_piece(0, s + i));
#pragma unroll
                for (int r = 0; r < 16; ++r) low[r] *= 1.f / kSeqLow;
            }
            // (loads return in order: requested before the weights, the tape would be waited for with them)
            load_step(t - 1);
            if (has_pair) {
#pragma unroll
                for (int i = 0; i < AHEAD; ++i)
                    if (s + i < s1) low = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[i][0], dg_piece(0, s + i), low, 0, 0, 0);
            }
            __syncthreads();                               // every product has read the staged gradients
            if (has_pair) {
                const int j = lane & 31;
                if (t < sdesc[j * 4 + 2]) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = rt * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
                        if (row < hidden) row_of(j)[128 * half + row] = low[r];
                    }
                }
            }
            __syncthreads();
        }
        // what is left: the gradient of the state the path started from, dh (in two parts) beside dc in the path's row, added by whole wavefronts so
        // that an atomic instruction covers contiguous bytes
        const int tid = seq_opaque(threadIdx.x), sj = tid / TP, part = tid % TP, lane = tid & 63;
        if (__any(sdesc[(lane & 31) * 4] >= 0)) {           // (the same for every wavefront)
#pragma unroll
            for (int it = 0; it < IT; ++it) reinterpret_cast<float *>(&z[1][sj][0])[TP * it + part] = dcv[it];
            if (part == 0) row_of(sj)[256] = back;
            __syncthreads();
            for (int j = wave; j < kSeqRevJobs; j += 8) {
                const int from = sdesc[j * 4];
                if (from < 0) continue;
                const float *dh = row_of(j), *dc = reinterpret_cast<const float *>(&z[1][j][0]);
                for (int u = lane; u < hidden; u += 64) {
                    __hip_atomic_fetch_add(A.gh + (size_t)from * hidden + u, __builtin_ldexpf((dh[u] + dh[128 + u]) * dh[256], sun[u]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_add(A.gc + (size_t)from * hidden + u, dc[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (A.pending) {
                // once the wavefront has seen its atomics complete, its paths are counted off
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                const int from = lane < kSeqRevJobs / 8 ? sdesc[(wave + 8 * lane) * 4] : -1;
                if (from >= 0 && A.publish) __hip_atomic_fetch_sub(A.pending + from, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
    }
}

// Weight gradients: a contraction over many rows on the matrix cores, dW [4H, columns] = sum over rows of dG[row] z[row]^T.  A
// workgroup of 4 wavefronts stages 32 rows at a time in LDS, wavefront w accumulates 64 rows of dW (gate tiles 2 w and 2 w + 1) against all
// column tiles; every workgroup ends with its own partial sums, which a second kernel adds up in a fixed order (so the weight
// gradients do not depend on timing).  blockIdx.y selects a slab of 256 rows of dW (hidden > 64 has two), blockIdx.z one of 32 NCT columns.
//
// The operands are cut into pieces once, by the thread that loads them: a thread takes one column of dG for all 32 rows, so its
// loads are contiguous over a wavefront, eight rows make one 16-byte operand of a 32x32x16 matrix instruction per piece, and the sums of dG over a
// node's rows run in its registers.  The matrix cores cut what they add to the size of the accumulator, always in the same direction, and a
// gradient adds hundreds of thousands of rows: the products of 32 rows therefore begin at zero and join the running sums in rounded additions.
//   Over the cells (SEG): two fp16 pieces (seq_halves2_low), three products.  h is bounded; the 32 numbers of a column of dG are brought into range by the power of two
//     that their largest asks for, with a sign that alternates over columns and chunks (so that half of the products are cut upwards), undone in the addition.  A chunk
//     with a run of rows whose largest h of a unit is below kSeqHLeast (an output gate that is all but closed), or with infinite gradients, takes fp32 products.
//   Over the nodes, whose features have no bound: three bf16 pieces, six products, the large ones apart from the small ones.  A chunk with numbers beyond bf16's
//     range, or with a run of rows whose largest is so small that last pieces would be lost, takes fp32 products of the numbers as they are (kSeqSplitMost, kSeqSplitLeast).
// 3.35 M cells of 64 units: 1.02 ms (4.4 TB/s; vector instructions 61 % of the time, matrix cores 17 %), with fp32 matrix instructions 1.41; 0.85 M cells of 128 units: 0.85 (3.3 TB/s,
// 62 and 24 %) and 1.33 ms.  Where every chunk takes fp32 products, training steps take 10 to 26 % longer (half of the units closed) and 1 to 4 % (a column of features of 1e-36).  Error of the training step's results against 64 bits 4e-7 (fp32 instructions 1.2e-6) and 5.1e-7 (6.7e-7).
//
// SEG: the rows are cells, taken in the order of the input row they read (`at`, ascending `seg`), z is h_prev, and while a row of dG is at hand
// it is also added to s[seg], the sum of dG over the cells that read one node: dG is read once for both.  A workgroup takes a
// contiguous range of rows; the part of a node that an earlier range began goes to edge_first, the part of one that a later range
// goes on with to edge_last, and seq_edges_kernel adds those up in order.
// Without SEG the rows are the nodes themselves: dG is s, z is x, and the column sums are the gradient of the bias.
struct SeqWgradArgs {
    const float *dg;         // [rows, 4H]
    const float *z, *z2;     // SEG: tape_h and h_state; else x, z2 unused
    const int32_t *at, *prev, *seg;   // SEG: cell, where its h_prev lives (>= 0: that tape row, -1: zero, <= -2: state row -(value) - 2), node; else at = used
    int64_t rows, range;     // range: rows per workgroup, a multiple of the 32 staged at a time
    int32_t cols, hidden;    // columns of z
    float *partial;          // [gridDim.x][4H * 32 * column tiles + 4H]
    float *s, *edge_first, *edge_last;   // SEG: [nodes, 4H], [gridDim.x, 4H] twice
};
constexpr int kSeqWgradRows = 32;
constexpr int kSeqWgradGroups = 512;        // workgroups at most, over all slabs of gate rows: two per compute unit
constexpr int64_t kSeqWgradPartialFloats = 64 << 20;   // and no more partial sums than this many floats

// element at a byte offset from a wave-uniform address in device memory; lane c's value of a 64-bit number, as a scalar
typedef float __attribute__((address_space(1))) *seq_global_t;
__device__ __forceinline__ seq_global_t seq_at(uint64_t row, uint32_t off) { return (seq_global_t)((char __attribute__((address_space(1))) *)row + off); }
__device__ __forceinline__ uint64_t seq_lane64(uint64_t v, int c) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, c) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), c) << 32;
}

// NCT: column tiles of 32 of a workgroup, rounded up to 1, 2 or 4; kp: columns of a row of the partial sums.
template <int NCT, bool SEG>
__global__ __launch_bounds__(256, 2) void seq_weight_grad_kernel(SeqWgradArgs A, int kp) {
    constexpr int CK = kSeqWgradRows, ZW = NCT * 32, CPT = CK * ZW / 256;   // CPT: rows of z per thread
    // eight rows (k) of a column per 16-byte slot, slot q of column c at q ^ (c / 4 % 4): eight neighbouring columns cover all banks
    constexpr int P = SEG ? 2 : 3;                         // pieces per operand: fp16 over the cells, bf16 over the nodes
    __shared__ uint4 sdg[P][256][CK / 8], sz[P][ZW][CK / 8];
    __shared__ __align__(16) float sback[SEG ? 256 : 4];   // SEG: what undoes the factors of a column of dG and of h
    __shared__ int32_t far_chunk;                          // the last chunk whose numbers the pieces do not hold
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows4 = 4 * A.hidden, cols = A.cols;
    const int row0 = blockIdx.y * 256, n_rt = (rows4 - row0 < 256 ? rows4 - row0 : 256) / 32;
    const int col0 = blockIdx.z * (NCT * 32), n_ct = (cols - col0 + 31) / 32;
    // Threads beyond the last gate row repeat it: they load, add and write what its own thread does, and no product reads their column.
    const uint32_t gate_off = (uint32_t)((row0 + tid < rows4 ? row0 + tid : rows4 - 1) - row0) * 4;
    // a thread takes column tid % ZW of z and rows CPT * (tid / ZW) on of the 32 (indices are derived again where they are used: registers are short)
    seq_acc_t acc[2][NCT];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int c = 0; c < NCT; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][c][r] = 0.f;
    float sum = 0.f;                                       // the running sum of dG[.][row0 + tid]
    const int64_t first = (int64_t)blockIdx.x * A.range, last = first + A.range < A.rows ? first + A.range : A.rows;
    bool begun_before = false;                             // SEG: the running sum belongs to a node that an earlier range began
    if (SEG && first > 0 && first < last) begun_before = A.seg[first - 1] == A.seg[first];
    // The next 32 rows are requested into registers before the products of the current ones, and their places a chunk before that.  Lane c works out where
    // row c lies and the wavefront reads it there as a scalar: as scalar arithmetic per row this took as long as the products.  Places past the end
    // are those of the last row, and what they hold is cleared before it is used; so is z where h_prev is the zero state (zero: the rows to clear).
    float rg[CK], rz[CPT];
    int32_t rs = -1, ig = 0, iz = 0;                       // of row lane % 32; rs: of row lane, one more than the chunk: where the last row's node ends
    uint32_t zero = 0;
    if (tid == 0) far_chunk = -1;
    __syncthreads();
    auto request_ids = [&](int64_t c0) {
        int64_t at = c0 + (seq_opaque(threadIdx.x) & (CK - 1));
        at = at < last ? at : last - 1;
        ig = SEG ? A.at[at] : (int32_t)at;
        iz = SEG ? A.prev[at] : A.at[at];
    };
    auto request = [&](int64_t c0) {
        const int tid = seq_opaque(threadIdx.x), lane = tid & 63, zc = tid % ZW, zq = tid / ZW;
        const uint64_t g_row = (uint64_t)(A.dg + row0) + (uint64_t)(uint32_t)ig * (uint32_t)(rows4 * 4);
        const bool state = SEG && iz <= -2;
        const uint64_t z_row = (uint64_t)(state ? A.z2 : A.z) + (uint64_t)(uint32_t)(state ? -iz - 2 : iz < 0 ? 0 : iz) * (uint32_t)(cols * 4);
        zero = (uint32_t)__ballot(iz == -1 || c0 + (lane & (CK - 1)) >= last);
        const uint32_t g_off = (uint32_t)seq_opaque((int)gate_off);
#pragma unroll
        for (int c = 0; c < CK; ++c) rg[c] = *seq_at(seq_lane64(g_row, c), g_off);
        const uint32_t z_off = (uint32_t)(col0 + zc < cols ? col0 + zc : cols - 1) * 4;   // (columns of padding read the row's last: no result reads them)
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            if constexpr (ZW >= 64) rz[c] = *seq_at(seq_lane64(z_row, wave * 64 / ZW * CPT + c), z_off);   // a wavefront has one run of rows
            else rz[c] = *seq_at((uint64_t)__shfl((unsigned long long)z_row, zq * CPT + c), z_off);
        }
        if (SEG) rs = lane <= CK && c0 + lane < A.rows ? A.seg[c0 + lane] : -1;
    };
    if (first < last) {
        request_ids(first);
        request(first);
        request_ids(first + CK);
    }
    for (int64_t c0 = first; c0 < last; c0 += CK) {
        const int here = last - c0 < CK ? (int)(last - c0) : CK;
        if (here < CK) {
#pragma unroll
            for (int c = 0; c < CK; ++c) rg[c] = c < here ? rg[c] : 0.f;
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            rz[c] = (zero >> ((seq_opaque(threadIdx.x) / ZW) * CPT + c)) & 1 ? 0.f : rz[c];
        const int tid = seq_opaque(threadIdx.x), zc = tid % ZW, zq = tid / ZW;
        float by = 1.f, most_g = 0.f, most_z = 0.f;
#pragma unroll
        for (int c = 0; c < CK; ++c) most_g = fmaxf(most_g, fabsf(rg[c]));
#pragma unroll
        for (int c = 0; c < CPT; ++c) most_z = fmaxf(most_z, fabsf(rz[c]));
        if constexpr (SEG) {
            const int up = seq_up(most_g);
            const float one = ((int)(c0 / CK) + tid) & 1 ? -1.f : 1.f;
            by = __builtin_ldexpf(one, up);
            sback[tid] = __builtin_ldexpf(one, -up) / kSeqHScale;
            if (!(most_g < INFINITY) || (most_z > 0.f && most_z < kSeqHLeast)) far_chunk = (int32_t)((c0 - first) / CK);
        } else if (fmaxf(most_g, most_z) > kSeqSplitMost || (most_g > 0.f && most_g < kSeqSplitLeast) || (most_z > 0.f && most_z < kSeqSplitLeast)) {
            far_chunk = (int32_t)((c0 - first) / CK);
        }
        auto cut = [&](float a, float b, float by, uint32_t (&p)[P]) {
            if constexpr (SEG) seq_halves2_low(a * by, b * by, p);
            else seq_split2(a, b, p);
        };
#pragma unroll
        for (int q = 0; q < CK / 8; ++q) {
            uint32_t w[P][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t p[P];
                cut(rg[8 * q + 2 * k], rg[8 * q + 2 * k + 1], by, p);
#pragma unroll
                for (int i = 0; i < P; ++i) w[i][k] = p[i];
            }
#pragma unroll
            for (int i = 0; i < P; ++i) sdg[i][tid][q ^ ((tid >> 2) & 3)] = make_uint4(w[i][0], w[i][1], w[i][2], w[i][3]);
        }
        {
            uint32_t w[P][CPT / 2];
#pragma unroll
            for (int k = 0; k < CPT / 2; ++k) {
                uint32_t p[P];
                cut(rz[2 * k], rz[2 * k + 1], kSeqHScale, p);
#pragma unroll
                for (int i = 0; i < P; ++i) w[i][k] = p[i];
            }
#pragma unroll
            for (int i = 0; i < P; ++i) {
                if constexpr (CPT >= 8) {
#pragma unroll
                    for (int q = 0; q < CPT / 8; ++q)
                        sz[i][zc][(zq * (CPT / 8) + q) ^ ((zc >> 2) & 3)] = make_uint4(w[i][4 * q], w[i][4 * q + 1], w[i][4 * q + 2], w[i][4 * q + 3]);
                } else {
                    reinterpret_cast<uint2 *>(&sz[i][zc][(zq / 2) ^ ((zc >> 2) & 3)])[zq & 1] = make_uint2(w[i][0], w[i][1]);
                }
            }
        }
        if (SEG) {
            // bit c: the node of row c ends there, or the range does
            const int lane = seq_opaque(threadIdx.x) & 63;
            const int32_t after = __shfl_down(rs, 1);
            const bool ends = lane < here && (rs != after || lane + 1 + c0 == last);
            const uint32_t stops = (uint32_t)__ballot(ends);
            const bool goes_on = c0 + here == last && __builtin_amdgcn_readlane(rs, here - 1) == __builtin_amdgcn_readlane(rs, here);   // the last row's node, beyond this range
            float *out = begun_before && stops && lane == __builtin_ctz(stops) ? A.edge_first + (size_t)blockIdx.x * rows4
                       : goes_on && lane == here - 1 ? A.edge_last + (size_t)blockIdx.x * rows4 : A.s + (size_t)(uint32_t)(rs < 0 ? 0 : rs) * (uint32_t)rows4;
            const uint64_t out_row = (uint64_t)(out + row0);
            if (stops) begun_before = false;
#pragma unroll
            for (int c = 0; c < CK; ++c) {
                sum += rg[c];
                if (!((stops >> c) & 1)) continue;
                *seq_at(seq_lane64(out_row, c), gate_off) = sum;
                sum = 0.f;
            }
        } else {
            // the rows of a chunk among themselves first: fewer roundings at the size of the running sum
            float part[CK / 2];
#pragma unroll
            for (int c = 0; c < CK / 2; ++c) part[c] = rg[c] + rg[c + CK / 2];
#pragma unroll
            for (int n = CK / 4; n > 0; n /= 2)
#pragma unroll
                for (int c = 0; c < n; ++c) part[c] += part[c + n];
            sum += part[0];
        }
        __syncthreads();
        const bool far = __builtin_amdgcn_readfirstlane(far_chunk) == (int32_t)((c0 - first) / CK);
        if (far) {                                         // the numbers as they are take the place of the pieces, row by row
            const int tid = seq_opaque(threadIdx.x), zc = tid % ZW, zq = tid / ZW;
#pragma unroll
            for (int c = 0; c < CK; ++c) reinterpret_cast<float *>(sdg)[c * 256 + tid] = rg[c];
#pragma unroll
            for (int c = 0; c < CPT; ++c) reinterpret_cast<float *>(sz)[(zq * CPT + c) * ZW + zc] = rz[c];
            __syncthreads();
            const int l32 = seq_opaque(threadIdx.x) & 31, half = (seq_opaque(threadIdx.x) >> 5) & 1;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int rt = 2 * wave + g;
                if (rt >= n_rt) continue;
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    seq_acc_t t;
#pragma unroll
                    for (int r = 0; r < 16; ++r) t[r] = 0.f;
#pragma unroll 1
                    for (int k = 0; k < CK; k += 2)
                        t = __builtin_amdgcn_mfma_f32_32x32x2f32(reinterpret_cast<const float *>(sdg)[(k + half) * 256 + rt * 32 + l32], reinterpret_cast<const float *>(sz)[(k + half) * ZW + ct * 32 + l32], t, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[g][ct][r] += t[r];
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (c0 + CK < last) {
            request(c0 + CK);
            request_ids(c0 + 2 * CK);
        }
        __builtin_amdgcn_sched_barrier(0);
        const int l32 = seq_opaque(threadIdx.x) & 31, half = (seq_opaque(threadIdx.x) >> 5) & 1;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int rt = 2 * wave + g;
            if (far || rt >= n_rt) continue;
            typedef typename std::conditional<SEG, seq_h8_t, seq_b8_t>::type piece_t;
            piece_t a[CK / 16][P];
#pragma unroll
            for (int k = 0; k < CK / 16; ++k)
#pragma unroll
                for (int p = 0; p < P; ++p) a[k][p] = *reinterpret_cast<const piece_t *>(&sdg[p][rt * 32 + l32][(2 * k + half) ^ ((l32 >> 2) & 3)]);
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                auto z_piece = [&](int k, int p) { return *reinterpret_cast<const piece_t *>(&sz[p][ct * 32 + l32][(2 * k + half) ^ ((l32 >> 2) & 3)]); };
                seq_acc_t t;
#pragma unroll
                for (int r = 0; r < 16; ++r) t[r] = 0.f;
                if constexpr (SEG) {
                    piece_t b[CK / 16];
#pragma unroll
                    for (int k = 0; k < CK / 16; ++k) {
                        b[k] = z_piece(k, 0);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[k][1], b[k], t, 0, 0, 0);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[k][0], z_piece(k, 1), t, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) t[r] *= 1.f / kSeqLow;
#pragma unroll
                    for (int k = 0; k < CK / 16; ++k) t = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[k][0], b[k], t, 0, 0, 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 back = *reinterpret_cast<const float4 *>(&sback[rt * 32 + 8 * q + 4 * half]);
                        acc[g][ct][4 * q] = fmaf(t[4 * q], back.x, acc[g][ct][4 * q]);
                        acc[g][ct][4 * q + 1] = fmaf(t[4 * q + 1], back.y, acc[g][ct][4 * q + 1]);
                        acc[g][ct][4 * q + 2] = fmaf(t[4 * q + 2], back.z, acc[g][ct][4 * q + 2]);
                        acc[g][ct][4 * q + 3] = fmaf(t[4 * q + 3], back.w, acc[g][ct][4 * q + 3]);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < CK / 16; ++k) {
                        const piece_t b0 = z_piece(k, 0), b1 = z_piece(k, 1), b2 = z_piece(k, 2);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k][2], b0, t, 0, 0, 0);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k][1], b0, t, 0, 0, 0);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k][1], b1, t, 0, 0, 0);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k][0], b1, t, 0, 0, 0);
                        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k][0], b2, t, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) { acc[g][ct][r] += t[r]; t[r] = 0.f; }
#pragma unroll
                    for (int k = 0; k < CK / 16; ++k) t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k][0], z_piece(k, 0), t, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[g][ct][r] += t[r];
                }
                if (NCT == 4) __builtin_amdgcn_sched_barrier(0);   // (one column tile at a time: registers are short)
            }
        }
        __syncthreads();
    }
    float *out = A.partial + (size_t)blockIdx.x * ((size_t)rows4 * kp + rows4);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int rt = 2 * wave + g;
        if (rt >= n_rt) continue;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            if (ct >= n_ct) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = row0 + rt * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
                out[(size_t)row * kp + col0 + ct * 32 + (lane & 31)] = acc[g][ct][r];
            }
        }
    }
    if (!SEG && blockIdx.z == 0 && row0 + tid < rows4) out[(size_t)rows4 * kp + row0 + tid] = sum;
}

// s of the nodes that several ranges share: the part of the range that begins the node, then those of the ranges that go on with
// it, in order.  One workgroup per range whose last node goes on.
__global__ __launch_bounds__(256) void seq_edges_kernel(const int32_t *__restrict__ seg, int64_t rows, int64_t range, const float *__restrict__ edge_first,
                                                       const float *__restrict__ edge_last, float *__restrict__ s, int rows4) {
    const int64_t first = (int64_t)blockIdx.x * range, last = first + range;
    if (last >= rows) return;                              // the last range: nothing goes on
    const int node = seg[last - 1];
    if (seg[last] != node || (first > 0 && seg[first - 1] == node)) return;   // ends here, or began before this range
    for (int k = threadIdx.x; k < rows4; k += 256) {
        float sum = edge_last[(size_t)blockIdx.x * rows4 + k];
        for (int64_t b = blockIdx.x + 1; b * range < rows && seg[b * range] == node; ++b) sum += edge_first[(size_t)b * rows4 + k];
        s[(size_t)node * rows4 + k] = sum;
    }
}

// adds the workgroups' partial sums in a fixed order (eight interleaved sums, then those) and writes gate-major rows; `g_b` is NULL where
// the column sums are not wanted.  32 outputs per workgroup, eight threads each; the first `split` workgroups serve one contraction, the others the other.
struct SeqReduceArgs { const float *partial; float *g_w, *g_b; int32_t groups, cols, kp; };
__global__ __launch_bounds__(256) void seq_weight_grad_reduce_kernel(SeqReduceArgs first, SeqReduceArgs second, unsigned split, int hidden) {
    __shared__ float part[8][32];
    const SeqReduceArgs A = blockIdx.x < split ? first : second;
    const int64_t per = (int64_t)4 * hidden * A.kp + 4 * hidden, wanted = A.g_b ? per : per - 4 * hidden;
    const int o = threadIdx.x & 31, p = threadIdx.x >> 5;
    const int64_t i = (int64_t)(blockIdx.x - (blockIdx.x < split ? 0 : split)) * 32 + o;
    const bool in_use = i < wanted && (i >= (int64_t)4 * hidden * A.kp || (int)(i % A.kp) < A.cols);   // (padding columns were never written)
    float sum = 0.f;
    if (in_use)
        for (int g = p; g < A.groups; g += 8) sum += A.partial[(size_t)g * per + i];
    part[p][o] = sum;
    __syncthreads();
    if (p != 0 || !in_use) return;
#pragma unroll
    for (int k = 1; k < 8; ++k) sum += part[k][o];
    if (i < (int64_t)4 * hidden * A.kp) {
        const int r = (int)(i / A.kp), k = (int)(i % A.kp);
        A.g_w[(size_t)((r & 3) * hidden + (r >> 2)) * A.cols + k] = sum;
    } else {
        const int r = (int)(i - (int64_t)4 * hidden * A.kp);
        A.g_b[(r & 3) * hidden + (r >> 2)] = sum;
    }
}

// g_x[used[i]] = W_ih^T s[i]: 64 nodes per workgroup, the gate rows in chunks of 128 through LDS, wavefront w taking column tiles w and w + 4.
__global__ __launch_bounds__(256) void seq_input_grad_kernel(const float *__restrict__ s, const int32_t *__restrict__ used, int64_t n_used,
                                                            const float *__restrict__ wxt, float *__restrict__ g_x, int d, int hidden) {
    constexpr int KC = 128, ZS = KC + 2;
    __shared__ __align__(16) float sh[64 * ZS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rows4 = 4 * hidden, n_dt = (d + 31) / 32;
    const int64_t blocks = (n_used + 63) / 64;
    for (int64_t bt = blockIdx.x; bt < blocks; bt += gridDim.x) {
        seq_acc_t acc[2][2];                               // [column tile][half of the nodes]
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][g][r] = 0.f;
        for (int k0 = 0; k0 < rows4; k0 += KC) {
            const int kc = rows4 - k0 < KC ? rows4 - k0 : KC;   // a multiple of 32
            __syncthreads();
            for (int i = threadIdx.x; i < 64 * (KC / 4); i += 256) {
                const int row = i / (KC / 4), k = (i % (KC / 4)) * 4;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (bt * 64 + row < n_used && k < kc) v = *reinterpret_cast<const float4 *>(s + (size_t)(bt * 64 + row) * rows4 + k0 + k);
                *reinterpret_cast<float2 *>(&sh[row * ZS + k]) = make_float2(v.x, v.y);
                *reinterpret_cast<float2 *>(&sh[row * ZS + k + 2]) = make_float2(v.z, v.w);
            }
            __syncthreads();
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int tile = wave + 4 * a;
                if (tile >= n_dt) continue;
                const float4 *wq = reinterpret_cast<const float4 *>(wxt) + ((size_t)tile * (rows4 / 8) + k0 / 8) * 64 + lane;
                const float *zl = &sh[(lane & 31) * ZS + (lane >> 5)];
                for (int q = 0; q < kc / 8; ++q) {
                    const float4 w = wq[q * 64];
                    const float w4[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int g = 0; g < 2; ++g)
                            acc[a][g] = __builtin_amdgcn_mfma_f32_32x32x2f32(zl[g * 32 * ZS + 2 * (4 * q + r)], w4[r], acc[a][g], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int col = (wave + 4 * a) * 32 + (lane & 31);
            if (col >= d) continue;
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t at = bt * 64 + g * 32 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4);
                    if (at < n_used) g_x[(size_t)used[at] * d + col] = acc[a][g][r];
                }
        }
        __syncthreads();
    }
}

// How a weight-gradient contraction cuts its columns: `tiles` column tiles of 32 per workgroup (1, 2 or 4: a template argument), `slabs` of them side by side
// along z, of which none begins beyond the last column.  Over the cells a workgroup takes all columns (128 at most); over the nodes, most often few beside the cells,
// slabs of 64 leave registers free and cost a read of s each.  Where there are as many nodes as cells (200 k nodes in lists of two that share none), training steps with
// three and four slabs take 0.86 (d = 160, hidden 40), 1.11 (160, 64) and 1.17 ms (196, 56), with all columns in one workgroup and fp32 products 1.04, 1.32 and 1.33.
struct SeqWgradSlabs { int64_t tiles, slabs; };
static constexpr SeqWgradSlabs seq_wgrad_slabs(int64_t cols, bool over_cells) {
    const int64_t ct = (cols + 31) / 32, most = over_cells ? 4 : 2, rounded = ct <= 1 ? 1 : ct <= 2 ? 2 : 4, tiles = rounded < most ? rounded : most;
    return {tiles, (ct + tiles - 1) / tiles};
}

// The two weight-gradient contractions: column tiles of a row of partial sums, floats of one workgroup's partial sums,
// workgroups along x and rows per workgroup (a multiple of the rows staged at a time).
struct SeqWgradShape { int nct; int64_t per, groups, range; };
static SeqWgradShape seq_wgrad_shape(int64_t rows, int64_t cols, int64_t hidden) {
    SeqWgradShape w;
    const int64_t ct = (cols + 31) / 32;
    w.nct = ct <= 1 ? 1 : ct <= 2 ? 2 : ct <= 4 ? 4 : 8;
    w.per = 4 * hidden * 32 * w.nct + 4 * hidden;
    const int64_t most = std::max<int64_t>(std::min<int64_t>(kSeqWgradGroups / ((4 * hidden + 255) / 256), kSeqWgradPartialFloats / w.per), 1);
    const int64_t chunks = (rows + kSeqWgradRows - 1) / kSeqWgradRows;
    const int64_t each = std::max<int64_t>((chunks + most - 1) / most, 1);
    w.range = each * kSeqWgradRows;
    w.groups = std::max<int64_t>((chunks + each - 1) / each, 1);
    return w;
}

template <bool SEG>
static int launch_wgrad(const SeqWgradArgs &g, const SeqWgradShape &w, int64_t hidden, hipStream_t s) {
    const SeqWgradSlabs z = seq_wgrad_slabs(g.cols, SEG);
    const dim3 grid((unsigned)w.groups, (unsigned)((4 * hidden + 255) / 256), (unsigned)z.slabs), block(256);
    const int kp = 32 * w.nct;
    if (z.tiles == 1) hipLaunchKernelGGL((seq_weight_grad_kernel<1, SEG>), grid, block, 0, s, g, kp);
    else if (z.tiles == 2) hipLaunchKernelGGL((seq_weight_grad_kernel<2, SEG>), grid, block, 0, s, g, kp);
    else if constexpr (SEG) hipLaunchKernelGGL((seq_weight_grad_kernel<4, true>), grid, block, 0, s, g, kp);
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

}  // namespace hag

using namespace hag;

extern "C" {

int hag_seq_search(int64_t n, const int64_t *rowptr, const int32_t *col, int64_t capacity, int64_t *n_merges, int32_t *left,
                   int32_t *right, int32_t *redundancy, int64_t *hrowptr, int32_t *hcol);

int hag_seq_create(int64_t n, const int64_t *rowptr, const int32_t *col, int64_t capacity, hag_seq_t **out) {
    if (!out) { set_error("out is NULL"); return HAG_EINVAL; }
    *out = nullptr;
    if (n < 0 || capacity < 0 || !rowptr) { set_error("n < 0, capacity < 0 or rowptr is NULL"); return HAG_EINVAL; }
    try {
        const int64_t e = rowptr[n];
        std::vector<int64_t> hrowptr(n + 1, 0);
        std::vector<int32_t> hcol((size_t)std::max<int64_t>(e, 1));
        const int64_t cap = std::min(capacity, e);
        std::vector<int32_t> left((size_t)std::max<int64_t>(cap, 1)), right(left.size()), red(left.size());
        int64_t a = 0;
        // capacity 0 still goes through the search: it validates the lists and copies them
        int rc = hag_seq_search(n, rowptr, col, cap, &a, left.data(), right.data(), red.data(), hrowptr.data(), hcol.data());
        if (rc) return rc;
        if (n + a + e + n >= (int64_t)INT32_MAX) { set_error("too many states for 32-bit ids"); return HAG_EINVAL; }
        auto *h = new hag_seq();
        h->n = n; h->e = e; h->n_merges = a;
        if (const char *v = getenv("HAG_SEQ_ONE_LAUNCH")) h->one_launch = atoi(v) != 0;
        if (const char *v = getenv("HAG_SPIN_LIMIT")) h->spin_limit = (int32_t)std::min<long long>(std::max<long long>(atoll(v), 1), INT32_MAX);
        const bool share = capacity > 0;
        // shared states: the one-element prefixes in use, then the aggregation nodes (a state's predecessor
        // has a smaller index)
        std::vector<int32_t> first_id(n, -1);
        int32_t n_first = 0;
        auto need_first = [&](int32_t u) { if (first_id[u] < 0) first_id[u] = n_first++; };
        if (share) {
            for (int64_t i = 0; i < a; ++i) if (left[i] < n) need_first(left[i]);
            for (int64_t v = 0; v < n; ++v)
                if (hrowptr[v + 1] > hrowptr[v] && hcol[hrowptr[v]] < n) need_first(hcol[hrowptr[v]]);
        }
        const int64_t S = (int64_t)n_first + a;
        h->n_states = S;
        auto state_of = [&](int32_t id) { return id < n ? first_id[id] : n_first + (id - (int32_t)n); };
        std::vector<int32_t> prev((size_t)S, -1), xrow((size_t)S, 0), depth((size_t)S, 1);
        for (int64_t u = 0; u < n; ++u) if (first_id[u] >= 0) xrow[first_id[u]] = (int32_t)u;
        for (int64_t i = 0; i < a; ++i) {
            const int32_t st = n_first + (int32_t)i;
            prev[st] = state_of(left[i]); xrow[st] = right[i]; depth[st] = depth[prev[st]] + 1;
        }
        // every node's private remainder: what follows the shared state of its list's head
        struct R { int32_t start, beg, len, node; };
        std::vector<R> rem;
        std::vector<int32_t> consumers((size_t)S, 0), tail((size_t)S, -1);   // tail: the longest remainder starting at the state
        std::vector<int64_t> weight((size_t)S, 1);
        std::vector<uint8_t> is_final((size_t)S, 0);
        h->final_state.assign(n, -1);
        for (int64_t v = 0; v < n; ++v) {
            const int64_t b0 = hrowptr[v], b1 = hrowptr[v + 1];
            if (b1 == b0) continue;
            if (!share) { rem.push_back(R{-1, (int32_t)b0, (int32_t)(b1 - b0), (int32_t)v}); h->final_state[v] = -2;
                          h->longest = std::max<int64_t>(h->longest, b1 - b0); continue; }
            const int32_t st = state_of(hcol[b0]);
            h->longest = std::max<int64_t>(h->longest, depth[st] + (b1 - b0 - 1));
            if (b1 - b0 == 1) { h->final_state[v] = st; is_final[st] = 1; continue; }
            h->final_state[v] = -2;
            ++consumers[st];
            weight[st] += b1 - b0 - 1;
            if (tail[st] < 0 || rem[tail[st]].len < (int32_t)(b1 - b0 - 1)) tail[st] = (int32_t)rem.size();
            rem.push_back(R{st, (int32_t)(b0 + 1), (int32_t)(b1 - b0 - 1), (int32_t)v});
        }
        for (int32_t f : h->final_state) { h->n_empty += f == -1; h->n_from_state += f >= 0; }
        // a state hands its running (h, c) to the successor with the most evaluations below it, or, with no
        // successor state, to its longest remainder
        std::vector<int32_t> cont((size_t)S, -1);
        for (int64_t st = S - 1; st >= 0; --st) {
            const int32_t p = prev[st];
            if (p < 0) continue;
            weight[p] += weight[st];
            ++consumers[p];
            if (cont[p] < 0 || weight[cont[p]] <= weight[st]) cont[p] = (int32_t)st;   // ties: the smaller index
        }
        std::vector<uint8_t> rem_used(rem.size(), 0);
        std::vector<int32_t> level((size_t)S, 0);
        struct P { int32_t start, head, len, node, level, rem; };   // head: first state (-1: a bare remainder `rem`)
        std::vector<P> ps;
        for (int64_t st = 0; st < S; ++st) {
            const int32_t p = prev[st];
            const bool is_head = p < 0 || cont[p] != st;
            level[st] = p < 0 ? 0 : (is_head ? level[p] + 1 : level[p]);
            if (!is_head) continue;
            int32_t len = 0, t = (int32_t)st, r = -1;
            for (;; t = cont[t]) { ++len; if (cont[t] < 0) break; }
            if (tail[t] >= 0) { r = tail[t]; rem_used[r] = 1; len += rem[r].len; }
            ps.push_back(P{p, (int32_t)st, len, r >= 0 ? rem[r].node : -1, level[st], r});
        }
        for (size_t r = 0; r < rem.size(); ++r)
            if (!rem_used[r]) ps.push_back(P{rem[r].start, -1, rem[r].len, rem[r].node, rem[r].start < 0 ? 0 : level[rem[r].start] + 1, (int32_t)r});
        std::stable_sort(ps.begin(), ps.end(), [](const P &p, const P &q) { return p.level != q.level ? p.level < q.level : p.len > q.len; });
        int32_t levels = 0;
        for (const P &p : ps) levels = std::max(levels, p.level + 1);
        h->level_ptr.assign((size_t)levels + 1, 0);
        h->paths.reserve(ps.size() * 4);
        for (const P &p : ps) {
            ++h->level_ptr[(size_t)p.level + 1];
            const int32_t beg = (int32_t)h->step_x.size();
            if (p.head >= 0) {
                for (int32_t t = p.head; t >= 0; t = cont[t]) {
                    // the continuation takes the state along; anything else that needs it reads it from memory
                    const bool handed_on = cont[t] >= 0 || (p.rem >= 0);
                    const bool kept = is_final[t] || consumers[t] > (handed_on ? 1 : 0);
                    h->step_x.push_back(xrow[t]);
                    h->step_out.push_back(kept ? t : -1);
                }
            }
            if (p.rem >= 0)
                for (int32_t k = 0; k < rem[p.rem].len; ++k) { h->step_x.push_back(hcol[rem[p.rem].beg + k]); h->step_out.push_back(-1); }
            h->paths.push_back(p.start); h->paths.push_back(beg); h->paths.push_back(p.len); h->paths.push_back(p.node);
        }
        for (int32_t l = 0; l < levels; ++l) h->level_ptr[(size_t)l + 1] += h->level_ptr[l];
        h->tile_ptr.assign((size_t)levels + 1, 0);
        for (int32_t l = 0; l < levels; ++l)
            h->tile_ptr[(size_t)l + 1] = h->tile_ptr[l] + (h->level_ptr[(size_t)l + 1] - h->level_ptr[l] + kSeqJobs - 1) / kSeqJobs;
        {
            const int64_t np = (int64_t)(h->paths.size() / 4);
            std::vector<int32_t> key((size_t)np), order((size_t)np);
            int32_t groups = 0;
            for (int64_t i = 0; i < np; ++i) {
                const int32_t start = h->paths[i * 4];
                key[i] = start < 0 ? 0 : depth[start];
                order[i] = (int32_t)i;
                groups = std::max(groups, key[i] + 1);
            }
            std::stable_sort(order.begin(), order.end(), [&](int32_t p, int32_t q) {
                return key[p] != key[q] ? key[p] < key[q] : h->paths[(size_t)p * 4 + 2] > h->paths[(size_t)q * 4 + 2];
            });
            h->depth_ptr.assign((size_t)groups + 1, 0);
            h->paths_by_depth.reserve(h->paths.size());
            for (int32_t i : order) {
                ++h->depth_ptr[(size_t)key[i] + 1];
                h->paths_by_depth.insert(h->paths_by_depth.end(), h->paths.begin() + (size_t)i * 4, h->paths.begin() + (size_t)i * 4 + 4);
            }
            h->depth_tile_ptr.assign((size_t)groups + 1, 0);
            for (int32_t g = 0; g < groups; ++g) {
                h->depth_tile_ptr[(size_t)g + 1] = h->depth_tile_ptr[g] + (h->depth_ptr[(size_t)g + 1] + kSeqJobs - 1) / kSeqJobs;
                h->depth_ptr[(size_t)g + 1] += h->depth_ptr[g];
            }
        }
        {
            const int64_t cells = (int64_t)h->step_x.size(), np = (int64_t)(h->paths.size() / 4);
            std::vector<int32_t> step_prev((size_t)cells, -1);
            h->pending_init.assign((size_t)std::max<int64_t>(h->n_states, 1), 0);
            for (int64_t i = 0; i < np; ++i) {
                const int32_t start = h->paths[i * 4], beg = h->paths[i * 4 + 1], len = h->paths[i * 4 + 2];
                if (start >= 0 && len > 0) ++h->pending_init[start];
                for (int32_t t = 0; t < len; ++t) step_prev[(size_t)beg + t] = t > 0 ? beg + t - 1 : (start >= 0 ? -start - 2 : -1);
            }
            std::vector<int32_t> xt_ptr((size_t)n + 1, 0);
            for (int64_t a2 = 0; a2 < cells; ++a2) ++xt_ptr[(size_t)h->step_x[a2] + 1];
            for (int64_t u = 0; u < n; ++u) xt_ptr[(size_t)u + 1] += xt_ptr[u];
            h->xt_idx.resize((size_t)cells);
            std::vector<int32_t> place((size_t)n, 0);
            for (int64_t u = 0; u < n; ++u)
                if (xt_ptr[(size_t)u + 1] > xt_ptr[u]) { place[u] = (int32_t)h->used.size(); h->used.push_back((int32_t)u); }
            h->step_g.resize((size_t)cells);
            for (int64_t a2 = 0; a2 < cells; ++a2) h->step_g[a2] = place[h->step_x[a2]];
            std::vector<int32_t> at(xt_ptr.begin(), xt_ptr.end() - 1);
            for (int64_t a2 = 0; a2 < cells; ++a2) h->xt_idx[(size_t)at[h->step_x[a2]]++] = (int32_t)a2;
            h->xt_prev.resize((size_t)cells);
            h->xt_seg.resize((size_t)cells);
            for (int64_t k = 0; k < cells; ++k) { h->xt_prev[k] = step_prev[h->xt_idx[k]]; h->xt_seg[k] = h->step_g[h->xt_idx[k]]; }
        }
        *out = h;
        return HAG_OK;
    } catch (const std::bad_alloc &) {
        set_error("out of host memory");
        return HAG_ENOMEM;
    } catch (const std::exception &ex) {
        set_error(ex.what());
        return HAG_EINVAL;
    }
}

void hag_seq_free(hag_seq_t *h) {
    if (!h) return;
    if (h->d_final) (void)hipFree(h->d_final);
    if (h->d_paths) (void)hipFree(h->d_paths);
    if (h->d_paths_by_depth) (void)hipFree(h->d_paths_by_depth);
    if (h->d_xt_prev) (void)hipFree(h->d_xt_prev);
    if (h->d_xt_seg) (void)hipFree(h->d_xt_seg);
    if (h->d_used) (void)hipFree(h->d_used);
    if (h->d_step_g) (void)hipFree(h->d_step_g);
    if (h->d_xt_idx) (void)hipFree(h->d_xt_idx);
    if (h->d_pending_init) (void)hipFree(h->d_pending_init);
    if (h->d_step_out) (void)hipFree(h->d_step_out);
    if (h->d_gave_up) (void)hipFree(h->d_gave_up);
    delete h;
}

int64_t hag_seq_cells(const hag_seq_t *h) { return h ? (int64_t)h->step_x.size() : 0; }
int64_t hag_seq_ranks(const hag_seq_t *h) { return h ? h->longest : 0; }
int64_t hag_seq_launches(const hag_seq_t *h) {
    if (!h) return 0;
    const int64_t levels = (int64_t)h->level_ptr.size() - 1;
    return h->one_launch ? std::min<int64_t>(levels, 1) : levels;
}
int64_t hag_seq_weight_grad_slabs(int64_t cols, int32_t over_cells, int64_t *slab_cols) {
    if (cols <= 0) return 0;
    const SeqWgradSlabs z = seq_wgrad_slabs(cols, over_cells != 0);
    if (slab_cols) *slab_cols = 32 * z.tiles;
    return z.slabs;
}
int64_t hag_seq_merges(const hag_seq_t *h) { return h ? h->n_merges : 0; }

// Forward kernel variants: hidden up to 32, 64, 128.
static int seq_variant(int64_t hidden) { return hidden <= 32 ? 0 : hidden <= 64 ? 1 : 2; }
typedef void (*seq_kernel_t)(SeqChainArgs);
static const seq_kernel_t kSeqVariants[3] = {seq_chain_kernel<32, false>, seq_chain_kernel<64, false>, seq_chain_kernel<128, false>};
// the same with the tape written (training)
static const seq_kernel_t kSeqTapeVariants[3] = {seq_chain_kernel<32, true>, seq_chain_kernel<64, true>, seq_chain_kernel<128, true>};
static unsigned seq_block(int variant) { return variant == 2 ? 1024 : 512; }
typedef void (*seq_reverse_t)(SeqRevArgs);
static const seq_reverse_t kSeqReverseVariants[3] = {seq_reverse_narrow_kernel, seq_reverse_kernel, seq_reverse_wide_kernel};
static unsigned seq_reverse_block(int variant) { return variant == 1 ? 1024 : 512; }

int hag_seq_get_plan(const hag_seq_t *h, int32_t order, int64_t *n_states, int64_t *n_paths, const int32_t **paths,
                     const int32_t **step_x, const int32_t **step_out, int64_t *n_levels, const int64_t **level_ptr,
                     const int32_t **final_state) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    if (order != 0 && order != 1) { set_error("order must be 0 (levels) or 1 (depth of the start state)"); return HAG_EINVAL; }
    if (n_states) *n_states = h->n_states;
    if (n_paths) *n_paths = (int64_t)(h->paths.size() / 4);
    if (paths) *paths = order ? h->paths_by_depth.data() : h->paths.data();
    if (step_x) *step_x = h->step_x.data();
    if (step_out) *step_out = h->step_out.data();
    if (n_levels) *n_levels = (int64_t)(order ? h->depth_ptr.size() : h->level_ptr.size()) - 1;
    if (level_ptr) *level_ptr = order ? h->depth_ptr.data() : h->level_ptr.data();
    if (final_state) *final_state = h->final_state.data();
    return HAG_OK;
}

int hag_seq_upload(hag_seq_t *h) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    if (h->d_final) return HAG_OK;
    HIP_TRY(hipGetDevice(&h->device));
    auto put = [](int32_t **dst, const std::vector<int32_t> &src) -> hipError_t {
        hipError_t e = hipMalloc(dst, std::max<size_t>(src.size(), 1) * sizeof(int32_t));
        if (e == hipSuccess && !src.empty()) e = hipMemcpy(*dst, src.data(), src.size() * sizeof(int32_t), hipMemcpyHostToDevice);
        return e;
    };
    {
        // every group padded to whole tiles with empty paths (no start state, no steps, no node)
        auto padded = [](const std::vector<int32_t> &paths, const std::vector<int64_t> &ptr, const std::vector<int64_t> &tiles) {
            std::vector<int32_t> out;
            out.reserve((size_t)tiles.back() * kSeqJobs * 4);
            for (size_t l = 0; l + 1 < ptr.size(); ++l) {
                out.insert(out.end(), paths.begin() + ptr[l] * 4, paths.begin() + ptr[l + 1] * 4);
                while ((int64_t)out.size() < tiles[l + 1] * kSeqJobs * 4) { out.push_back(-1); out.push_back(0); out.push_back(0); out.push_back(-1); }
            }
            return out;
        };
        HIP_TRY(put(&h->d_paths, padded(h->paths, h->level_ptr, h->tile_ptr)));
        HIP_TRY(put(&h->d_paths_by_depth, padded(h->paths_by_depth, h->depth_ptr, h->depth_tile_ptr)));
    }
    HIP_TRY(put(&h->d_step_out, h->step_out));
    HIP_TRY(put(&h->d_xt_prev, h->xt_prev));
    HIP_TRY(put(&h->d_xt_seg, h->xt_seg));
    HIP_TRY(put(&h->d_used, h->used));
    HIP_TRY(put(&h->d_step_g, h->step_g));
    HIP_TRY(put(&h->d_xt_idx, h->xt_idx));
    HIP_TRY(put(&h->d_pending_init, h->pending_init));
    HIP_TRY(put(&h->d_gave_up, std::vector<int32_t>(1, 0)));
    {
        // workgroups of each kernel variant that the device holds at once (at most the two per compute unit the
        // kernel is tuned for): the grid of a one-launch pass
        int cus = 0;
        HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h->device));
        for (int k = 0; k < 3; ++k) {
            int per_cu = 0;
            HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kSeqVariants[k], (int)seq_block(k), 0));
            h->resident[k] = (int64_t)std::min(per_cu, 2) * cus;
            HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kSeqTapeVariants[k], (int)seq_block(k), 0));
            h->resident_tape[k] = (int64_t)std::min(per_cu, 2) * cus;
            HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kSeqReverseVariants[k], (int)seq_reverse_block(k), 0));
            h->resident_reverse[k] = (int64_t)std::min(per_cu, 2) * cus;
        }
    }
    HIP_TRY(put(&h->d_final, h->final_state));
    return HAG_OK;
}

int hag_seq_set_option(hag_seq_t *h, int32_t option, int64_t value) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    switch (option) {
        case HAG_OPT_SEQ_ONE_LAUNCH: h->one_launch = value != 0; return HAG_OK;
        case HAG_OPT_SPIN_LIMIT: h->spin_limit = (int32_t)std::min<int64_t>(std::max<int64_t>(value, 1), INT32_MAX); return HAG_OK;
        case HAG_OPT_TEST_WAIT_UNREACHABLE: h->wait_unreachable = value != 0; return HAG_OK;
        default: set_error("unknown option"); return HAG_EINVAL;
    }
}

int hag_seq_check(const hag_seq_t *h, void *stream) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    if (!h->d_final) { set_error("hag_seq_upload has not been called on this handle"); return HAG_ESTATE; }
    hipStream_t s = (hipStream_t)stream;
    int32_t word = 0;
    HIP_TRY(hipMemcpyAsync(&word, h->d_gave_up, sizeof(word), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (!word) return HAG_OK;
    HIP_TRY(hipMemsetAsync(h->d_gave_up, 0, sizeof(word), s));
    HIP_TRY(hipStreamSynchronize(s));
    set_error("a pass of the LSTM aggregator gave up waiting for a state: its output is not valid");
    return HAG_ETIMEOUT;
}

// Layout of the forward workspace, in bytes.
struct SeqLayout { int64_t dp, ks; size_t wx, wq, bp, h, c, flags, gx, total; };
static SeqLayout seq_layout(const hag_seq_t *h, int64_t d, int64_t hidden) {
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t states = (size_t)std::max<int64_t>(h->n_states, 1), H = (size_t)hidden, f = sizeof(float);
    SeqLayout L;
    L.dp = (d + 7) / 8 * 8;
    L.ks = hidden > 64 ? (hidden + 15) / 16 : hidden > 32 ? 4 : 2;
    size_t at = 0;
    L.wx = at; at += up(4 * H * (size_t)L.dp * f);
    L.wq = at; at += up((H / 8) * (size_t)L.ks * 2 * 512 * sizeof(uint16_t));
    L.bp = at; at += up(12 * H * f);
    L.h = at; at += up(states * H * f);
    L.c = at; at += up(states * H * f);
    L.flags = at; at += up(states * sizeof(int32_t));
    L.gx = at; at += up(h->used.size() * 4 * H * f);
    L.total = at;
    return L;
}
size_t hag_seq_workspace_bytes(const hag_seq_t *h, int64_t d, int64_t hidden) {
    if (!h || d <= 0 || hidden <= 0) return 0;
    return seq_layout(h, d, hidden).total;
}

static int seq_forward(const hag_seq_t *h, int64_t d, int64_t hidden, const float *x, const float *w_ih, const float *w_hh,
                       const float *b, float *a_out, void *workspace, void *stream, float *tape_g, float *tape_c, float *tape_h) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    if (!h->d_final) { set_error("hag_seq_upload has not been called on this handle"); return HAG_ESTATE; }
    if (d <= 0 || d % 4 != 0 || hidden <= 0 || hidden % 8 != 0 || hidden > 128 || d + hidden > kSeqMaxK) {
        set_error("d must be a multiple of 4, hidden a multiple of 8 up to 128, d + hidden at most 256");
        return HAG_EINVAL;
    }
    if (h->n == 0) return HAG_OK;
    if (!x || !w_ih || !w_hh || !b || !a_out || !workspace) { set_error("NULL pointer"); return HAG_EINVAL; }
    if (((uintptr_t)x | (uintptr_t)workspace | (uintptr_t)a_out) & 15) { set_error("x, a_out and workspace must be 16-byte aligned"); return HAG_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    const SeqLayout L = seq_layout(h, d, hidden);
    char *w = (char *)workspace;
    float *wx = (float *)(w + L.wx), *bp = (float *)(w + L.bp), *hst = (float *)(w + L.h), *cst = (float *)(w + L.c), *gx = (float *)(w + L.gx);
    uint16_t *wq = (uint16_t *)(w + L.wq);
    int32_t *flags = (int32_t *)(w + L.flags);              // [n_states]
    {
        const int64_t total = std::min<int64_t>(std::max(h->n_states, h->n_empty > 0 ? h->n : 0), 1 << 20);   // counters and nodes with an empty list
        hipLaunchKernelGGL(seq_pack_kernel, dim3((unsigned)std::max<int64_t>((total + 255) / 256, hidden)), dim3(256), 0, s, w_ih, w_hh, b, wx, wq, bp, (int)d,
                           (int)L.dp, (int)hidden, (int)L.ks, flags, h->n_states, h->n_empty > 0 ? h->d_final : nullptr, a_out, h->n);
        HIP_TRY(hipGetLastError());
    }
    if (const int64_t n_used = (int64_t)h->used.size(); n_used > 0) {
        hipLaunchKernelGGL(seq_input_gates_kernel, dim3((unsigned)std::min<int64_t>((n_used + 63) / 64, 1 << 20)), dim3(256),
                           (size_t)64 * (size_t)(L.dp + 2) * sizeof(float), s, x, h->d_used, n_used, wx, bp, gx, (int)d, (int)L.dp, (int)hidden);
        HIP_TRY(hipGetLastError());
    }
    const int64_t levels = (int64_t)h->tile_ptr.size() - 1;
    const int variant = seq_variant(hidden);
    const int64_t resident = tape_g ? h->resident_tape[variant] : h->resident[variant];
    const bool fused = levels > 1 && h->one_launch && resident > 0;
    for (int64_t l = 0; l < (fused ? 1 : levels); ++l) {
        SeqChainArgs c;
        const int64_t t0 = fused ? 0 : h->tile_ptr[l], t1 = fused ? h->depth_tile_ptr.back() : h->tile_ptr[l + 1];
        c.chains = fused ? h->d_paths_by_depth : h->d_paths + t0 * kSeqJobs * 4;
        c.n_path_tiles = t1 - t0;
        c.flags = fused ? flags : nullptr;
        c.spin_limit = h->spin_limit;
        c.publish = h->wait_unreachable ? 0 : 1;
        c.gave_up = h->d_gave_up;
        c.step_g = h->d_step_g; c.step_out = h->d_step_out;
        c.gx = gx; c.wq = wq; c.unscale = bp + 4 * hidden; c.h = hst; c.c = cst; c.a_out = a_out;
        c.tape_g = tape_g; c.tape_c = tape_c; c.tape_h = tape_h;
        c.hidden = (int32_t)hidden;
        if (c.n_path_tiles <= 0) continue;
        const dim3 grid((unsigned)std::min<int64_t>(c.n_path_tiles, fused ? resident : (variant == 2 ? 256 : 512))), block(seq_block(variant));
        hipLaunchKernelGGL(tape_g ? kSeqTapeVariants[variant] : kSeqVariants[variant], grid, block, 0, s, c);
        HIP_TRY(hipGetLastError());
    }
    if (h->n_from_state > 0) {
        hipLaunchKernelGGL(seq_output_kernel, dim3((unsigned)((h->n + 255) / 256)), dim3(256), 0, s, h->d_final, hst, a_out, h->n,
                           (int)hidden);
        HIP_TRY(hipGetLastError());
    }
    return HAG_OK;
}

int hag_seq_lstm_forward(const hag_seq_t *h, int64_t d, int64_t hidden, const float *x, const float *w_ih, const float *w_hh,
                         const float *b, float *a_out, void *workspace, void *stream) {
    return seq_forward(h, d, hidden, x, w_ih, w_hh, b, a_out, workspace, stream, nullptr, nullptr, nullptr);
}

// Layout of the training workspace: the forward workspace, then the tape and the backward pass's own buffers.
struct SeqTrainLayout { SeqWgradShape hh, ih; size_t fwd, tape_g, tape_c, tape_h, gh, gc, pending, wqt, unscale, wxt, s, edge_first, edge_last, partial_hh, partial_ih, total; };
static SeqTrainLayout seq_train_layout(const hag_seq_t *h, int64_t d, int64_t hidden) {
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t cells = std::max<size_t>(h->step_x.size(), 1), states = (size_t)std::max<int64_t>(h->n_states, 1);
    const size_t H = (size_t)hidden, f = sizeof(float), used = std::max<size_t>(h->used.size(), 1);
    SeqTrainLayout L;
    L.hh = seq_wgrad_shape((int64_t)h->step_x.size(), hidden, hidden);
    L.ih = seq_wgrad_shape((int64_t)h->used.size(), d, hidden);
    size_t at = up(hag_seq_workspace_bytes(h, d, hidden));
    L.fwd = 0;
    L.tape_g = at; at += up(cells * 4 * H * f);
    L.tape_c = at; at += up(cells * H * f);
    L.tape_h = at; at += up(cells * H * f);
    L.gh = at; at += up(states * H * f);
    L.gc = at; at += up(states * H * f);
    L.pending = at; at += up(states * sizeof(int32_t));
    L.wqt = at; at += up((H + 31) / 32 * 32 * 4 * H * f);
    L.unscale = at; at += up(H * f);
    L.wxt = at; at += up(((size_t)d + 31) / 32 * 32 * 4 * H * f);
    L.s = at; at += up(used * 4 * H * f);
    L.edge_first = at; at += up((size_t)L.hh.groups * 4 * H * f);
    L.edge_last = at; at += up((size_t)L.hh.groups * 4 * H * f);
    L.partial_hh = at; at += up((size_t)L.hh.groups * (size_t)L.hh.per * f);
    L.partial_ih = at; at += up((size_t)L.ih.groups * (size_t)L.ih.per * f);
    L.total = at;
    return L;
}
static bool seq_backward_supported(int64_t d, int64_t hidden) {
    return d > 0 && d % 4 == 0 && hidden > 0 && hidden % 8 == 0 && hidden <= 128 && d + hidden <= kSeqMaxK;
}

size_t hag_seq_train_workspace_bytes(const hag_seq_t *h, int64_t d, int64_t hidden) {
    if (!h || !seq_backward_supported(d, hidden)) return 0;
    return seq_train_layout(h, d, hidden).total;
}

int hag_seq_lstm_forward_train(const hag_seq_t *h, int64_t d, int64_t hidden, const float *x, const float *w_ih, const float *w_hh,
                               const float *b, float *a_out, void *workspace, void *stream) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    if (!seq_backward_supported(d, hidden)) {
        set_error("d must be a multiple of 4, hidden a multiple of 8 up to 128, d + hidden at most 256");
        return HAG_EINVAL;
    }
    if (!workspace) { set_error("NULL pointer"); return HAG_EINVAL; }
    const SeqTrainLayout L = seq_train_layout(h, d, hidden);
    char *w = (char *)workspace;
    return seq_forward(h, d, hidden, x, w_ih, w_hh, b, a_out, workspace, stream, (float *)(w + L.tape_g), (float *)(w + L.tape_c),
                       (float *)(w + L.tape_h));
}

int hag_seq_lstm_backward(const hag_seq_t *h, int64_t d, int64_t hidden, const float *x, const float *w_ih, const float *w_hh,
                          const float *g_a, float *g_x, float *g_w_ih, float *g_w_hh, float *g_b, void *workspace, void *stream) {
    if (!h) { set_error("NULL handle"); return HAG_EINVAL; }
    if (!h->d_final) { set_error("hag_seq_upload has not been called on this handle"); return HAG_ESTATE; }
    if (!seq_backward_supported(d, hidden)) {
        set_error("d must be a multiple of 4, hidden a multiple of 8 up to 128, d + hidden at most 256");
        return HAG_EINVAL;
    }
    if (h->n == 0) return HAG_OK;
    if (!x || !w_ih || !w_hh || !g_a || !g_x || !g_w_ih || !g_w_hh || !g_b || !workspace) { set_error("NULL pointer"); return HAG_EINVAL; }
    if (((uintptr_t)x | (uintptr_t)workspace | (uintptr_t)g_a | (uintptr_t)g_x) & 15) { set_error("x, g_a, g_x and workspace must be 16-byte aligned"); return HAG_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    const SeqTrainLayout L = seq_train_layout(h, d, hidden);
    char *w = (char *)workspace;
    const SeqLayout F = seq_layout(h, d, hidden);           // the forward pass left its state rows there
    const float *hst = (const float *)(w + F.h), *cst = (const float *)(w + F.c);
    float *tape_g = (float *)(w + L.tape_g), *tape_c = (float *)(w + L.tape_c), *tape_h = (float *)(w + L.tape_h);
    float *gh = (float *)(w + L.gh), *gc = (float *)(w + L.gc), *wxt = (float *)(w + L.wxt), *sums = (float *)(w + L.s);
    uint16_t *wqt = (uint16_t *)(w + L.wqt);
    int32_t *unscale = (int32_t *)(w + L.unscale);
    const int64_t cells = (int64_t)h->step_x.size(), n_used = (int64_t)h->used.size();
    auto blocks = [](int64_t total) { return dim3((unsigned)std::min<int64_t>((total + 255) / 256, 65535 * 16)); };
    const int64_t levels = (int64_t)h->tile_ptr.size() - 1;
    const int rv = seq_variant(hidden);
    const int64_t resident = h->resident_reverse[rv];
    const bool fused = levels > 1 && h->one_launch && resident > 0;
    int32_t *pending = (int32_t *)(w + L.pending);
    {
        const int64_t n_state_grads = (int64_t)((L.pending - L.gh) / sizeof(float));   // (gh and gc are adjacent)
        const int64_t n_g_x = n_used < h->n ? h->n * d : 0, n_states = fused ? h->n_states : 0;
        const int64_t total = std::max({4 * hidden * (d + 31) / 32 * 32, (hidden + 31) / 32 * 32 * 256, n_state_grads, n_g_x, n_states});
        hipLaunchKernelGGL(seq_backward_start_kernel, blocks(total), dim3(256), 0, s, w_ih, w_hh, wqt, unscale, wxt, (int)d, (int)hidden, gh, n_state_grads, g_x, n_g_x,
                           h->d_pending_init, pending, n_states);
        HIP_TRY(hipGetLastError());
    }
    if (h->n_from_state > 0) {
        hipLaunchKernelGGL(seq_final_grad_kernel, dim3((unsigned)((h->n + 255) / 256)), dim3(256), 0, s, h->d_final, g_a, gh, h->n, (int)hidden);
        HIP_TRY(hipGetLastError());
    }
    for (int64_t l = fused ? 0 : levels - 1; l >= 0; --l) {
        SeqRevArgs r;
        // one launch: the tiles of the depth order, last first (what starts deeper comes earlier); else level by level, last first
        r.paths = fused ? h->d_paths_by_depth : h->d_paths + h->tile_ptr[l] * kSeqJobs * 4;
        r.n_path_tiles = fused ? h->depth_tile_ptr.back() : h->tile_ptr[l + 1] - h->tile_ptr[l];
        r.pending = fused ? pending : nullptr;
        r.reversed = fused ? 1 : 0;
        r.gave_up = h->d_gave_up;
        r.spin_limit = h->spin_limit;
        r.publish = h->wait_unreachable ? 0 : 1;
        r.step_out = h->d_step_out;
        r.step_g = h->d_step_g; r.gx = (const float *)(w + F.gx); r.wq = (const uint16_t *)(w + F.wq); r.unscale = (const float *)(w + F.bp) + 4 * hidden;
        r.wqt = wqt; r.wqt_unscale = unscale; r.tape_g = tape_g; r.tape_c = tape_c; r.tape_h = tape_h; r.h_state = hst; r.c_state = cst; r.g_a = g_a; r.gh = gh; r.gc = gc;
        r.hidden = (int32_t)hidden;
        if (r.n_path_tiles <= 0) continue;
        const int64_t cap = fused ? resident : 512;
        hipLaunchKernelGGL(kSeqReverseVariants[rv], dim3((unsigned)std::min<int64_t>(r.n_path_tiles * (rv > 0 ? kSeqJobs / kSeqRevJobs : 1), cap)), dim3(seq_reverse_block(rv)), 0, s, r);
        HIP_TRY(hipGetLastError());
    }
    {
        // recurrent weights and the per-node sums of dG, over the cells (the partial sums are added up with the others, below)
        SeqWgradArgs g{};
        g.dg = tape_g; g.z = tape_h; g.z2 = hst; g.at = h->d_xt_idx; g.prev = h->d_xt_prev; g.seg = h->d_xt_seg;
        g.rows = cells; g.range = L.hh.range; g.cols = (int32_t)hidden; g.hidden = (int32_t)hidden;
        g.partial = (float *)(w + L.partial_hh); g.s = sums; g.edge_first = (float *)(w + L.edge_first); g.edge_last = (float *)(w + L.edge_last);
        if (int rc = launch_wgrad<true>(g, L.hh, hidden, s)) return rc;
        if (L.hh.groups > 1) {
            hipLaunchKernelGGL(seq_edges_kernel, dim3((unsigned)L.hh.groups), dim3(256), 0, s, h->d_xt_seg, cells, L.hh.range, g.edge_first, g.edge_last,
                               sums, (int)(4 * hidden));
            HIP_TRY(hipGetLastError());
        }
    }
    {
        // input weights, bias and g_x, over the nodes
        SeqWgradArgs g{};
        g.dg = sums; g.z = x; g.at = h->d_used;
        g.rows = n_used; g.range = L.ih.range; g.cols = (int32_t)d; g.hidden = (int32_t)hidden; g.partial = (float *)(w + L.partial_ih);
        if (int rc = launch_wgrad<false>(g, L.ih, hidden, s)) return rc;
        const SeqReduceArgs hh{(const float *)(w + L.partial_hh), g_w_hh, nullptr, (int32_t)L.hh.groups, (int32_t)hidden, 32 * L.hh.nct};
        const SeqReduceArgs ih{g.partial, g_w_ih, g_b, (int32_t)L.ih.groups, (int32_t)d, 32 * L.ih.nct};
        const unsigned split = (unsigned)((L.hh.per + 31) / 32);
        hipLaunchKernelGGL(seq_weight_grad_reduce_kernel, dim3(split + (unsigned)((L.ih.per + 31) / 32)), dim3(256), 0, s, hh, ih, split, (int)hidden);
        HIP_TRY(hipGetLastError());
        if (n_used > 0) {
            hipLaunchKernelGGL(seq_input_grad_kernel, dim3((unsigned)std::min<int64_t>((n_used + 63) / 64, 1 << 20)), dim3(256), 0, s, sums, h->d_used, n_used,
                               wxt, g_x, (int)d, (int)hidden);
            HIP_TRY(hipGetLastError());
        }
    }
    return HAG_OK;
}

}  // extern "C"
