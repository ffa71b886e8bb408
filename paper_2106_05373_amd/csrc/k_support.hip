// Support and per-HCU activation: s = b + x w over the active input HCUs, then softmax (or
// argmax) within every hidden HCU (Alg. 1 support and softmax lines; Sec. 2).
//
// Design (gfx950):
//  * The weights are stored masked, so a hidden HCU only needs the rows of its active input
//    HCUs.  Each hidden HCU keeps an ascending list of them; the contraction for one hidden
//    HCU is a dense [B x K_h] . [K_h x M_out] product with K_h = n_active * M_in.  Silent
//    blocks are never read.
//  * The products accumulate in fp64 on the matrix cores (v_mfma_f64_16x16x4f64).  x and w are
//    fp32, so every product is exact in fp64 and the sum's rounding error stays far below the
//    fp32 rounding of the stored support.  (An fp32 accumulation of a few hundred terms of
//    magnitude ~10 drifts by ~1e-5, the size of the tolerance on the activities.)
//  * One workgroup owns one hidden HCU and kR tiles of 16 batch rows, i.e. complete softmax
//    segments, so the softmax runs in the epilogue from LDS and the support never round-trips
//    through HBM.
//  * A wave owns kTPW tiles of 16 columns; a narrow hidden HCU (few column tiles) also splits its
//    k-steps over the waves that its columns would leave idle (`parts`), and the shares' fp64 sums
//    are added through LDS in a fixed order.
//  * What bounds the short launches is instruction issue, not memory: 64 KiB of weights reach a
//    CU's LDS in 0.6 us, but an fp64 MFMA takes its SIMD for 64 cycles and no vector instruction
//    of any wave passes beside it (measured: one conversion per MFMA 71 cycles, five integer
//    instructions 87, MFMAs alone 65).  So the weight rows go straight to LDS (global_load_lds:
//    1 KiB per instruction, no registers, no LDS stores) at a row stride kS that is a compile-time
//    constant, and the operand reads of a run of k-steps need no address arithmetic; the input is
//    gathered as wide as an input HCU allows (a gather costs a cycle per distinct line) and
//    converted to fp64 once, on its way into LDS.  The product loop is then the MFMA, one LDS read
//    of each operand and one conversion per k-step.
//  * A layer whose active units do not fit one panel streams them in chunks through two stage
//    buffers, the next chunk's loads in flight during the products.  The buffers are separate
//    arrays named at compile time, so that the compiler does not make a chunk's LDS reads wait
//    for the next chunk's loads.  With one row tile they take most of a CU's LDS; where more
//    workgroups than CUs follow one another, two of them share a CU with half of the stages each,
//    for the widths that gain from it (two_per_cu).
//  * A batch of many rows may take kR = 4: the weights are then loaded and converted once for four
//    row tiles, and two workgroups share a CU, so that one's gather, softmax and stores pass under
//    the other's products.  Which form a launch takes is a matter of what its rounds of workgroups
//    cost (launch_cost).
//  * For a single row the matrix cores would compute 15 rows of padding: the same lanes then
//    accumulate their own column and units with fp64 FMAs, and the lane groups are added.
//  * The softmax of an HCU of up to 128 MCUs takes 16 lanes per row, four rows per wave: a third
//    of the instructions of one row per wave.
//  * Measured, against weights and input through registers and operand addresses in the product loop
//    (MNIST-shaped layer: 156 active units x 100 MCUs x 30 HCUs): batch 1 8.8 -> 6.5 us, batch 8192
//    472 -> 267 us (28.8 TFLOP/s), training batch of 128 11.2 -> 9.7 us by its stamps; 501 units x 70
//    MCUs x 17 HCUs at 75 rows 28.2 -> 19.5 us; STL-shaped training batch 609 -> 550 us.
//  * In training, workgroups past the support's split the batch input into the contraction
//    operands of the trace kernels, 16 rows x 64 columns per wave, beside the support.
//
// MFMA f64 16x16x4 lane layout (verified on gfx950): A[i][k] from lane i + 16 k, B[k][j] from
// lane j + 16 k, and lane l holds D[l / 16 + 4 r][l % 16] in result register r.
#include <initializer_list>
#include <mutex>
#include <type_traits>

#include "bcpnn_internal.h"
#include "device_common.h"
#include "support_layout.h"

namespace bcpnn {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef int32_t i4 __attribute__((ext_vector_type(4)));

typedef void __attribute__((address_space(3))) lds_void;

// A count as a type.
template <int V>
struct Count { static constexpr int value = V; };

// Writes the 16 batch entries of unit u in k-step ks (one row tile) as bf16 hi and lo parts
// (hi = bf16(v), lo = bf16(v - hi), round to nearest even): two 16-byte fragment chunks each.
__device__ __forceinline__ void write_split_column(const float (&v)[kRows], uint16_t* hi,
                                                   uint16_t* lo, int64_t u, int ks, int32_t n_ks) {
    uint32_t h[kRows / 2], l[kRows / 2];
#pragma unroll
    for (int q = 0; q < kRows / 2; ++q) {
        const __bf16 h0 = (__bf16)v[2 * q], h1 = (__bf16)v[2 * q + 1];
        const __bf16 l0 = (__bf16)(v[2 * q] - (float)h0), l1 = (__bf16)(v[2 * q + 1] - (float)h1);
        h[q] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
        l[q] = (uint32_t)__builtin_bit_cast(uint16_t, l0) | ((uint32_t)__builtin_bit_cast(uint16_t, l1) << 16);
    }
    const int64_t c0 = frag_chunk(u, ks, 0, n_ks), c1 = frag_chunk(u, ks, 1, n_ks);
    *reinterpret_cast<uint4*>(hi + c0) = make_uint4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<uint4*>(hi + c1) = make_uint4(h[4], h[5], h[6], h[7]);
    *reinterpret_cast<uint4*>(lo + c0) = make_uint4(l[0], l[1], l[2], l[3]);
    *reinterpret_cast<uint4*>(lo + c1) = make_uint4(l[4], l[5], l[6], l[7]);
}

// The same for one half (rows 8 h .. 8 h + 7) of the 16 entries: one 16-byte chunk each.
__device__ __forceinline__ void write_split_half(const float (&v)[kRows / 2], uint16_t* hi,
                                                 uint16_t* lo, int64_t u, int ks, int h,
                                                 int32_t n_ks) {
    uint32_t hh[kRows / 4], ll[kRows / 4];
#pragma unroll
    for (int q = 0; q < kRows / 4; ++q) {
        const __bf16 h0 = (__bf16)v[2 * q], h1 = (__bf16)v[2 * q + 1];
        const __bf16 l0 = (__bf16)(v[2 * q] - (float)h0), l1 = (__bf16)(v[2 * q + 1] - (float)h1);
        hh[q] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
        ll[q] = (uint32_t)__builtin_bit_cast(uint16_t, l0) | ((uint32_t)__builtin_bit_cast(uint16_t, l1) << 16);
    }
    const int64_t c = frag_chunk(u, ks, h, n_ks);
    *reinterpret_cast<uint4*>(hi + c) = make_uint4(hh[0], hh[1], hh[2], hh[3]);
    *reinterpret_cast<uint4*>(lo + c) = make_uint4(ll[0], ll[1], ll[2], ll[3]);
}

// How the column sums over 16 rows are formed: row by row, the sums of rows 0-7 and 8-15 added, or
// one or the other by the width of the hidden HCU's share of the input the unit belongs to (an
// out_hcu-th of the input HCUs; halves up to 256 units).
enum SumOrder { kRowByRow = 0, kHalves = 1, kByShare = 2 };

// Contraction operands of 16 rows (row tile rt) x 64 columns (pass p, lane = column) of a batch
// array [B][n], by one wave: each column split into bf16 hi / lo parts in fragment order, plus its
// sum over these rows.  kPaired (the input, with complement pairs): only the first unit of each
// input HCU enters the contraction, at the HCU's index (every unit keeps its column sum), and
// every pair (x_2p, x_2p+1) of these rows must add up to 1: passes start at an even column, so the
// partner of an even column is the next lane's.  A violation sets the layer's flag.
// The rows are read through a buffer resource over the batch, so the rows past B read as zero
// and all 16 loads are unconditional and go out together.  (The launch checks that the offsets
// fit in 32 bits.)
__device__ __forceinline__ void split_columns(const Geometry& g, const float* src, int64_t n, int32_t B,
                                              uint16_t* hi, uint16_t* lo, float* sums, int32_t n_ks,
                                              bool paired, int32_t* pair_error, int order, int rt,
                                              int p, int lane) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(src), (short)0, (int)(uint32_t)((int64_t)B * n * 4), 0x00020000);
    const int64_t i = (int64_t)p * 64 + lane;
    const bool in = i < n;
    const int64_t ic = in ? i : n - 1;
    const int row0 = rt * kRows;
    float v[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
        v[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
            rs, (uint32_t)(((int64_t)(row0 + r) * n + ic) * 4), 0, 0));
    float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
    for (int r = 0; r < kRows / 2; ++r) {
        s0 += v[r];
        s1 += v[r + kRows / 2];
    }
    float sum = s0 + s1;
    if (order != kHalves) {
        float all = s0;
#pragma unroll
        for (int r = kRows / 2; r < kRows; ++r) all += v[r];
        if (order == kRowByRow) {
            sum = all;
        } else {
            const uint32_t ih = (uint32_t)g.in_hcu, oh = (uint32_t)g.out_hcu;   // products < 2^26
            const uint32_t share = (((uint32_t)ic / g.in_mcu + 1) * oh - 1) / ih;
            const uint32_t width = ((share + 1) * ih / oh - share * ih / oh) * g.in_mcu;
            sum = width <= 256 ? sum : all;
        }
    }
    if (paired) {
        const bool first = in && (i & 1) == 0;
        bool bad = false;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float nb = __shfl_down(v[r], 1, 64);
            bad |= first && row0 + r < B && !(fabsf(v[r] + nb - 1.0f) <= kPairTolerance);
        }
        if (bad) *pair_error = 1;
    }
    if (in) {
        if (!paired) write_split_column(v, hi, lo, i, rt, n_ks);
        else if ((i & 1) == 0) write_split_column(v, hi, lo, i >> 1, rt, n_ks);
        sums[(int64_t)rt * n + i] = sum;
    }
}

__device__ __forceinline__ void split_input(const Geometry& g, const float* x, int32_t B,
                                            const TraceOperands& ops, int order, int rt, int p,
                                            int lane) {
    split_columns(g, x, g.n_in, B, ops.x_hi, ops.x_lo, ops.x_sum, ops.n_ks, ops.paired != 0,
                  ops.pair_error, order, rt, p, lane);
}

// Training with a target whose activities nobody asked for: the traces take the target, so the
// support and its softmax would go nowhere.  Only the operands are written: the input's, then the
// target's, a wave per 16 rows x 64 columns.
template <bool kStamp>
__global__ void __launch_bounds__(256)
split_kernel(Geometry g, const float* __restrict__ x, int32_t B, const float* __restrict__ target,
             TraceOperands ops, int order, unsigned long long* stamp) {
    stamp_start<kStamp>(stamp);
    __builtin_amdgcn_s_setprio(3);
    const int lane = threadIdx.x & 63;
    const int task = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int px = (int)((g.n_in + 63) / 64), pt = (int)((g.n_out + 63) / 64);
    const int tiles = (B + kRows - 1) / kRows;
    if (task < px * tiles) {
        split_input(g, x, B, ops, order, task / px, task % px, lane);
    } else if (task < (px + pt) * tiles) {
        const int t = task - px * tiles;
        split_columns(g, target, g.n_out, B, ops.t_hi, ops.t_lo, ops.t_sum, ops.n_ks, false, nullptr,
                      kHalves, t / pt, t % pt, lane);
    }
    stamp_end<kStamp>(stamp);
}

constexpr int kThinUnits = 512;           // active units from which a narrow layer goes row by row,
constexpr int kThinRows = 1024;           // up to so many rows
constexpr int kThinThreads = 512;
constexpr int kThinColumns = 16;

// The last step of the row-by-row kernels, by 16 lanes: column tid of `row` has the sum v; its support,
// then the softmax or argmax.
__device__ __forceinline__ void thin_finish(const Geometry& g, int row, int tid, double v, float bias,
                                            float gain, int mode, float* y, float* s,
                                            int32_t* winner) {
    const int M = g.out_mcu;
    const bool in = tid < M;
    const int64_t o = (int64_t)row * M + tid;
    const float sv = (float)(v + (double)bias);
    if (s && in) s[o] = sv;
    if (mode == 0) {
        const float mx = row16_max(in ? sv : -INFINITY);
        const float e = in ? expf(gain * (sv - mx)) : 0.0f;
        const float inv = 1.0f / row16_sum(e);
        if (y && in) y[o] = e * inv;
    } else {
        // (a NaN takes no part, wherever it stands)
        const bool part = in && sv > -INFINITY;
        float bv = part ? sv : -INFINITY;
        int bi = part ? tid : 0x7fffffff;
        for (int off = kThinColumns / 2; off > 0; off >>= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (tid == 0) winner[row] = bi;
    }
}

// A single narrow hidden HCU with many active units and a small batch (a readout: 3000 units to 10
// classes, 128 rows): by row tiles it would fill a handful of CUs, each with a long chain of
// chunks.  Here a workgroup takes one row: a thread accumulates all M_out (<= 16) columns of its
// units k, k + 512, ... with fp64 FMAs (W: floats per weight load), the waves add their lanes by
// halving exchanges (after which lanes hold single columns), and 16 lanes add the waves in order,
// then take the softmax or argmax.  Nothing waits between the loads and the reduction, and the
// weights are read by every workgroup from L2.  128 rows, 2900 of 3000 units -> 10: 12.3 us (in chunks of
// units, 8 workgroups: 27).
template <int W>
__global__ void __launch_bounds__(kThinThreads)
support_thin_kernel(Geometry g, const float* __restrict__ x, const float* __restrict__ w,
                    const float* __restrict__ bias, const int32_t* __restrict__ act_list,
                    const int32_t* __restrict__ act_count, uint32_t mcu_magic, float gain, int mode,
                    float* __restrict__ y, float* __restrict__ s, int32_t* __restrict__ winner) {
    typedef float wvec __attribute__((ext_vector_type(W)));
    __shared__ double sums[kThinThreads / 64][kThinColumns];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = blockIdx.x;
    const int M = g.out_mcu;
    const int32_t k_total = act_count[0] * g.in_mcu;
    const float* xrow = x + (int64_t)row * g.n_in;
    double acc[kThinColumns];
#pragma unroll
    for (int c = 0; c < kThinColumns; ++c) acc[c] = 0.0;
    const bool full = k_total == g.n_in;                       // every input HCU active: unit k
#pragma unroll 3
    for (int32_t k = tid; k < k_total; k += kThinThreads) {
        int32_t u = k;
        if (!full) {
            const int32_t h = mcu_magic ? (int32_t)__umulhi((uint32_t)k, mcu_magic) : k;
            u = (act_list[h] - h) * g.in_mcu + k;
        }
        const float* wr = w + (int64_t)u * M;
        wvec wv[kThinColumns / W];
#pragma unroll
        for (int q = 0; q < kThinColumns / W; ++q) {
            wv[q] = wvec(0.0f);
            if (W * q < M) wv[q] = *reinterpret_cast<const wvec*>(wr + W * q);
        }
        const double xv = (double)xrow[u];
#pragma unroll
        for (int q = 0; q < kThinColumns / W; ++q)
            if (W * q < M) {
#pragma unroll
                for (int e = 0; e < W; ++e) acc[W * q + e] = fma(xv, (double)wv[q][e], acc[W * q + e]);
            }
    }
    // halving exchanges: after the step of lane distance 32, 16, 8, 4 a lane holds 8, 4, 2, 1
    // columns (the upper half where its lane bit is set); the last two steps add within quads
#pragma unroll
    for (int half = kThinColumns / 2, off = 32; half >= 1; half /= 2, off /= 2) {
        const bool upper = (lane & off) != 0;
#pragma unroll
        for (int c = 0; c < half; ++c) {
            const double send = upper ? acc[c] : acc[c + half];
            const double keep = upper ? acc[c + half] : acc[c];
            acc[c] = keep + __shfl_xor(send, off, 64);
        }
    }
    acc[0] += __shfl_xor(acc[0], 2, 64);
    acc[0] += __shfl_xor(acc[0], 1, 64);
    if ((lane & 3) == 0) sums[wave][lane >> 2] = acc[0];       // lane bits 5..2 are the column's
    lds_barrier();
    if (tid >= kThinColumns) return;
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kThinThreads / 64; ++q) v += sums[q][tid];
    thin_finish(g, row, tid, v, bias[tid < M ? tid : 0], gain, mode, y, s, winner);
}

// The same for a layer whose single hidden HCU sees every input unit (M_out of 4 to 16): its weights
// are then one contiguous array, read 16 bytes per lane.  T threads, T the largest up to 512 whose
// 4 T elements are whole rows, so that a thread keeps its four columns from pass to pass and needs
// two inputs per pass (its elements span at most two units); the passes' loads go out together.  The
// threads' sums are [4 T / M][M] in LDS, added up by 32 lanes per column.  Elements past the last
// whole vector belong to the last unit and are added at the end.  Bound by its instructions and its
// round trips of memory, so there is no division, an input is converted once, and the LDS reads of
// the sum go out together.  128 rows, 3000 -> 10: 6.3 us; with divisions, a conversion per product
// and the sum in a loop 10.6; the kernel above 11.3.
template <int kBatch>
__device__ __forceinline__ void flat_passes(const float* __restrict__ xrow, const f4* __restrict__ w4,
                                            int n_vec, int n_pass, int T, int U, int M, int n_in,
                                            int u0, int tid, double (&acc)[4]) {
    const int c0 = 4 * tid - u0 * M, u3 = u0 + (c0 + 3 >= M);
    for (int p0 = 0; p0 < n_pass; p0 += kBatch) {
        f4 wv[kBatch];
        float xa[kBatch], xb[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {                     // (past the end: the last vector)
            const int v = tid + T * (p0 + q);
            wv[q] = w4[v < n_vec ? v : n_vec - 1];
            const int a = u0 + U * (p0 + q), b = u3 + U * (p0 + q);
            xa[q] = xrow[a < n_in ? a : n_in - 1];
            xb[q] = xrow[b < n_in ? b : n_in - 1];
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            if (tid + T * (p0 + q) >= n_vec) continue;
            const double da = (double)xa[q], db = (double)xb[q];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] = fma(c0 + e < M ? da : db, (double)wv[q][e], acc[e]);
        }
    }
}

__global__ void __launch_bounds__(kThinThreads)
support_flat_kernel(Geometry g, const float* __restrict__ x, const float* __restrict__ w,
                    const float* __restrict__ bias, int T, int U, uint32_t col_magic,
                    float gain, int mode, float* __restrict__ y, float* __restrict__ s, int32_t* __restrict__ winner) {
    __shared__ double part[4 * kThinThreads];
    __shared__ double sums[kThinThreads / 64][kThinColumns];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = blockIdx.x;
    const int M = g.out_mcu, n_in = (int)g.n_in;
    const float* xrow = x + (int64_t)row * n_in;
    const int n_vec = n_in * M / 4;
    const int n_pass = (n_in + U - 1) / U;                     // (the last may hold no whole vector)
    const int c = tid & (kThinColumns - 1), cc = c < M ? c : 0;
    const float bias_c = bias[cc];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (tid < T) {
        const f4* w4 = reinterpret_cast<const f4*>(w);
        const int u0 = (int)__umulhi(4u * tid, col_magic);     // 4 tid / M
        if (n_pass > 8) flat_passes<16>(xrow, w4, n_vec, n_pass, T, U, M, n_in, u0, tid, acc);
        else flat_passes<8>(xrow, w4, n_vec, n_pass, T, U, M, n_in, u0, tid, acc);
#pragma unroll
        for (int e = 0; e < 4; ++e) part[4 * tid + e] = acc[e];
    }
    lds_barrier();
    double v = 0.0;
    constexpr int kGroups = kThinThreads / kThinColumns;       // U is at most 512 (M = 4)
#pragma unroll
    for (int k = 0; k < kThinThreads / kGroups; ++k) {
        const int r = tid / kThinColumns + kGroups * k;
        const double t = part[r < U ? r * M + cc : 0];
        v += r < U ? t : 0.0;
    }
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (lane < kThinColumns) sums[wave][lane] = v;
    lds_barrier();
    if (tid >= kThinColumns) return;
    v = 0.0;
#pragma unroll
    for (int q = 0; q < kThinThreads / 64; ++q) v += sums[q][tid];
    const int rest = n_in * M - 4 * n_vec;                     // columns M - rest .. of the last unit
    if (tid < M && tid >= M - rest)
        v = fma((double)xrow[n_in - 1], (double)w[(int64_t)(n_in - 1) * M + tid], v);
    thin_finish(g, row, tid, v, bias_c, gain, mode, y, s, winner);
}

// kR: row tiles per workgroup.  kV: input elements per load of the one-chunk forms (2 when input HCUs
// have an even number of MCUs).  kS: row stride of the weight panel in LDS (panel_stride).
// kMulti: several chunks (else the one chunk holds every active unit).  kFew: a single row, on
// fp64 FMAs.  kOps: training (the contraction operands are written).  kStamp: the launch stamps
// its start and end (training launches that profiling times).  kPair: stages of half the size, so that
// two workgroups share a CU.
template <int kR, int kS, int kV, bool kMulti, bool kFew, bool kOps, bool kStamp, bool kPair = false>
__global__ void __launch_bounds__(64 * kMaxWaves)
support_kernel(Geometry g, SupportLayout lay, const float* __restrict__ x, int32_t B,
               const float* __restrict__ w, const float* __restrict__ bias,
               const int32_t* __restrict__ act_list, const int32_t* __restrict__ act_count,
               float gain, int mode, float* __restrict__ y, float* __restrict__ s,
               int32_t* __restrict__ winner, const float* __restrict__ target,
               TraceOperands ops, unsigned long long* stamp) {
    constexpr int kTPW = tiles_per_wave(kS);
    constexpr bool kNarrow = kS <= 128;
    constexpr int kStage = !kMulti ? 16 : stage_bytes(kR, kPair);
    __shared__ f4 stage0[kStage / 16];
    __shared__ f4 stage1[kStage / 16];
    __shared__ int32_t utab[kMulti ? 4 : kOneUnits];
    extern __shared__ f4 dyn[];   // the unit table (kMulti) or the panels, then the support tile
    stamp_start<kStamp>(stamp);
    // Highest wave priority: on a CU shared with the silent sweep (second stream), the SIMD
    // arbiter issues this kernel's instructions first.
    __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_waves = lay.groups * lay.parts;
    const int n_thr = 64 * n_waves;
    if constexpr (kOps) {
        if ((int)blockIdx.x >= lay.n_main) {
            const int n_pass = (int)((g.n_in + 63) / 64);
            const int n_task = n_pass * lay.n_row_tiles;
            for (int task = ((int)blockIdx.x - lay.n_main) * n_waves + wave; task < n_task;
                 task += lay.n_split * n_waves)
                split_input(g, x, B, ops, lay.sum_order, task / n_pass, task % n_pass, lane);
            stamp_end<kStamp>(stamp);
            return;
        }
    }
    const int kc = lay.kc, mpad = lay.mpad, xstride = lay.xstride;
    const int work = (int)xcd_linear_index(blockIdx.x, lay.n_main);
    const int hj = lay.row_major ? work % g.out_hcu : work / lay.n_row_groups;
    const int row0 = (lay.row_major ? work / g.out_hcu : work % lay.n_row_groups) * (kR * kRows);
    const int part = wave / lay.groups, grp = wave - part * lay.groups;
    const int lg = lane >> 4, lj = lane & 15;

    const int32_t k_total = act_count[hj] * g.in_mcu;
    const int32_t* alist = act_list + (int64_t)hj * g.in_hcu;
    const int64_t col_base = (int64_t)hj * g.out_mcu;
    // The table is filled up to the largest K_h of the layer (and past it, with its first entry),
    // so its loads do not wait for the count; entries past k_total take no part.  It begins at
    // unit k_tab: where it has no room for all of them, it is filled again every lay.win chunks.
    int32_t* units = kMulti ? reinterpret_cast<int32_t*>(dyn) : utab;
    const int k_alloc = kMulti ? lay.k_alloc : (kc + 63) & ~63;
    int k_tab = 0;
    auto fill_units = [&]() __attribute__((always_inline)) {
        for (int32_t k = tid; k < k_alloc; k += n_thr) {
            const int32_t kk = k_tab + k < lay.max_k ? k_tab + k : 0;
            const int32_t h = lay.mcu_magic ? (int32_t)__umulhi((uint32_t)kk, lay.mcu_magic) : kk;
            units[k] = (alist[h] - h) * g.in_mcu + kk;
        }
    };
    fill_units();
    // Column of tile t of this wave (a tile past the last repeats it, its result discarded).
    int col_of[kTPW];
    float bias_r[kTPW];
#pragma unroll
    for (int t = 0; t < kTPW; ++t) {
        const int nt = grp + t * lay.groups;
        const int c = (nt < lay.n_tiles ? nt : lay.n_tiles - 1) * 16 + lj;
        col_of[t] = c < g.out_mcu ? c : g.out_mcu - 1;
        bias_r[t] = bias[col_base + col_of[t]];
    }
    const int x_live = B - row0 < kR * kRows ? B - row0 : kR * kRows;     // rows of this workgroup
    lds_barrier();

    // The weight rows of chunk k0 into a stage, [kc][kS], a vector being 16 bytes, or 4 where the
    // rows are not 16-byte aligned.  Where kS is a multiple of 64, row r is rotated by 16 (r mod 4)
    // columns, so that the four rows of an operand read fall on different banks.
    auto request_w_as = [&](int k0, f4* st, auto vec_c) __attribute__((always_inline)) {
        constexpr int V = decltype(vec_c)::value;
        constexpr int kRowVecs = kS / V;
        constexpr bool kRotate = kS % 64 == 0;
        const int live = k_total - k0 < kc ? k_total - k0 : kc;
        const uint64_t wb = reinterpret_cast<uint64_t>(w + col_base);
        const uint32_t row_bytes = (uint32_t)g.n_out * 4u;
        if constexpr (kRowVecs <= 64) {
            // one or more whole rows per instruction: wave w takes the 64-vector pieces w,
            // w + n_waves, ...; a lane keeps its place in the row, its unit is read one piece ahead
            // (an LDS round trip)
            constexpr int kRowsPer = 64 / kRowVecs;
            const int lr = lane / kRowVecs;
            const int c0 = lr < kRowsPer ? V * (lane - lr * kRowVecs) : kS;   // (kS: an idle lane)
            char* dst = reinterpret_cast<char*>(st) + 4 * kS * kRowsPer * wave;
            int r = kRowsPer * wave + lr;
            const int dr = kRowsPer * n_waves;
            uint32_t u_next = (uint32_t)units[k0 - k_tab + (r < live ? r : 0)];
            for (int first = kRowsPer * wave; first < live; first += dr) {
                const uint32_t u = u_next;
                const int c = kRotate ? (c0 - 16 * (r & 3)) & (kS - 1) : c0;
                const bool in = r < live && c < g.out_mcu;
                r += dr;
                u_next = (uint32_t)units[k0 - k_tab + (r < live ? r : 0)];
                const char* src = reinterpret_cast<const char*>(
                    wb + (uint64_t)u * row_bytes + 4u * (uint32_t)c);
                if (in) {
                    if constexpr (V == 4)
                        __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)dst, 16, 0, 0);
                    else
                        __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)dst, 4, 0, 0);
                }
                dst += 4 * kS * dr;
            }
        } else {
            // several instructions per row: wave w takes the rows w, w + n_waves, ..., whose
            // addresses are wave-uniform; lane i holds the units of its row i (64 at a time)
            constexpr int kPieces = (kRowVecs + 63) / 64;
            for (int first = wave; first < live; first += 64 * n_waves) {
                const int mine = first + n_waves * lane;
                const int ul = units[k0 - k_tab + (mine < live ? mine : 0)];
                int i = 0;
                for (int r = first; r < live && i < 64; r += n_waves, ++i) {
                    uint64_t row = wb + (uint64_t)(uint32_t)__builtin_amdgcn_readlane(ul, i) * row_bytes;
                    asm("" : "+s"(row));                  // in scalar registers
                    float* dst = reinterpret_cast<float*>(st) + kS * r;
                    int at0 = V * lane - (kRotate ? 16 * (r & 3) : 0);
                    if constexpr (kPieces > 1) asm volatile("" : "+v"(at0));
#pragma unroll
                    for (int q = 0; q < kPieces; ++q) {
                        const int c = kRotate ? (at0 + 64 * V * q) & (kS - 1) : at0 + 64 * V * q;
                        if (c < g.out_mcu) {
                            const char* src = reinterpret_cast<const char*>(row) + 4u * (uint32_t)c;
                            if constexpr (V == 4)
                                __builtin_amdgcn_global_load_lds(
                                    (const void*)src, (lds_void*)(dst + 256 * q), 16, 0, 0);
                            else
                                __builtin_amdgcn_global_load_lds(
                                    (const void*)src, (lds_void*)(dst + 64 * q), 4, 0, 0);
                        }
                    }
                }
            }
        }
    };
    auto request_w = [&](int k0, f4* st) __attribute__((always_inline)) {
        if (lay.vec4) request_w_as(k0, st, Count<4>{});
        else request_w_as(k0, st, Count<1>{});
    };
    // The input panel [16 kR][xstride] of chunk k0, after the weights: wave w takes rows w,
    // w + n_waves, ... (rw of them).  With one chunk it is gathered into registers, kV units per
    // lane in runs of 64 kV, and stored as fp64; slot q is (run q / rw, row q % rw), so that a
    // row's address is wave-uniform and a run's units are read once.  With several chunks it goes
    // straight to LDS in fp32 (registers would have to hold it during the products).
    typedef float xvec __attribute__((ext_vector_type(kV)));
    constexpr int kSlots = kXRegs / kV;
    xvec xr[kSlots];
    auto load_x = [&](int k0) __attribute__((always_inline)) {
        int i = 0, kb = kV * lane;
        uint32_t off = 0;
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
            if (q < lay.x_slots) {                                         // uniform
                if (i == 0) off = (uint32_t)units[k0 + (kb < kc ? kb : 0)] * 4u;
                int row = wave + n_waves * i;
                row = row0 + (row < x_live ? row : x_live - 1);
                const char* xrow = reinterpret_cast<const char*>(x + (int64_t)row * g.n_in);
                xr[q] = *reinterpret_cast<const xvec*>(xrow + off);
                if (++i == lay.rw) { i = 0; kb += 64 * kV; }
            }
        }
    };
    auto store_x = [&](f4* st) __attribute__((always_inline)) {
        double* xp = reinterpret_cast<double*>(reinterpret_cast<float*>(st) + kc * kS);
        int i = 0, kb = kV * lane;
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
            if (q < lay.x_slots) {
                const int row = wave + n_waves * i;
                if (row < x_live && kb < kc) {
                    double* dst = xp + row * xstride + kb;
#pragma unroll
                    for (int e = 0; e < kV; ++e) dst[e] = (double)xr[q][e];
                }
                if (++i == lay.rw) { i = 0; kb += 64 * kV; }
            }
        }
    };
    auto request_x = [&](int k0, f4* st) __attribute__((always_inline)) {
        float* xp = reinterpret_cast<float*>(st) + kc * kS;
        for (int kb = 0; kb < kc; kb += 64) {
            const uint32_t off = (uint32_t)units[k0 - k_tab + kb + lane] * 4u;
            const bool in = kb + lane < kc;
            for (int row = wave; row < x_live; row += n_waves) {
                const char* src = reinterpret_cast<const char*>(x + (int64_t)(row0 + row) * g.n_in) + off;
                if (in) __builtin_amdgcn_global_load_lds((const void*)src,
                                                         (lds_void*)(xp + row * xstride + kb), 4, 0, 0);
            }
        }
    };

    d4 acc[kR][kTPW];
    double accf[kTPW];
#pragma unroll
    for (int t = 0; t < kTPW; ++t) {
        accf[t] = 0.0;
#pragma unroll
        for (int r = 0; r < kR; ++r) acc[r][t] = d4{0.0, 0.0, 0.0, 0.0};
    }
    // This wave's k-steps of a chunk are per part .. per part + per - 1 (step ks: lane group lg
    // holds unit 4 ks + lg).  The operands of kSteps steps are read from LDS together, during the
    // products of the kSteps before them.
    constexpr int kSteps = kR * kTPW >= 4 ? 2 : 4;
    typedef std::conditional_t<kMulti, float, double> xelem;
    struct Operands {
        xelem a[kSteps][kR];
        float b[kSteps][kTPW];
    };
    int b_of[kTPW];                        // this lane's column in its rotated rows
#pragma unroll
    for (int t = 0; t < kTPW; ++t)
        b_of[t] = kS % 64 == 0 ? (col_of[t] + 16 * lg) & (kS - 1) : col_of[t];
    auto read_ops = [&](Operands& o, const xelem* ap, const float* bp, int u0)
                        __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
#pragma unroll
            for (int t = 0; t < kTPW; ++t) o.b[u][t] = bp[4 * kS * (u0 + u) + b_of[t]];
#pragma unroll
            for (int r = 0; r < kR; ++r) o.a[u][r] = ap[4 * (u0 + u) + r * kRows * xstride];
        }
    };
    auto step = [&](const xelem (&a)[kR], const float (&b)[kTPW]) __attribute__((always_inline)) {
        double bv[kTPW];
#pragma unroll
        for (int t = 0; t < kTPW; ++t) bv[t] = (double)b[t];
        if constexpr (kFew) {
#pragma unroll
            for (int t = 0; t < kTPW; ++t) accf[t] = fma((double)a[0], bv[t], accf[t]);
        } else {
#pragma unroll
            for (int r = 0; r < kR; ++r) {
                const double av = (double)a[r];
#pragma unroll
                for (int t = 0; t < kTPW; ++t)
                    acc[r][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[t], acc[r][t], 0, 0, 0);
            }
        }
    };
    auto steps_of = [&](const Operands& o) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kSteps; ++u) step(o.a[u], o.b[u]);
    };
    auto products = [&](int k0, const f4* st) __attribute__((always_inline)) {
        const int live = k_total - k0 < kc ? k_total - k0 : kc;
        const int first = lay.per * part;
        const int all = (live + 3) / 4;
        const int end = first + lay.per < all ? first + lay.per : all;   // this wave's last step + 1
        if (first >= end) return;
        const int last = end == all ? live : 4 * end;                    // its units end here
        const float* ws = reinterpret_cast<const float*>(st);
        const xelem* ap = reinterpret_cast<const xelem*>(ws + kc * kS) +
                          (kFew ? 0 : lj * xstride) + 4 * first + lg;
        const float* bp = ws + (4 * first + lg) * kS;
        // the last kSteps steps.  A share of whole k-steps ends before those past its end; in a
        // partial one these, and the units past it, take zeros.  (Blanking every share's last steps
        // took 4 to 11%: 200 MCUs, 1000 units, 100 HCUs at 208 rows 398 against 356 us.)
        auto finish = [&](Operands& o, int ks) __attribute__((always_inline)) {
            if (last == 4 * end) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kSteps; ++u)
                    if (ks + u < end) step(o.a[u], o.b[u]);
                return;
            }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                const bool in = 4 * (ks + u) + lg < last;
#pragma unroll
                for (int t = 0; t < kTPW; ++t) o.b[u][t] = in ? o.b[u][t] : 0.0f;
#pragma unroll
                for (int r = 0; r < kR; ++r) o.a[u][r] = in ? o.a[u][r] : xelem(0);
            }
            steps_of(o);
        };
        Operands p, q;               // (reads past the panel after the last step: never used)
        read_ops(p, ap, bp, 0);
        int ks = first;
        for (; ks + 2 * kSteps < end; ks += 2 * kSteps) {
            read_ops(q, ap, bp, kSteps);
            steps_of(p);
            ap += 4 * 2 * kSteps;
            bp += 4 * kS * 2 * kSteps;
            read_ops(p, ap, bp, 0);
            steps_of(q);
        }
        if (ks + kSteps < end) {
            read_ops(q, ap, bp, kSteps);
            steps_of(p);
            finish(q, ks + kSteps);
        } else {
            finish(p, ks);
        }
    };

    if constexpr (kMulti) {
        // a chunk: its loads have arrived in every wave, the next one's go out (into the buffer
        // that every wave has finished reading), then its products
        auto chunk = [&](int c, f4* st, f4* next) __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(0);
            lds_barrier();
            if ((c + 1) * kc < k_total) {
                if ((c + 1) * kc - k_tab >= lay.win * kc) {    // (every wave is done with the table)
                    k_tab = (c + 1) * kc;
                    fill_units();
                    lds_barrier();
                }
                request_w((c + 1) * kc, next);
                request_x((c + 1) * kc, next);
            }
            products(c * kc, st);
        };
        request_w(0, stage0);
        request_x(0, stage0);
        for (int c = 0; c * kc < k_total; c += 2) {
            chunk(c, stage0, stage1);
            if ((c + 1) * kc < k_total) chunk(c + 1, stage1, stage0);
        }
    } else {
        request_w(0, dyn);
        load_x(0);
        __builtin_amdgcn_s_waitcnt(0);
        store_x(dyn);
        lds_barrier();
        products(0, dyn);
    }

    // The support tile [16 kR][mpad] takes the stages (half of its rows in each) or, with one
    // chunk, the panels' LDS; the shares' sums come after its rows in the first stage (one row
    // tile) or take the dynamic LDS, the table and panels being done.
    lds_barrier();
    float* const tile0 = kMulti ? reinterpret_cast<float*>(stage0) : reinterpret_cast<float*>(dyn);
    float* const tile1 = kMulti ? reinterpret_cast<float*>(stage1) - 8 * kR * mpad : tile0;
    auto tile_row = [&](int r) { return (r < 8 * kR ? tile0 : tile1) + r * mpad; };
    double* red = kMulti && kR == 1 ? reinterpret_cast<double*>(tile0 + 8 * mpad)
                                    : reinterpret_cast<double*>(reinterpret_cast<float*>(dyn) +
                                                                (kMulti ? 0 : kR * kRows * mpad));
    if constexpr (kFew) {
        // the lane groups' shares of each column
#pragma unroll
        for (int t = 0; t < kTPW; ++t) {
            accf[t] += __shfl_xor(accf[t], 16, 64);
            accf[t] += __shfl_xor(accf[t], 32, 64);
        }
    }
    if (lay.parts > 1) {
        constexpr int kVals = kFew ? kTPW : 4 * kR * kTPW;     // doubles per lane
        if (part > 0) {
            double* mine = red + ((part - 1) * lay.groups + grp) * (kVals * 64) + lane;
            if constexpr (kFew) {
#pragma unroll
                for (int t = 0; t < kTPW; ++t) mine[t * 64] = accf[t];
            } else {
#pragma unroll
                for (int r = 0; r < kR; ++r)
#pragma unroll
                    for (int t = 0; t < kTPW; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            mine[((r * kTPW + t) * 4 + e) * 64] = acc[r][t][e];
            }
        }
        lds_barrier();
        if (part == 0) {
            for (int p = 1; p < lay.parts; ++p) {
                const double* from = red + ((p - 1) * lay.groups + grp) * (kVals * 64) + lane;
                if constexpr (kFew) {
#pragma unroll
                    for (int t = 0; t < kTPW; ++t) accf[t] += from[t * 64];
                } else {
#pragma unroll
                    for (int r = 0; r < kR; ++r)
#pragma unroll
                        for (int t = 0; t < kTPW; ++t)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[r][t][e] += from[((r * kTPW + t) * 4 + e) * 64];
                }
            }
        }
    }
    if (part == 0) {
#pragma unroll
        for (int t = 0; t < kTPW; ++t) {
            const int c = (grp + t * lay.groups) * 16 + lj;
            if (c < g.out_mcu) {
                const double bj = (double)bias_r[t];
                if constexpr (kFew) {
                    if (lg == 0) tile0[c] = (float)(accf[t] + bj);
                } else {
#pragma unroll
                    for (int r = 0; r < kR; ++r)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            tile_row(r * kRows + lg + 4 * e)[c] = (float)(acc[r][t][e] + bj);
                }
            }
        }
    }
    lds_barrier();

    // Softmax (or argmax) per row: kLanes lanes hold its columns l, l + kLanes, ... (kPer of them,
    // straight-line; the columns past the last repeat it and take no part).
    constexpr int kLanes = kNarrow ? 16 : 64;
    constexpr int kRowsPerWave = 64 / kLanes;
    const int l = lane & (kLanes - 1);
    auto activate = [&](auto per_c) __attribute__((always_inline)) {
        constexpr int kPer = decltype(per_c)::value;
        for (int rw = wave * kRowsPerWave; rw < x_live; rw += n_waves * kRowsPerWave) {
            const int row = rw + lane / kLanes;
            const bool valid = row < x_live;
            float* sr = tile_row(valid ? row : rw);
            const int64_t o = (int64_t)(row0 + row) * g.n_out + col_base;
            float e[kPer];
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int m = l + kLanes * q;
                e[q] = sr[m < g.out_mcu ? m : g.out_mcu - 1];
            }
            if (s) {
#pragma unroll
                for (int q = 0; q < kPer; ++q)
                    if (valid && l + kLanes * q < g.out_mcu) s[o + l + kLanes * q] = e[q];
            }
            if (mode == 0) {
                float mx = e[0];
#pragma unroll
                for (int q = 1; q < kPer; ++q) mx = fmaxf(mx, e[q]);
                mx = kNarrow ? row16_max(mx) : wave_max_dpp(mx);
#pragma unroll
                for (int q = 0; q < kPer; ++q)
                    e[q] = l + kLanes * q < g.out_mcu ? expf(gain * (e[q] - mx)) : 0.0f;
                // The sum is that of 64 lanes holding columns l, l + 64, ... added up a binary
                // tree, in both layouts: columns l and l + 64, then four rows of 16 lanes.
                float d;
                if constexpr (kNarrow) {
                    float t4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int q = 0; q < kPer; ++q) t4[q & 3] += e[q];
#pragma unroll
                    for (int q = 0; q < (kPer < 4 ? kPer : 4); ++q) t4[q] = row16_sum(t4[q]);
                    d = (t4[3] + t4[2]) + (t4[1] + t4[0]);
                } else {
                    d = 0.0f;
#pragma unroll
                    for (int q = 0; q < kPer; ++q) d += e[q];
                    d = wave_sum_dpp(d);
                }
                const float inv = 1.0f / d;
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    const int m = l + kLanes * q;
                    if (valid && m < g.out_mcu) {
                        const float yv = e[q] * inv;
                        if constexpr (kOps) sr[m] = yv;   // kept for the contraction operands
                        if (y) y[o + m] = yv;             // training may not ask for them
                    }
                }
            } else {
                float bv = -INFINITY;
                int bi = 0x7fffffff;
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    const int m = l + kLanes * q;
                    if (m < g.out_mcu && e[q] > bv) { bv = e[q]; bi = m; }
                }
                for (int off = kLanes / 2; off > 0; off >>= 1) {
                    const float ov = __shfl_xor(bv, off, 64);
                    const int oi = __shfl_xor(bi, off, 64);
                    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
                }
                if (valid && l == 0) winner[(int64_t)(row0 + row) * g.out_hcu + hj] = bi;
            }
        }
    };
    if constexpr (kNarrow) {
        if (g.out_mcu <= 32) activate(Count<2>{});
        else if (g.out_mcu <= 64) activate(Count<4>{});
        else activate(Count<8>{});
    } else {
        activate(Count<kS / 64>{});
    }
    if constexpr (kOps) {
        // Contraction operands of this workgroup's hidden HCU: its columns of t (the activity
        // above, or the target), each split into bf16 hi / lo parts in fragment order, plus the
        // column sums per row tile.  Rows past B are written as zeros.
        // The columns go out in halves of 8 rows (one 16-byte fragment chunk of hi and of lo per
        // half), so that 2 M_out threads share a row tile; the two halves of a column sit in
        // neighbouring lanes and add their row sums with one lane exchange.
        lds_barrier();
        const int n_half = 2 * g.out_mcu;
        const int tiles = (x_live + kRows - 1) / kRows;
        for (int base = 0; base < n_half * tiles; base += n_thr) {     // uniform trip count
            const int q = base + tid;
            const bool live = q < n_half * tiles;
            const int rtl = kR == 1 || !live ? 0 : q / n_half;         // row tile
            const int m = live ? (q - rtl * n_half) >> 1 : 0;
            const int half = q & 1;
            float v[kRows / 2];
            float sum = 0.0f;
#pragma unroll
            for (int i = 0; i < kRows / 2; ++i) {
                const int r = rtl * kRows + 8 * half + i;
                v[i] = live && r < x_live
                           ? (target ? target[(int64_t)(row0 + r) * g.n_out + col_base + m]
                                     : tile_row(r)[m])
                           : 0.0f;
                sum += v[i];
            }
            const float total = sum + __shfl_xor(sum, 1, 64);           // same bits in both lanes
            if (live) {
                const int64_t col = col_base + m;
                const int rt = row0 / kRows + rtl;
                write_split_half(v, ops.t_hi, ops.t_lo, col, rt, half, ops.n_ks);
                if (half == 0) ops.t_sum[(int64_t)rt * g.n_out + col] = total;
            }
        }
        stamp_end<kStamp>(stamp);
    }
}

// Calls f with the kernel of a shape, panel stride and input vector (which the one-chunk forms gather
// with: the others have a vector of 1).
template <bool kOps, bool kStamp, typename F>
hipError_t with_kernel(int shape, int stride, int xv, F&& f) {
    auto narrow = [&](auto s_c) -> hipError_t {
        constexpr int S = decltype(s_c)::value;
        switch (shape) {
            case kOneChunk:
                return xv == 2 ? f(support_kernel<1, S, 2, false, false, kOps, kStamp>)
                               : f(support_kernel<1, S, 1, false, false, kOps, kStamp>);
            case kChunks: return f(support_kernel<1, S, 1, true, false, kOps, kStamp>);
            case kManyRows: return f(support_kernel<kManyTiles, S, 1, true, false, kOps, kStamp>);
            case kTwoPerCu:
                if constexpr (S == 128) return f(support_kernel<1, S, 1, true, false, kOps, kStamp, true>);
                break;
            default: break;
        }
        if constexpr (!kOps) {
            if (shape == kFewOne)
                return xv == 2 ? f(support_kernel<1, S, 2, false, true, false, false>)
                               : f(support_kernel<1, S, 1, false, true, false, false>);
            if (shape == kFewChunks) return f(support_kernel<1, S, 1, true, true, false, false>);
        }
        return hipErrorInvalidValue;
    };
    switch (stride) {
        case 16: return narrow(Count<16>{});
        case 80: return narrow(Count<80>{});
        case 128: return narrow(Count<128>{});
        case 256:
            return shape == kTwoPerCu ? f(support_kernel<1, 256, 1, true, false, kOps, kStamp, true>)
                                      : f(support_kernel<1, 256, 1, true, false, kOps, kStamp>);
        case 512: return f(support_kernel<1, 512, 1, true, false, kOps, kStamp>);
        case 1024: return f(support_kernel<1, 1024, 1, true, false, kOps, kStamp>);
        default: return hipErrorInvalidValue;
    }
}

// Order of the input's column sums.
int input_sum_order(const Geometry& g, int32_t max_k) {
    const int64_t narrow = (int64_t)(g.in_hcu / g.out_hcu) * g.in_mcu;    // the narrowest share
    if (max_k <= 12 || narrow > 256) return kRowByRow;
    return g.in_hcu % g.out_hcu == 0 || narrow + g.in_mcu <= 256 ? kHalves : kByShare;
}

// Lets every support variant of one mode take dynamic LDS up to the workgroup's limit.
template <bool kOps, bool kStamp>
void raise_lds_limit() {
    for (int xv = 1; xv <= 2; ++xv)
        for (int stride : {16, 80, 128, 256, 512, 1024})
            for (int v = kOneChunk; v < kShapes; ++v)
                (void)with_kernel<kOps, kStamp>(v, stride, xv, [](auto kernel) {
                    return hipFuncSetAttribute((const void*)kernel,
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)kLdsLimit);
                });
}

}  // namespace

hipError_t launch_support(hipStream_t stream, const Geometry& g, const float* x, int32_t B,
                          const float* w, const float* bias, const int32_t* act_list,
                          const int32_t* act_count, int32_t max_active, float gain, int mode,
                          float* y, float* s, int32_t* winner, const float* target,
                          const TraceOperands* ops, hipEvent_t start, hipEvent_t stop,
                          unsigned long long* stamp) {
    const int32_t max_k = max_active * g.in_mcu;
    const int64_t row_tiles = (B + kRows - 1) / kRows;
    // the input rows of the last row tile (up to 15 past B) must have 32-bit byte offsets
    if (row_tiles * kRows * g.n_in * 4 > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    // (the target's rows must have 32-bit byte offsets too)
    if (ops && target && !y && !s && row_tiles * kRows * g.n_out * 4 <= (int64_t)UINT32_MAX) {
        const int64_t tasks = row_tiles * ((g.n_in + 63) / 64 + (g.n_out + 63) / 64);
        return launch_timed(stamp ? split_kernel<true> : split_kernel<false>,
                            dim3((unsigned)((tasks + 3) / 4)), dim3(256), 0, stream, start, stop, g, x,
                            B, target, *ops, input_sum_order(g, max_k), stamp);
    }
    if (!ops && g.out_mcu <= kThinColumns && max_k >= kThinUnits &&
        g.out_hcu == 1 && B <= kThinRows) {
        const int width = g.out_mcu % 4 == 0 ? 4 : g.out_mcu % 2 == 0 ? 2 : 1;
        const uint32_t magic = g.in_mcu > 1 ? magic_of(g.in_mcu) : 0;
        // every input unit active (a single hidden HCU: its count is max_active) and no more than two
        // units in four consecutive weights: the contiguous form, 6.3 against 11.3 us (3000 -> 10)
        if (max_active == g.in_hcu && g.out_mcu >= 4) {
            const int whole = g.out_mcu % 4 == 0 ? g.out_mcu / 4 : g.out_mcu % 2 == 0 ? g.out_mcu / 2 : g.out_mcu;
            const int T = kThinThreads / whole * whole;
            return launch_timed(support_flat_kernel, dim3((unsigned)B), dim3(kThinThreads), 0, stream,
                                start, stop, g, x, w, bias, T, 4 * T / g.out_mcu, magic_of(g.out_mcu),
                                gain, mode, y, s, winner);
        }
        return launch_timed(width == 4 ? support_thin_kernel<4>
                            : width == 2 ? support_thin_kernel<2> : support_thin_kernel<1>,
                            dim3((unsigned)B), dim3(kThinThreads), 0, stream, start, stop,
                            g, x, w, bias, act_list, act_count, magic, gain, mode, y, s, winner);
    }
    SupportLayout lay;
    size_t lds = 0;
    const int shape = choose_layout(g, B, max_k, ops != nullptr, &lay, &lds);
    if (shape < 0) return hipErrorInvalidValue;
    const int stride = panel_stride(g.out_mcu), xv = input_vec(g);
    const int n_waves = lay.groups * lay.parts;
    int64_t blocks = lay.n_main;
    lay.sum_order = input_sum_order(g, max_k);
    if (ops) {
        lay.n_split = (int)split_workgroups(g, lay);
        blocks += lay.n_split;
    }
    // allow dynamic LDS beyond 64 KB (gfx950 has 160 KB per workgroup): raised once, for
    // every variant a launch can pick, to the largest size a launch can ask for
    static std::once_flag raised;
    std::call_once(raised, [] {
        raise_lds_limit<false, false>();
        raise_lds_limit<true, false>();
        raise_lds_limit<true, true>();
        (void)hipGetLastError();
    });
    const TraceOperands o = ops ? *ops : TraceOperands{};
    // the events (when given) are recorded around the launch
    auto go = [&](auto kernel) {
        return launch_timed(kernel, dim3((unsigned)blocks), dim3(64 * n_waves), lds, stream, start,
                            stop, g, lay, x, B, w, bias, act_list, act_count, gain, mode, y, s,
                            winner, target, o, stamp);
    };
    if (!ops) return stamp ? hipErrorInvalidValue : with_kernel<false, false>(shape, stride, xv, go);
    return stamp ? with_kernel<true, true>(shape, stride, xv, go) : with_kernel<true, false>(shape, stride, xv, go);
}

}  // namespace bcpnn
