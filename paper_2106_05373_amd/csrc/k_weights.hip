// Initial state, weight recompute, mask application.
//
// Initial state and mask application are whole-matrix passes: each workgroup takes one row i of the
// [N_in][N_out] matrices per iteration of a grid-stride loop over rows; within a row the lanes walk
// consecutive columns, so every wave touches contiguous spans.  The mask row [out_hcu] of the row's
// input HCU is read through the cache.
//
// The weight recompute (Alg. 1 weight and mask lines) touches the active blocks only, unless these are
// most of the matrix or of its lines (whole_matrix below).  A silent
// weight is 0, and every writer of w keeps it so: the initial state, the upload (apply_mask_kernel),
// the structural update (which zeroes what it silences) and the batches (which write active blocks).
// Rewriting those zeros was 95% of the pass on the STL-shaped layer: with its reads coming from HBM
// between the stores, 690 us (2.3 GB, 3.4 TB/s; 390 us when the reads are repeated and stay in the
// Infinity Cache), against 54 us for the 221 MB of the active blocks.
#include <algorithm>
#include <numeric>

#include "bcpnn_internal.h"
#include "device_common.h"

namespace bcpnn {
namespace {

constexpr int kSweepThreads = 256;

__global__ void __launch_bounds__(kSweepThreads)
init_state_kernel(Geometry g, const uint8_t* __restrict__ mask, float pij0, float noise,
                  uint64_t seed, int drop, float* __restrict__ pij, float* __restrict__ w) {
    const float p0 = round_storage(pij0, drop);
    for (int64_t i = blockIdx.x; i < g.n_in; i += gridDim.x) {
        const uint8_t* mrow = mask + (int64_t)(i / g.in_mcu) * g.out_hcu;
        float* prow = pij + i * g.n_out;
        float* wrow = w + i * g.n_out;
        for (int64_t j = threadIdx.x; j < g.n_out; j += kSweepThreads) {
            prow[j] = p0;
            float v = 0.0f;
            if (mrow[j / g.out_mcu]) {
                const float u = splitmix_uniform(seed, (uint64_t)(i * g.n_out + j));
                v = __fmul_rn(noise, 2.0f * u - 1.0f);   // 2u - 1 is exact in fp32
            }
            wrow[j] = round_storage(v, drop);
        }
    }
}

// w of one hidden HCU's active units, V floats per lane: `lanes` (a power of two, at most 64) lanes
// take a unit's row segment, kWeightRows rows per lane in flight.  Workgroups past n_work store the
// bias.  (A row per 32 lanes leaves 7 of 32 idle at 100 MCUs; the pass waits for memory, not lanes.)
constexpr int kWeightRows = 4;
template <int V>
__global__ void __launch_bounds__(kSweepThreads)
recompute_active_kernel(Geometry g, const int32_t* __restrict__ act_list,
                        const int32_t* __restrict__ act_count, uint32_t per_hcu, uint32_t n_work,
                        uint32_t n_bias, int lanes, uint32_t mcu_magic, const float* __restrict__ pi,
                        const float* __restrict__ pj, const float* __restrict__ pij, float eps,
                        float bias_gain, int drop, float* __restrict__ w, float* __restrict__ b) {
    typedef float vec __attribute__((ext_vector_type(V)));
    for (uint32_t work = blockIdx.x; work < n_work + n_bias; work += gridDim.x) {
        if (work >= n_work) {
            const int64_t j = (int64_t)(work - n_work) * kSweepThreads + threadIdx.x;
            if (j < g.n_out) b[j] = bias_gain * __logf(fmaxf(pj[j], eps));
            continue;
        }
        const int hj = work / per_hcu;
        const int rows_at_once = kSweepThreads / lanes;
        const int step = rows_at_once * kWeightRows;
        const int c0 = V * (threadIdx.x & (lanes - 1));
        const int k_total = act_count[hj] * g.in_mcu;
        const int32_t* list = act_list + (int64_t)hj * g.in_hcu;
        const int64_t col0 = (int64_t)hj * g.out_mcu;
        // (one pass, unless a captured launch is replayed under a mask of more active units)
        for (int r0 = (work % per_hcu) * step + threadIdx.x / lanes; r0 < k_total;
             r0 += per_hcu * step) {
            int64_t row[kWeightRows];
            float pr[kWeightRows];
#pragma unroll
            for (int q = 0; q < kWeightRows; ++q) {
                const int k = r0 + rows_at_once * q;
                const int kk = k < k_total ? k : 0;
                const int h = mcu_magic ? (int)__umulhi((uint32_t)kk, mcu_magic) : kk;
                const int64_t i = (int64_t)list[h] * g.in_mcu + (kk - h * g.in_mcu);
                pr[q] = pi[i];
                row[q] = i * g.n_out + col0;
            }
            for (int c = c0; c < g.out_mcu; c += V * lanes) {
                const vec pc = *reinterpret_cast<const vec*>(pj + col0 + c);
                vec p[kWeightRows];
#pragma unroll
                for (int q = 0; q < kWeightRows; ++q)
                    p[q] = *reinterpret_cast<const vec*>(pij + row[q] + c);
#pragma unroll
                for (int q = 0; q < kWeightRows; ++q) {
                    if (r0 + rows_at_once * q >= k_total) continue;
                    vec v;
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        v[e] = round_storage(log_ratio(p[q][e], pr[q], pc[e], eps), drop);
                    *reinterpret_cast<vec*>(w + row[q] + c) = v;
                }
            }
        }
    }
}

// w of the whole matrix, a row per workgroup, V floats per lane: 0 where the mask is not set, and
// Pij is read only where it is.  A column's hidden HCU is the high word of 2 j * ceil(2^31 / out_mcu)
// (magic), exact while j * out_mcu < 2^31.  Eight accesses of a lane in flight, w
// stored with the non-temporal hint.  Workgroups past the rows store the bias.
constexpr int kRowUnroll = 8;
template <int V>
__global__ void __launch_bounds__(kSweepThreads)
recompute_rows_kernel(Geometry g, const uint8_t* __restrict__ mask, uint32_t magic,
                      const float* __restrict__ pi, const float* __restrict__ pj,
                      const float* __restrict__ pij, float eps, float bias_gain, int drop,
                      float* __restrict__ w, float* __restrict__ b) {
    typedef float vec __attribute__((ext_vector_type(V)));
    const int64_t i = blockIdx.x;
    if (i >= g.n_in) {
        const int64_t j = (i - g.n_in) * kSweepThreads + threadIdx.x;
        if (j < g.n_out) b[j] = bias_gain * __logf(fmaxf(pj[j], eps));
        return;
    }
    const uint32_t n_vec = (uint32_t)(g.n_out / V);
    const uint8_t* mrow = mask + (int64_t)(i / g.in_mcu) * g.out_hcu;
    const float pii = pi[i];
    const vec* pj_v = reinterpret_cast<const vec*>(pj);
    const vec* prow = reinterpret_cast<const vec*>(pij + i * g.n_out);
    vec* wrow = reinterpret_cast<vec*>(w + i * g.n_out);
    for (uint32_t q0 = threadIdx.x; q0 < n_vec; q0 += kSweepThreads * kRowUnroll) {
        vec p[kRowUnroll], pc[kRowUnroll];
        uint32_t live[kRowUnroll];                     // bit e: column V q + e is in an active block
#pragma unroll
        for (int u = 0; u < kRowUnroll; ++u) {
            const uint32_t q = q0 + u * kSweepThreads;
            live[u] = 0;
            p[u] = pc[u] = vec(0.0f);
            if (q < n_vec) {
                const uint32_t h0 = __umulhi(2 * V * q, magic);
                const uint32_t h1 = __umulhi(2 * V * q + 2 * (V - 1), magic);
                const uint32_t m0 = mrow[h0] != 0, m1 = mrow[h1] != 0;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const uint32_t h = __umulhi(2 * V * q + 2 * e, magic);
                    const uint32_t m = h == h0 ? m0 : h == h1 ? m1 : (mrow[h] != 0);
                    live[u] |= m << e;
                }
                if (live[u]) {
                    p[u] = prow[q];
                    pc[u] = pj_v[q];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kRowUnroll; ++u) {
            const uint32_t q = q0 + u * kSweepThreads;
            if (q >= n_vec) continue;
            vec v;
#pragma unroll
            for (int e = 0; e < V; ++e)
                v[e] = live[u] >> e & 1u ? round_storage(log_ratio(p[u][e], pii, pc[u][e], eps), drop)
                                         : 0.0f;
            __builtin_nontemporal_store(v, wrow + q);
        }
    }
}

__global__ void __launch_bounds__(kSweepThreads)
bias_kernel(int64_t n_out, const float* __restrict__ pj, float eps, float bias_gain,
            float* __restrict__ b) {
    const int64_t j = (int64_t)blockIdx.x * kSweepThreads + threadIdx.x;
    if (j < n_out) b[j] = bias_gain * __logf(fmaxf(pj[j], eps));
}

__global__ void __launch_bounds__(kSweepThreads)
apply_mask_kernel(Geometry g, const uint8_t* __restrict__ mask, float* __restrict__ w) {
    for (int64_t i = blockIdx.x; i < g.n_in; i += gridDim.x) {
        const uint8_t* mrow = mask + (int64_t)(i / g.in_mcu) * g.out_hcu;
        float* wrow = w + i * g.n_out;
        for (int64_t j = threadIdx.x; j < g.n_out; j += kSweepThreads)
            if (!mrow[j / g.out_mcu]) wrow[j] = 0.0f;
    }
}

unsigned sweep_blocks(const Geometry& g) {
    const int64_t cap = 8192;
    return (unsigned)(g.n_in < cap ? g.n_in : cap);
}

// Whether the weight pass takes the whole matrix: where the 128-byte lines that hold the active
// blocks' rows, each fetched and stored once per block, amount to most of the matrix or more.  A
// block's row of 4 out_mcu bytes begins at a multiple of the greatest common divisor of the two
// lengths.  While Pij and w stay in the Infinity Cache a line fetched twice is cheap, so the active
// blocks win up to 1.6 times the matrix, beyond it up to 0.88 (a fifth less where a block's row is no
// multiple of 16 bytes: they move 4 bytes per lane; 2984 x 16000 of 50 MCUs, half set: 84 and 108 us).
// Fewer than 512 rows, or rows that leave lanes of a workgroup idle, hold the whole matrix back in
// proportion.  Whole and active blocks, us (1.0 = full mask): 10000 x 3000 of 3 MCUs, 1.0: 57 and 158, 0.15: 56 and 81; 12000 x 10000 of 100 MCUs, 1.0:
// 193 and 266, 0.7: 185 and 204, 0.5: 186 and 159; 8000 x 7680 of 256 MCUs, 1.0: 102 and 105, 0.7:
// 94 and 75; 1568 x 3000 of 100 MCUs, 1.0: 9.7 and 10.2, 0.7: 9.5 and 8.6; 3000 x 1650 of 33 MCUs,
// 1.0: 12.5 and 22.6, 0.5: 11.9 and 13.2; 1200 x 800 of 4 MCUs, 1.0: 4.4 and 10.1, 0.15: 4.3 and 3.8.
bool whole_matrix(const Geometry& g, int64_t n_active) {
    const int row = 4 * g.out_mcu, step = std::gcd(row, 128);
    const double lines = (row + 128 - step) / (double)row;            // (on average, over positions)
    const double share = lines * (double)n_active / ((double)g.in_hcu * g.out_hcu);
    const bool cached = (double)g.n_in * (double)g.n_out < 22e6;
    const double most = (cached ? 1.6 : 0.88) * (g.out_mcu % 4 == 0 ? 1.0 : 0.8);
    return share > most * std::max(1.0, 512.0 / (double)g.n_in) * std::max(1.0, 768.0 / (double)g.n_out);
}

}  // namespace

hipError_t launch_init_state(hipStream_t stream, const Geometry& g, const uint8_t* mask,
                             float pij0, float init_noise, uint64_t seed, int drop_bits,
                             float* pij, float* w) {
    init_state_kernel<<<sweep_blocks(g), kSweepThreads, 0, stream>>>(g, mask, pij0, init_noise,
                                                                      seed, drop_bits, pij, w);
    return hipGetLastError();
}

hipError_t launch_recompute_weights(hipStream_t stream, const Geometry& g, const uint8_t* mask,
                                    const int32_t* act_list, const int32_t* act_count,
                                    int32_t max_active, int64_t n_active, const float* pi,
                                    const float* pj, const float* pij, float eps, float bias_gain,
                                    int drop_bits, float* w, float* b, hipEvent_t start,
                                    hipEvent_t stop) {
    const int64_t n_bias = (g.n_out + kSweepThreads - 1) / kSweepThreads;
    if (whole_matrix(g, n_active) && g.n_in + n_bias < 1 << 24 &&
        g.n_out * g.out_mcu < 1ll << 31) {
        const uint32_t magic = (uint32_t)(((1ull << 31) + g.out_mcu - 1) / g.out_mcu);
        return launch_timed(g.n_out % 4 == 0 ? recompute_rows_kernel<4> : recompute_rows_kernel<1>,
                            dim3((unsigned)(g.n_in + n_bias)), dim3(kSweepThreads), 0, stream, start,
                            stop, g, mask, magic, pi, pj, pij, eps, bias_gain, drop_bits, w, b);
    }
    // 16 bytes per lane where every row segment is 16-byte aligned
    const int V = g.out_mcu % 4 == 0 && g.n_out % 4 == 0 ? 4 : 1;
    int lanes = 1;
    while (lanes < 64 && lanes * V < g.out_mcu) lanes *= 2;
    const int64_t rows = (int64_t)(kSweepThreads / lanes) * kWeightRows;
    const int64_t per_hcu = ((int64_t)max_active * g.in_mcu + rows - 1) / rows;
    const int64_t n_work = per_hcu * g.out_hcu;
    if (n_work + n_bias >= (1ll << 31)) return hipErrorInvalidValue;
    const int64_t cap = 1 << 22;                        // (a launch holds less than 2^32 work-items)
    const int64_t blocks = n_work + n_bias < cap ? n_work + n_bias : cap;
    const uint32_t magic = g.in_mcu > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)g.in_mcu - 1) /
                                                     (uint64_t)g.in_mcu)
                                        : 0;
    return launch_timed(V == 4 ? recompute_active_kernel<4> : recompute_active_kernel<1>,
                        dim3((unsigned)blocks), dim3(kSweepThreads), 0, stream, start, stop, g,
                        act_list, act_count, (uint32_t)per_hcu, (uint32_t)n_work, (uint32_t)n_bias,
                        lanes, magic, pi, pj, pij, eps, bias_gain, drop_bits, w, b);
}

hipError_t launch_bias(hipStream_t stream, const Geometry& g, const float* pj, float eps,
                       float bias_gain, float* b) {
    bias_kernel<<<(unsigned)((g.n_out + kSweepThreads - 1) / kSweepThreads), kSweepThreads, 0,
                  stream>>>(g.n_out, pj, eps, bias_gain, b);
    return hipGetLastError();
}

hipError_t launch_apply_mask(hipStream_t stream, const Geometry& g, const uint8_t* mask,
                             float* w) {
    apply_mask_kernel<<<sweep_blocks(g), kSweepThreads, 0, stream>>>(g, mask, w);
    return hipGetLastError();
}

}  // namespace bcpnn
