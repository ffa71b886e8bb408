// Initial state, weight recompute, mask application.
//
// Initial state and mask application are whole-matrix passes: each workgroup takes one row i of the
// [N_in][N_out] matrices per iteration of a grid-stride loop over rows; within a row the lanes walk
// consecutive columns, so every wave touches contiguous spans.  The mask row [out_hcu] of the row's
// input HCU is read through the cache.
//
// The weight recompute (Alg. 1 weight and mask lines) touches the active blocks only.  A silent
// weight is 0, and every writer of w keeps it so: the initial state, the upload (apply_mask_kernel),
// the structural update (which zeroes what it silences) and the batches (which write active blocks).
// Rewriting those zeros was 95% of the pass on the STL-shaped layer: with its reads coming from HBM
// between the stores, 690 us (2.3 GB, 3.4 TB/s; 390 us when the reads are repeated and stay in the
// Infinity Cache), against 54 us for the 221 MB of the active blocks.
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
        const int r0 = (work % per_hcu) * rows_at_once * kWeightRows + threadIdx.x / lanes;
        const int c0 = V * (threadIdx.x & (lanes - 1));
        const int k_total = act_count[hj] * g.in_mcu;
        if (r0 >= k_total) continue;
        const int32_t* list = act_list + (int64_t)hj * g.in_hcu;
        const int64_t col0 = (int64_t)hj * g.out_mcu;
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
            for (int q = 0; q < kWeightRows; ++q) p[q] = *reinterpret_cast<const vec*>(pij + row[q] + c);
#pragma unroll
            for (int q = 0; q < kWeightRows; ++q) {
                if (r0 + rows_at_once * q >= k_total) continue;
                vec v;
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = round_storage(log_ratio(p[q][e], pr[q], pc[e], eps), drop);
                *reinterpret_cast<vec*>(w + row[q] + c) = v;
            }
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

}  // namespace

hipError_t launch_init_state(hipStream_t stream, const Geometry& g, const uint8_t* mask,
                             float pij0, float init_noise, uint64_t seed, int drop_bits,
                             float* pij, float* w) {
    init_state_kernel<<<sweep_blocks(g), kSweepThreads, 0, stream>>>(g, mask, pij0, init_noise,
                                                                      seed, drop_bits, pij, w);
    return hipGetLastError();
}

hipError_t launch_recompute_weights(hipStream_t stream, const Geometry& g, const int32_t* act_list,
                                    const int32_t* act_count, int32_t max_active, const float* pi,
                                    const float* pj, const float* pij, float eps, float bias_gain,
                                    int drop_bits, float* w, float* b, hipEvent_t start,
                                    hipEvent_t stop) {
    // 16 bytes per lane where every row segment is 16-byte aligned
    const int V = g.out_mcu % 4 == 0 && g.n_out % 4 == 0 ? 4 : 1;
    int lanes = 1;
    while (lanes < 64 && lanes * V < g.out_mcu) lanes *= 2;
    const int64_t rows = (int64_t)(kSweepThreads / lanes) * kWeightRows;
    const int64_t per_hcu = ((int64_t)max_active * g.in_mcu + rows - 1) / rows;
    const int64_t n_work = per_hcu * g.out_hcu;
    const int64_t n_bias = (g.n_out + kSweepThreads - 1) / kSweepThreads;
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
