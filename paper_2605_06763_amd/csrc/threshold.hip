// Built-in threshold selection (appendix "Threshold Oracle Comparison"): a reservoir of R <= 256
// past keys per (sequence, KV head), kept uniform by reservoir sampling, and tau estimated from
// the query's dot products with it.
//
// Reservoir sampling in parallel.  Algorithm R processes positions in arrival order: position
// i < R fills slot i; position i >= R draws j uniform in [0, i] and overwrites slot j if j < R.
// The final occupant of a slot is therefore the LARGEST position that chose it, so any batch of
// positions can be handled by independent threads with an atomic max per accepted draw.  The
// draw is a counter-based hash of (seed, stream = sequence*H_kv + KV head, position): the
// splitmix64 finaliser, top 32 bits, j = floor(hash * (i+1) / 2^32).
#include "lvr_internal.h"

namespace {

__device__ __forceinline__ uint32_t hash32(uint64_t seed, uint64_t stream, uint64_t counter) {
    uint64_t z = seed + stream * 0xD1B54A32D192ED03ull + counter * 0x9E3779B97F4A7C15ull;
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (uint32_t)(z >> 32);
}

__global__ void reservoir_reset_kernel(int32_t *res, int total) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < total) res[i] = -1;
}

__global__ void reservoir_update_kernel(int32_t *res, int R, uint64_t seed, int64_t pos0, int64_t count) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int bh = blockIdx.y;
    const int64_t i = pos0 + k;
    int64_t j;
    if (i < R)
        j = i;
    else
        j = (int64_t)(((uint64_t)hash32(seed, (uint64_t)bh, (uint64_t)i) * (uint64_t)(i + 1)) >> 32);
    if (j < R) atomicMax(&res[(int64_t)bh * R + j], (int32_t)i);
}

// One 1024-thread workgroup per query head: scores of the reservoir keys (16 lanes per row), put in descending order,
// then the rule.  Bound by latency: positions, then rows, then the ordering.  A wave takes 16 slots: their positions come
// with one load and their rows are in flight together.  The order is found by counting: four threads per score compare it
// with a quarter of the 256 each (16 broadcast reads of LDS), and the score goes to the place its rank says.
// With four waves, a dependent load of position and row per four keys, a bitonic sort (36 barriers) and a serial count of
// the valid scores the launch took 28 us for 32 heads, with rows in flight and ranks but four waves 12.9; then 7.0 (threshold and step:
// 50.0, 33.6, 27.7 us).  With two instructions per compared pair instead of five the launch alone, 32 / 512 / 4096 heads: 6.4 / 11.2 / 65.9 -> 5.9 /
// 9.7 / 55.6 us (threshold and step: within what runs of one side differ by).  The gaps and the mean are taken by
// all threads: by one thread, 4096 heads, of which only two workgroups of 16 waves fit a compute unit, took 99.3 and 76.9 us
// where four waves each had taken 80.3 and 74.7; now 67.7 and 69.3.
template <typename KT>
__global__ void __launch_bounds__(1024)
threshold_kernel(const void *__restrict__ K, const int32_t *__restrict__ pos_slot, const int32_t *__restrict__ res,
                 const float *__restrict__ q, float *__restrict__ tau_out, int R, int64_t cap_rows, int64_t n_total,
                 int n_q_heads, int n_kv_heads, int G, int mode, float param) {
    __shared__ __align__(16) uint32_t s_key[256];
    __shared__ int s_rank[4][256];
    __shared__ float s[256];
    __shared__ float s_gap[4];
    __shared__ int s_at[4];
    __shared__ double s_sum[4];
    const int64_t hq = blockIdx.x;
    const int b = (int)(hq / n_q_heads), h = (int)(hq % n_q_heads);
    const int bh = b * n_kv_heads + h / G;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, sub = lane >> 4, li = lane & 15;
    const int32_t *rb = res + (int64_t)bh * R;
    const int32_t *pslot = pos_slot ? pos_slot + (int64_t)bh * cap_rows : nullptr;
    // lane li of every quarter holds the arena row of the wave's slot li
    const int mine = wave * 16 + li;
    const int pos = mine < R ? rb[mine] : -1;
    const bool have = pos >= 0 && pos < n_total;
    const int slot = have ? (pslot ? pslot[pos] : pos) : -1;
    float qv[8];
    {
        const float *qh = q + hq * LVR_D + li * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[e] = qh[e];
    }
    const char *Kb = static_cast<const char *>(K) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    lvr_raw8<KT> raw[4];
    int row[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        row[i] = __shfl(slot, 4 * i + sub, 64);
        lvr_load_raw(Kb, row[i] < 0 ? 0 : row[i], li, raw[i]);   // row 0 is part of the arena whatever it holds
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x[8];
        lvr_unpack(raw[i], x);
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) d += qv[e] * x[e];
        d = lvr_row16_sum(d);
        // unsigned keys in the order of the floats
        const uint32_t bits = __float_as_uint(row[i] >= 0 ? d : -INFINITY);
        if (li == 0) s_key[wave * 16 + 4 * i + sub] = bits ^ ((bits >> 31) ? 0xffffffffu : 0x80000000u);
    }
    __syncthreads();
    // descending order, equal scores in the order of their slots
    const int j = t & 255, quarter = __builtin_amdgcn_readfirstlane(t >> 8);
    const uint32_t key = s_key[j];
    {
        int rank = 0;
        auto count = [&](auto before) {   // before(o, i): score i comes before this thread's
#pragma unroll
            for (int i = quarter * 64; i < quarter * 64 + 64; i += 4) {
                const uint4 o = *reinterpret_cast<const uint4 *>(&s_key[i]);
                rank += before(o.x, i) ? 1 : 0;
                rank += before(o.y, i + 1) ? 1 : 0;
                rank += before(o.z, i + 2) ? 1 : 0;
                rank += before(o.w, i + 3) ? 1 : 0;
            }
        };
        // the slots of a quarter lie all below, all above or among those of a wave's threads: two instructions per pair instead of five
        const int mine = __builtin_amdgcn_readfirstlane(j >> 6);
        if (quarter < mine) count([&](uint32_t o, int) { return o >= key; });
        else if (quarter > mine) count([&](uint32_t o, int) { return o > key; });
        else count([&](uint32_t o, int i) { return o > key || (o == key && i < j); });
        s_rank[quarter][j] = rank;
    }
    const float score = __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xffffffffu));
    const int m = __syncthreads_count(t < 256 && score != -INFINITY);   // valid scores come first
    if (t < 256) s[s_rank[0][t] + s_rank[1][t] + s_rank[2][t] + s_rank[3][t]] = score;
    __syncthreads();
    if (mode == LVR_TAU_SAMPLE_GAP) {   // uniform: the first of the largest gaps of every wave of 64 (a gap that is no number counts for none)
        float gap = -1.0f;
        if (t < 256 && t + 1 < m) {
            const float g = s[t] - s[t + 1];
            if (g > gap) gap = g;
        }
        float most = gap;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) most = fmaxf(most, __shfl_xor(most, off, 64));
        const int at = __builtin_ctzll(__ballot(gap == most));   // some lane holds the maximum
        if (lane == 0 && wave < 4) {
            s_gap[wave] = most;
            s_at[wave] = wave * 64 + at;
        }
        __syncthreads();
    } else if (mode == LVR_TAU_SAMPLE_MEAN_MAX) {
        double sum = (t < 256 && t < m) ? (double)s[t] : 0.0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0 && wave < 4) s_sum[wave] = sum;
        __syncthreads();
    }
    if (t == 0) {
        float tau = -INFINITY;
        if (m > 0) {
            tau = s[0];
            if (mode == LVR_TAU_SAMPLE_MEAN_MAX) {
                const double sum = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
                tau = (float)(0.5 * ((double)s[0] + sum / (double)m));
            } else if (mode == LVR_TAU_SAMPLE_GAP) {
                int best = 0;
                float gap = -1.0f;
                for (int w = 0; w < 4; ++w) {
                    if (s_gap[w] > gap) {
                        gap = s_gap[w];
                        best = s_at[w];
                    }
                }
                tau = s[best];
            } else if (mode == LVR_TAU_SAMPLE_TOPK || mode == LVR_TAU_BUDGET) {
                int k = mode == LVR_TAU_SAMPLE_TOPK ? (int)param : (int)ceil((double)param * (double)m);
                if (k < 1) k = 1;
                if (k > m) k = m;
                tau = s[k - 1];
            }
        }
        tau_out[hq] = tau;
    }
}

}  // namespace

hipError_t lvr_launch_reservoir_reset(lvr_index *ix, hipStream_t st) {
    if (!ix->reservoir) return hipSuccess;
    const int total = lvr_n_bh(ix) * ix->cfg.reservoir_size;
    hipLaunchKernelGGL(reservoir_reset_kernel, dim3((total + 255) / 256), dim3(256), 0, st, ix->reservoir, total);
    return hipGetLastError();
}

hipError_t lvr_launch_reservoir_update(lvr_index *ix, int64_t pos0, int64_t count, hipStream_t st) {
    if (!ix->reservoir || count <= 0) return hipSuccess;
    dim3 grid((unsigned)((count + 255) / 256), (unsigned)lvr_n_bh(ix));
    hipLaunchKernelGGL(reservoir_update_kernel, grid, dim3(256), 0, st, ix->reservoir, ix->cfg.reservoir_size,
                       (uint64_t)ix->cfg.seed, pos0, count);
    return hipGetLastError();
}

hipError_t lvr_launch_threshold(lvr_index *ix, const float *q, int mode, float param, float *tau_out, hipStream_t st) {
    const int n_bhq = lvr_n_bhq(ix);
    if (ix->cfg.kv_dtype == LVR_BF16)
        hipLaunchKernelGGL(threshold_kernel<lvr_bf16_t>, dim3((unsigned)n_bhq), dim3(1024), 0, st, ix->K, ix->pos_slot,
                           ix->reservoir, q, tau_out, ix->cfg.reservoir_size, ix->cap_rows, ix->n_total,
                           ix->cfg.n_q_heads, ix->cfg.n_kv_heads, ix->G, mode, param);
    else
        hipLaunchKernelGGL(threshold_kernel<lvr_f32_t>, dim3((unsigned)n_bhq), dim3(1024), 0, st, ix->K, ix->pos_slot,
                           ix->reservoir, q, tau_out, ix->cfg.reservoir_size, ix->cap_rows, ix->n_total,
                           ix->cfg.n_q_heads, ix->cfg.n_kv_heads, ix->G, mode, param);
    return hipGetLastError();
}
