// Attention kernels.
//
//  sparse_attention_kernel attention restricted to a per-head index list (Sec. 2 "Sparse
//                         Attention"; App. "GPU Sparse Attention Kernel"): the list is cut into
//                         P splits, each wave gathers its K and V rows (256 B each for bf16),
//                         keeps running softmax statistics (m, l) and an fp32 accumulator o, and the
//                         last workgroup of a head merges the partial triples into the output.
//  dense_partial_kernel   the dense baseline (Sec. 2 "Attention"): every held key, contiguous
//                         streaming, the G query heads of a KV head served from one read.
//  carried_split_kernel   the same over lists that carry their scores, partials only.
//  combine_kernel         merges the P partial triples (m_p, l_p, o_p) into the output.
//
// Logits are taken in base-2 units (sigma * log2 e) so the exponentials are single exp2 instructions; the softmax is
// unchanged by the change of base.  Where a kernel forms the scores itself, q is pre-multiplied by that factor.  A raw score
// that is carried to it meets the factor and the running maximum in one fused multiply-add: a product of its own would
// be rounded at the size of the logit, the difference is rounded at its own (and how the maximum is rounded does not
// matter, all weights share it).
#include <hip/hip_ext.h>

#include "mfma_score.h"

namespace {

constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float exp2_safe(float a, float b) {   // 2^(a-b) with (-inf) - (-inf) -> 0
    return (a == -INFINITY) ? 0.f : exp2f(a - b);
}
__device__ __forceinline__ float exp2_carried(float score, float unit, float m) {   // 2^(score * unit - m), 0 for score -inf
    return (score == -INFINITY) ? 0.f : exp2f(__builtin_fmaf(score, unit, -m));
}

// Split geometry of the sparse attention: 16 entries per split (one gather batch) while the
// list fits in P_max splits, longer splits otherwise.  Returns the split length; *used = splits
// that hold entries.  carried_split_kernel and combine_kernel derive it from the same count.
__device__ __forceinline__ int64_t split_length(int64_t cnt, int P_max, int *used) {
    int64_t L = (((cnt + P_max - 1) / P_max) + 15) & ~(int64_t)15;
    if (L < 16) L = 16;
    *used = (int)((cnt + L - 1) / L);
    return L;
}

// One wave per part of a head's list, four waves to a workgroup, up to 64 workgroups.  The split's positions are fetched with one
// coalesced load, then rows are gathered 16 at a time (K and V of four row-quads in flight together).  A workgroup merges
// its waves in LDS; where a list fills more than one workgroup each of them stores its (m, l, o) and takes a ticket, and the one that
// draws the last merges them all, which saves the launch that used to do it.  A fence per workgroup that makes everything written so far visible would cost
// more than that launch on this multi-die part; here only the partials cross from one die to another: they are stored and
// read with accesses of device scope, and a workgroup waits for its own stores before it takes the ticket.  Every workgroup of
// a head takes one, whatever its share, and the counter wraps at their number (every number has a word of its own): it is back at zero
// after every launch, and after any set of launches that overlapped against the rules.
// us per call, a launch per stage and now, 80 / 330 / 1300 entries per head: 32 bf16 heads 7.4 / 7.8 / 9.6 and 5.7 / 6.1 / 8.4, 64 fp32 heads 8.9 /
// 11.0 / 20.3 and 7.8 / 8.8 / 19.6, 256 bf16 heads 14.0 / 16.3 / - and 8.2 / 13.3 / -.  (Workgroups of 16 waves: 32 bf16 heads 5.0 / 7.8 / 10.9.)
// 4000 / 8000 / 30000 entries, with room for as many: 32 bf16 heads 16.5 / 24.4 / 59.8 and 15.1 / 22.9 / 58.0, 32 fp32 heads 25.5 / 42.8 / 144.3 and
// 24.1 / 41.7 / 150 (142 to 150), one fp32 head 10.5 / 14.7 / 64.3 and 8.7 / 9.8 / 24.8.
// publish_count != NULL: the ticket's last also hands the head's counter over and clears it.
constexpr int SPLIT_WAVES = 4, SPLIT_WGS_MAX = 64;   // 64 x 4: as many splits as lvr_create takes; a wave's lanes hold the partials' weights

template <typename KT>
__global__ void __launch_bounds__(64 * SPLIT_WAVES)
sparse_attention_kernel(const int32_t *count, const int32_t *__restrict__ idx,   // count may alias head_count: not restrict
                        const float *__restrict__ q, const void *__restrict__ V, int64_t cap, int count_stride, int P,
                        int cap_rows, int n_total, int G, float qscale, const void *__restrict__ K,
                        const int32_t *__restrict__ pos_slot, float *part_ml, float *part_o, int32_t *ticket, float *__restrict__ out,
                        int32_t *head_count, int32_t *__restrict__ head_stat, int32_t *__restrict__ publish_count) {
    __shared__ float s_m[SPLIT_WAVES], s_l[SPLIT_WAVES];
    __shared__ float s_o[SPLIT_WAVES][LVR_D];
    __shared__ unsigned s_arrived;
    const int64_t hq = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = blockIdx.x * SPLIT_WAVES + wave;   // this wave's split
    const int bh = (int)((uint32_t)hq / (uint32_t)G);   // (hq / H_q) * H_kv + (hq % H_q) / G with H_q = H_kv * G: one 32-bit division
    const int lane = threadIdx.x & 63, sub = lane >> 4, li = lane & 15;

    const int32_t *my_idx = idx + hq * cap;
    // The split geometry depends on the count, and the positions on the geometry: two dependent
    // loads before the first gather.  The common geometry (16 entries per split) is assumed for a
    // speculative load of the positions that goes out together with the count.
    const int64_t e_spec = (int64_t)p * 16 + lane;
    const int32_t pos_spec = (lane < 16 && e_spec < cap) ? my_idx[e_spec] : -1;
    int64_t cnt = count[hq * count_stride];
    const int32_t true_cnt = (int32_t)cnt;
    if (cnt > cap) cnt = cap;
    if (cnt < 0) cnt = 0;
    int used;
    const int64_t L = split_length(cnt, P, &used);
    const int64_t start = (int64_t)p * L;
    const int64_t end = (start + L < cnt) ? start + L : cnt;   // past the splits in use: nothing

    float qv[8];
    {
        const float *qh = q + hq * LVR_D + li * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[e] = qh[e] * qscale;
    }
    const char *Kb = static_cast<const char *>(K) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const int32_t *pslot = pos_slot ? pos_slot + (int64_t)bh * cap_rows : nullptr;

    float m = -INFINITY, l = 0.f, acc[8];
    lvr_zero8(acc);
    for (int64_t c0 = start; c0 < end; c0 += 64) {          // uniform over the wave
        // positions of up to 64 entries, validated and mapped to arena rows once
        int64_t e = c0 + lane;
        int myslot = -1;
        if (e < end) {
            const int64_t pos = (L == 16) ? (int64_t)pos_spec : (int64_t)my_idx[e];
            if (pos >= 0 && pos < n_total) myslot = pslot ? pslot[pos] : (int)pos;
        }
        const int chunk = (int)((end - c0 < 64) ? end - c0 : 64);
        for (int b0 = 0; b0 < chunk; b0 += 16) {
            lvr_raw8<KT> kr[4], vr[4];
            int slot[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                slot[i] = __shfl(myslot, (b0 + i * 4 + sub) & 63, 64);
                if (b0 + i * 4 + sub >= chunk) slot[i] = -1;
                const int64_t sl = slot[i] < 0 ? 0 : slot[i];
                lvr_load_raw(Kb, sl, li, kr[i]);
                lvr_load_raw(Vb, sl, li, vr[i]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float vx[8];
                lvr_unpack(vr[i], vx);
                float kx[8];
                lvr_unpack(kr[i], kx);
                float d = 0.f;
#pragma unroll
                for (int c = 0; c < 8; ++c) d += qv[c] * kx[c];
                float s = lvr_row16_sum(d);
                s = (slot[i] >= 0) ? s : -INFINITY;
                const float m_new = fmaxf(m, s);
                const float alpha = exp2_safe(m, m_new);
                const float w = exp2_safe(s, m_new);
                l = l * alpha + w;
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] = acc[c] * alpha + w * vx[c];
                m = m_new;
            }
        }
    }
    // merge the four quarter rows of the wave, then the waves
    float m_all = fmaxf(m, __shfl_xor(m, 16, 64));
    m_all = fmaxf(m_all, __shfl_xor(m_all, 32, 64));
    const float sc = exp2_safe(m, m_all);
    l *= sc;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float a = acc[c] * sc;
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (sub == 0) s_o[wave][li * 8 + c] = a;
    }
    if (lane == 0) {
        s_m[wave] = m_all;
        s_l[wave] = l;
    }
    __syncthreads();
    const int wgs = (int)gridDim.x, used_wgs = (used + SPLIT_WAVES - 1) / SPLIT_WAVES;
    const int ch = threadIdx.x & (LVR_D - 1), slice = threadIdx.x >> 7;
    float M = -INFINITY, num = 0.f, den = 0.f;
    if (slice == 0) {
#pragma unroll
        for (int w = 0; w < SPLIT_WAVES; ++w) M = fmaxf(M, s_m[w]);
#pragma unroll
        for (int w = 0; w < SPLIT_WAVES; ++w) {
            const float wt = exp2_safe(s_m[w], M);
            den += wt * s_l[w];
            num += wt * s_o[w][ch];
        }
    }
    if (used_wgs <= 1) {   // uniform over the head's workgroups: the first one holds all of the list
        if (blockIdx.x == 0 && slice == 0) out[hq * LVR_D + ch] = (den > 0.f && M != -INFINITY) ? num / den : 0.f;
        if (!publish_count) return;
    } else if ((int)blockIdx.x < used_wgs && slice == 0) {
        __hip_atomic_store(&part_o[(hq * wgs + blockIdx.x) * LVR_D + ch], num, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ch == 0) {
            __hip_atomic_store(&part_ml[(hq * wgs + blockIdx.x) * 2], M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&part_ml[(hq * wgs + blockIdx.x) * 2 + 1], den, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have reached the memory all compute units share
    __syncthreads();
    if (threadIdx.x == 0) s_arrived = atomicInc(reinterpret_cast<unsigned *>(&ticket[hq * LVR_CNT_STRIDE]), (unsigned)wgs - 1u);
    __syncthreads();
    if (s_arrived != (unsigned)wgs - 1u) return;
    // every workgroup of the head has its partial in memory and has read the count
    if (publish_count && threadIdx.x == 0) {
        publish_count[hq] = true_cnt;
        head_stat[hq] = true_cnt;
        head_count[hq * LVR_CNT_STRIDE] = 0;
    }
    if (used_wgs <= 1) return;
    auto load = [](const float *x) { return __hip_atomic_load(x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // lane p of every wave holds the weight of partial p
    const float m_p = lane < used_wgs ? load(&part_ml[(hq * wgs + lane) * 2]) : -INFINITY;
    const float l_p = lane < used_wgs ? load(&part_ml[(hq * wgs + lane) * 2 + 1]) : 0.f;
    const float *po = part_o + hq * wgs * LVR_D + ch;
    constexpr int SLICES = SPLIT_WAVES / 2, EACH = 8;   // a slice takes every other partial, eight loads in flight
    float pv[EACH];
#pragma unroll
    for (int i = 0; i < EACH; ++i) pv[i] = SLICES * i + slice < used_wgs ? load(&po[(SLICES * i + slice) * LVR_D]) : 0.f;
    M = m_p;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    const float w_p = exp2_safe(m_p, M);
    den = w_p * l_p;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) den += __shfl_xor(den, off, 64);
    num = 0.f;
#pragma unroll
    for (int i = 0; i < EACH; ++i) num += __shfl(w_p, SLICES * i + slice, 64) * pv[i];   // past the partials in use: zero times zero
    for (int p0 = SLICES * EACH; p0 < used_wgs; p0 += SLICES * EACH) {   // uniform
#pragma unroll
        for (int i = 0; i < EACH; ++i) pv[i] = p0 + SLICES * i + slice < used_wgs ? load(&po[(p0 + SLICES * i + slice) * LVR_D]) : 0.f;
#pragma unroll
        for (int i = 0; i < EACH; ++i) num += __shfl(w_p, p0 + SLICES * i + slice, 64) * pv[i];
    }
    s_o[slice][ch] = num;
    __syncthreads();
    if (slice == 0) {
#pragma unroll
        for (int i = 1; i < SLICES; ++i) num += s_o[i][ch];
        out[hq * LVR_D + ch] = (den > 0.f && M != -INFINITY) ? num / den : 0.f;
    }
}

// Lists that carry their raw scores (written by the query kernel that made them) and are too long for the one-launch forms
// below: one wave per (query head, split), the partials merged by combine_kernel.  The split's positions and scores are fetched with
// one coalesced load each, then V rows are gathered 16 at a time.
template <typename KT>
__global__ void __launch_bounds__(64)
carried_split_kernel(const int32_t *__restrict__ count, const int32_t *__restrict__ idx, const float *__restrict__ scores,
                        const void *__restrict__ V, int64_t cap, int count_stride, int P,
                        int cap_rows, int n_total, int G, float qscale, const int32_t *__restrict__ pos_slot, float *__restrict__ part_ml, float *__restrict__ part_o) {
    const int64_t hq = blockIdx.y;
    const int p = blockIdx.x;
    const int bh = (int)((uint32_t)hq / (uint32_t)G);   // (hq / H_q) * H_kv + (hq % H_q) / G with H_q = H_kv * G: one 32-bit division
    const int lane = threadIdx.x & 63, sub = lane >> 4, li = lane & 15;

    const int32_t *my_idx = idx + hq * cap;
    // The split geometry depends on the count, and the positions on the geometry: two dependent
    // loads before the first gather.  The common geometry (16 entries per split) is assumed for a
    // speculative load of the positions that goes out together with the count.
    const int64_t e_spec = (int64_t)p * 16 + lane;
    const int32_t pos_spec = (lane < 16 && e_spec < cap) ? my_idx[e_spec] : -1;
    const float *my_sc = scores + hq * (int64_t)cap_rows;
    const float sc_spec = (lane < 16 && e_spec < cap && e_spec < cap_rows) ? my_sc[e_spec] : 0.f;
    int64_t cnt = count[hq * count_stride];
    if (cnt > cap) cnt = cap;
    if (cnt < 0) cnt = 0;
    int used;
    const int64_t L = split_length(cnt, P, &used);
    if (p >= used) return;     // the combine pass reads only the `used` partials
    const int64_t start = (int64_t)p * L;
    const int64_t end = (start + L < cnt) ? start + L : cnt;

    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const int32_t *pslot = pos_slot ? pos_slot + (int64_t)bh * cap_rows : nullptr;

    float m = -INFINITY, l = 0.f, acc[8];
    lvr_zero8(acc);
    for (int64_t c0 = start; c0 < end; c0 += 64) {          // uniform over the wave
        // positions of up to 64 entries, validated and mapped to arena rows once
        int64_t e = c0 + lane;
        int myslot = -1;
        float myscore = 0.f;
        if (e < end) {
            const int64_t pos = (L == 16) ? (int64_t)pos_spec : (int64_t)my_idx[e];
            myscore = (L == 16) ? sc_spec : my_sc[e];
            if (pos >= 0 && pos < n_total) myslot = pslot ? pslot[pos] : (int)pos;
        }
        const int chunk = (int)((end - c0 < 64) ? end - c0 : 64);
        for (int b0 = 0; b0 < chunk; b0 += 16) {
            lvr_raw8<KT> vr[4];
            int slot[4];
            float given[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                slot[i] = __shfl(myslot, (b0 + i * 4 + sub) & 63, 64);
                given[i] = __shfl(myscore, (b0 + i * 4 + sub) & 63, 64);
                if (b0 + i * 4 + sub >= chunk) slot[i] = -1;
                const int64_t sl = slot[i] < 0 ? 0 : slot[i];
                lvr_load_raw(Vb, sl, li, vr[i]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float vx[8];
                lvr_unpack(vr[i], vx);
                const float s = (slot[i] >= 0) ? given[i] : -INFINITY;
                const float m_new = fmaxf(m, s * qscale);
                const float alpha = exp2_safe(m, m_new);
                const float w = exp2_carried(s, qscale, m_new);
                l = l * alpha + w;
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] = acc[c] * alpha + w * vx[c];
                m = m_new;
            }
        }
    }
    // merge the four quarter rows of the wave
    float m_all = fmaxf(m, __shfl_xor(m, 16, 64));
    m_all = fmaxf(m_all, __shfl_xor(m_all, 32, 64));
    const float sc = exp2_safe(m, m_all);
    l *= sc;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float a = acc[c] * sc;
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        acc[c] = a;
    }
    if (sub == 0) {
        float *o = part_o + (hq * P + p) * LVR_D + li * 8;
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] = acc[c];
        if (li == 0) {
            part_ml[(hq * P + p) * 2] = m_all;
            part_ml[(hq * P + p) * 2 + 1] = l;
        }
    }
}

// Sparse attention in ONE launch: a 1024-thread workgroup (16 waves) per query head.  Each wave
// takes a contiguous share of the head's index list exactly as sparse_attention_kernel does,
// then the 16 partial triples are merged through LDS, so no partials travel through HBM and no
// combine launch follows.  Thread 0 also publishes (and clears) the head's internal counter
// when asked to.
template <typename KT>
__global__ void __launch_bounds__(1024)
sparse_attention_wg_kernel(const void *__restrict__ K, const void *__restrict__ V,
                           const int32_t *__restrict__ pos_slot, const float *__restrict__ q,
                           const int32_t *__restrict__ idx, const int32_t *count, int count_stride,   // may alias head_count: not restrict
                           int64_t cap, float *__restrict__ out, int64_t cap_rows, int64_t n_total, int n_q_heads,
                           int n_kv_heads, int G, float qscale, int32_t *head_count,
                           int32_t *__restrict__ head_stat, int32_t *__restrict__ publish_count) {
    constexpr int NW = 16;
    __shared__ float s_m[NW], s_l[NW];
    __shared__ float s_o[NW][LVR_D];
    const int64_t hq = blockIdx.x;
    const int bh = (int)((uint32_t)hq / (uint32_t)G);   // (hq / H_q) * H_kv + (hq % H_q) / G with H_q = H_kv * G: one 32-bit division
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane >> 4, li = lane & 15;

    int64_t cnt = count[hq * count_stride];
    const int32_t true_cnt = (int32_t)cnt;
    if (cnt > cap) cnt = cap;
    if (cnt < 0) cnt = 0;
    const int64_t L = (((cnt + NW - 1) / NW) + 15) & ~(int64_t)15;
    const int64_t start = (int64_t)wave * L;
    const int64_t end = (start + L < cnt) ? start + L : cnt;

    float qv[8];
    {
        const float *qh = q + hq * LVR_D + li * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[e] = qh[e] * qscale;
    }
    const char *Kb = static_cast<const char *>(K) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const int32_t *my_idx = idx + hq * cap;
    const int32_t *pslot = pos_slot ? pos_slot + (int64_t)bh * cap_rows : nullptr;

    float m = -INFINITY, l = 0.f, acc[8];
    lvr_zero8(acc);
    for (int64_t c0 = start; c0 < end; c0 += 64) {          // uniform over the wave
        int64_t e = c0 + lane;
        int myslot = -1;
        if (e < end) {
            const int64_t pos = my_idx[e];
            if (pos >= 0 && pos < n_total) myslot = pslot ? pslot[pos] : (int)pos;
        }
        const int chunk = (int)((end - c0 < 64) ? end - c0 : 64);
        for (int b0 = 0; b0 < chunk; b0 += 16) {
            lvr_raw8<KT> kr[4], vr[4];
            int slot[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                slot[i] = __shfl(myslot, (b0 + i * 4 + sub) & 63, 64);
                if (b0 + i * 4 + sub >= chunk) slot[i] = -1;
                const int64_t sl = slot[i] < 0 ? 0 : slot[i];
                lvr_load_raw(Kb, sl, li, kr[i]);
                lvr_load_raw(Vb, sl, li, vr[i]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float kx[8], vx[8];
                lvr_unpack(kr[i], kx);
                lvr_unpack(vr[i], vx);
                float d = 0.f;
#pragma unroll
                for (int c = 0; c < 8; ++c) d += qv[c] * kx[c];
                float s = lvr_row16_sum(d);
                s = (slot[i] >= 0) ? s : -INFINITY;
                const float m_new = fmaxf(m, s);
                const float alpha = exp2_safe(m, m_new);
                const float w = exp2_safe(s, m_new);
                l = l * alpha + w;
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] = acc[c] * alpha + w * vx[c];
                m = m_new;
            }
        }
    }
    float m_all = fmaxf(m, __shfl_xor(m, 16, 64));
    m_all = fmaxf(m_all, __shfl_xor(m_all, 32, 64));
    const float sc = exp2_safe(m, m_all);
    l *= sc;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float a = acc[c] * sc;
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (sub == 0) s_o[wave][li * 8 + c] = a;
    }
    if (lane == 0) {
        s_m[wave] = m_all;
        s_l[wave] = l;
    }
    __syncthreads();
    if (threadIdx.x < LVR_D) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wt = exp2_safe(s_m[w], M);
            den += wt * s_l[w];
            num += wt * s_o[w][threadIdx.x];
        }
        out[hq * LVR_D + threadIdx.x] = (den > 0.f && M != -INFINITY) ? num / den : 0.f;
    }
    if (publish_count && threadIdx.x == 0) {
        publish_count[hq] = true_cnt;
        head_stat[hq] = true_cnt;
        head_count[hq * LVR_CNT_STRIDE] = 0;
    }
}

// The one-launch form for lists that carry their scores (the decode step): a workgroup of NW waves per head, with the
// dependent round trips to memory cut to two (fp32: three).
//   trip 1  the count AND the positions and scores of the first 64 NW list entries: which entries a lane asks for
//           does not depend on the count (lane (quarter s, j) of wave w asks for entry j of batch w + NW s, a batch
//           being 16 consecutive entries), what lies beyond the count is dropped when it arrives;
//   trip 2  the V rows of ALL the wave's batches (up to four: 16 rows per lane quarter in flight), then the
//           softmax update over them.  fp32 rows are twice as wide: two batches are in flight and the other two follow
//           as a third trip.
// sparse_attention_wg_kernel pays count -> positions -> one trip per batch: five in a row for 656 keys per head.
// Lists longer than 64 NW entries take further rounds of the same trips.
template <typename KT, int NW>
__global__ void __launch_bounds__(64 * NW)
sparse_attention_wg_carry_kernel(const int32_t *count,   // may alias head_count: not restrict
                                 const int32_t *__restrict__ idx, const float *__restrict__ scores, const void *__restrict__ V,
                                 int64_t cap, int count_stride, int cap_rows, int n_total, int G,
                                 const int32_t *__restrict__ pos_slot, float *__restrict__ out, float qscale, int32_t *head_count,
                                 int32_t *__restrict__ head_stat, int32_t *__restrict__ publish_count) {
    __shared__ float s_m[NW], s_l[NW];
    __shared__ float s_o[NW][LVR_D];
    const int64_t hq = blockIdx.x;
    const int bh = (int)((uint32_t)hq / (uint32_t)G);   // (hq / H_q) * H_kv + (hq % H_q) / G with H_q = H_kv * G: one 32-bit division
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane >> 4, li = lane & 15;
    const int32_t *my_idx = idx + hq * cap;
    const float *my_sc = scores + hq * (int64_t)cap_rows;
    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const int32_t *pslot = pos_slot ? pos_slot + (int64_t)bh * cap_rows : nullptr;

    // trip 1 (the count first: it is read through the scalar unit, whose argument loads and the read itself form a
    // chain of their own that should start before the vector loads are set up, not after)
    int64_t cnt = count[hq * count_stride];
    const int64_t e_rel = (int64_t)(wave + NW * sub) * 16 + li;   // this lane's entry within a round of 64 NW
    int32_t pos = (e_rel < cap) ? my_idx[e_rel] : -1;
    float sc = (e_rel < cap && e_rel < cap_rows) ? my_sc[e_rel] : 0.f;
    const int32_t true_cnt = (int32_t)cnt;
    if (cnt > cap) cnt = cap;
    if (cnt < 0) cnt = 0;

    // m and l are the same in all lanes of the wave; acc holds the partial sums of this lane quarter's rows
    float m = -INFINITY, l = 0.f, acc[8];
    lvr_zero8(acc);
    for (int64_t base = 0; base < cnt; base += NW * 64) {   // uniform over the workgroup
        const int64_t e = base + e_rel;
        if (base > 0) {
            pos = (e < cnt) ? my_idx[e] : -1;
            sc = (e < cnt && e < cap_rows) ? my_sc[e] : 0.f;
        }
        int myslot = -1;
        if (e < cnt && pos >= 0 && pos < n_total) myslot = pslot ? pslot[pos] : (int)pos;
        // trip 2: batch bq of this wave is entries base + (wave + NW bq) * 16 ..; row i * 4 + sub of it is held by lane 16 bq + i * 4 + sub.
        // All four batches are in flight; fp32 rows are twice as wide: two batches at a time fit the registers of 16 waves
        constexpr int NB = sizeof(KT) == sizeof(lvr_bf16_t) ? 4 : 2;
        lvr_raw8<KT> vr[NB * 4];
        bool have[4];
#pragma unroll
        for (int bq = 0; bq < 4; ++bq) {
            have[bq] = base + (int64_t)(wave + NW * bq) * 16 < cnt;   // wave-uniform
            if (bq < NB && have[bq]) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int sl = __shfl(myslot, 16 * bq + i * 4 + sub, 64);
                    lvr_load_raw(Vb, sl < 0 ? 0 : sl, li, vr[bq * 4 + i]);
                }
            }
        }
        if (!have[0]) continue;   // wave-uniform: none of this wave's batches holds an entry in this round
        // The scores are here already, so the softmax weights of all 64 entries are formed while the rows travel:
        // one maximum and one sum over the wave, one exponential per lane, instead of a chain of rescalings per row.
        const float s_e = (myslot >= 0) ? sc : -INFINITY;
        float mw = s_e;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mw = fmaxf(mw, __shfl_xor(mw, off, 64));
        const float m_new = fmaxf(m, mw * qscale);
        const float w_e = exp2_carried(s_e, qscale, m_new);
        float lw = w_e;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) lw += __shfl_xor(lw, off, 64);
        const float alpha = exp2_safe(m, m_new);
        l = l * alpha + lw;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] *= alpha;
        m = m_new;
#pragma unroll
        for (int bq = 0; bq < 4; ++bq) {
            if (have[bq]) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float w = __shfl(w_e, 16 * bq + i * 4 + sub, 64);   // 0 for a masked entry
                    float vx[8];
                    lvr_unpack(vr[(bq % NB) * 4 + i], vx);
#pragma unroll
                    for (int c = 0; c < 8; ++c) acc[c] += w * vx[c];
                }
            }
            if (NB < 4 && bq == NB - 1) {   // the other half of the batches
#pragma unroll
                for (int b2 = NB; b2 < 4; ++b2) {
                    if (have[b2]) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int sl = __shfl(myslot, 16 * b2 + i * 4 + sub, 64);
                            lvr_load_raw(Vb, sl < 0 ? 0 : sl, li, vr[(b2 % NB) * 4 + i]);
                        }
                    }
                }
            }
        }
    }
    const float m_all = m;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float a = acc[c];
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (sub == 0) s_o[wave][li * 8 + c] = a;
    }
    if (lane == 0) {
        s_m[wave] = m_all;
        s_l[wave] = l;
    }
    __syncthreads();
    if (threadIdx.x < LVR_D) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wt = exp2_safe(s_m[w], M);
            den += wt * s_l[w];
            num += wt * s_o[w][threadIdx.x];
        }
        out[hq * LVR_D + threadIdx.x] = (den > 0.f && M != -INFINITY) ? num / den : 0.f;
    }
    // every thread's read of the count lies before the barrier above, so the counter can be handed over and cleared
    if (publish_count && threadIdx.x == 0) {
        publish_count[hq] = true_cnt;
        head_stat[hq] = true_cnt;
        head_count[hq * LVR_CNT_STRIDE] = 0;
    }
}

// The same with SPLIT workgroups per head (SPLIT = 2), each responsible for one half of the channels: it reads one cache line of
// every V row (eight lanes per row instead of sixteen) and writes 64 of the 128 outputs.  Both form the same
// softmax weights from the carried scores, so nothing has to be merged between them; what one compute unit has to
// pull through its 64 bytes per clock halves.  The two take a ticket once all their threads hold the count; the
// one that draws the second ticket publishes the count and clears the head's counter when it ends.
template <typename KT, int SPLIT>
__global__ void __launch_bounds__(1024)
sparse_attention_wg_carry_split_kernel(const int32_t *count,   // may alias head_count: not restrict
                                 const int32_t *__restrict__ idx, const float *__restrict__ scores, const void *__restrict__ V,
                                 int64_t cap, int count_stride, int cap_rows, int n_total, int G,
                                 const int32_t *__restrict__ pos_slot, float *__restrict__ out, float qscale, int32_t *head_count,
                                 int32_t *__restrict__ head_stat, int32_t *__restrict__ publish_count,
                                 int32_t *__restrict__ ticket) {
    constexpr int NW = 16;
    constexpr int LPR = 16 / SPLIT;          // lanes per row (16 bytes each)
    constexpr int RPL = 64 / LPR;            // rows per load instruction of a wave
    constexpr int NLOAD = 64 / RPL;          // load instructions that cover a wave's 64 entries
    constexpr int CH = LVR_D / SPLIT;        // channels this workgroup is responsible for
    __shared__ float s_m[NW], s_l[NW];
    __shared__ float s_o[NW][CH];
    const int64_t hq = blockIdx.x / SPLIT;
    const int part = blockIdx.x % SPLIT;
    const int bh = (int)((uint32_t)hq / (uint32_t)G);   // (hq / H_q) * H_kv + (hq % H_q) / G with H_q = H_kv * G: one 32-bit division
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane >> 4, li = lane & 15;
    const int grp = lane / LPR, lp = lane % LPR;   // this lane's row within a load, its 16-byte piece of the row part
    const int32_t *my_idx = idx + hq * cap;
    const float *my_sc = scores + hq * (int64_t)cap_rows;
    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const int32_t *pslot = pos_slot ? pos_slot + (int64_t)bh * cap_rows : nullptr;

    // trip 1 (the count first: it is read through the scalar unit, whose argument loads and the read itself form a
    // chain of their own that should start before the vector loads are set up, not after)
    int64_t cnt = count[hq * count_stride];
    const int64_t e_rel = (int64_t)(wave + NW * sub) * 16 + li;   // this lane's entry within a round of 1024
    int32_t pos = (e_rel < cap) ? my_idx[e_rel] : -1;
    float sc = (e_rel < cap && e_rel < cap_rows) ? my_sc[e_rel] : 0.f;
    const int32_t true_cnt = (int32_t)cnt;
    if (cnt > cap) cnt = cap;
    if (cnt < 0) cnt = 0;
    int drawn = 0;
    if constexpr (SPLIT > 1) {
        // the empty statement consumes the loaded value, so every thread waits for its copy of the count before the
        // barrier; behind the barrier the workgroup may announce that it no longer needs the counter
        asm volatile("" ::"v"(true_cnt));
        __syncthreads();
        if (threadIdx.x == 0) drawn = atomicAdd(&ticket[hq], 1);
    }

    // m and l are the same in all lanes of the wave; acc holds the partial sums of this lane group's rows
    float m = -INFINITY, l = 0.f, acc[8];
    lvr_zero8(acc);
    for (int64_t base = 0; base < cnt; base += NW * 64) {   // uniform over the workgroup
        const int64_t e = base + e_rel;
        if (base > 0) {
            pos = (e < cnt) ? my_idx[e] : -1;
            sc = (e < cnt && e < cap_rows) ? my_sc[e] : 0.f;
        }
        int myslot = -1;
        if (e < cnt && pos >= 0 && pos < n_total) myslot = pslot ? pslot[pos] : (int)pos;
        // trip 2: load j of the wave fetches the rows of the entries held by lanes j * RPL .. j * RPL + RPL - 1 (row
        // grp of them is this lane's); those lanes belong to batch (j * RPL) / 16 of the wave, entries
        // base + (wave + 16 bq) * 16 ..
        lvr_raw8<KT> vr[NLOAD];
        bool have[4];
#pragma unroll
        for (int bq = 0; bq < 4; ++bq) have[bq] = base + (int64_t)(wave + NW * bq) * 16 < cnt;   // wave-uniform
#pragma unroll
        for (int j = 0; j < NLOAD; ++j) {
            if (have[(j * RPL) / 16]) {
                const int sl = __shfl(myslot, j * RPL + grp, 64);
                lvr_load_raw(Vb, sl < 0 ? 0 : sl, part * LPR + lp, vr[j]);
            }
        }
        if (!have[0]) continue;   // wave-uniform: none of this wave's batches holds an entry in this round
        // The scores are here already, so the softmax weights of all 64 entries are formed while the rows travel:
        // one maximum and one sum over the wave, one exponential per lane, instead of a chain of rescalings per row.
        const float s_e = (myslot >= 0) ? sc : -INFINITY;
        float mw = s_e;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mw = fmaxf(mw, __shfl_xor(mw, off, 64));
        const float m_new = fmaxf(m, mw * qscale);
        const float w_e = exp2_carried(s_e, qscale, m_new);
        float lw = w_e;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) lw += __shfl_xor(lw, off, 64);
        const float alpha = exp2_safe(m, m_new);
        l = l * alpha + lw;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] *= alpha;
        m = m_new;
#pragma unroll
        for (int j = 0; j < NLOAD; ++j) {
            if (have[(j * RPL) / 16]) {
                const float w = __shfl(w_e, j * RPL + grp, 64);   // 0 for a masked entry
                float vx[8];
                lvr_unpack(vr[j], vx);
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] += w * vx[c];
            }
        }
    }
    const float m_all = m;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float a = acc[c];
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) a += __shfl_xor(a, off, 64);
        if (grp == 0) s_o[wave][lp * 8 + c] = a;
    }
    if (lane == 0) {
        s_m[wave] = m_all;
        s_l[wave] = l;
    }
    __syncthreads();
    if (threadIdx.x < CH) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wt = exp2_safe(s_m[w], M);
            den += wt * s_l[w];
            num += wt * s_o[w][threadIdx.x];
        }
        out[hq * LVR_D + part * CH + threadIdx.x] = (den > 0.f && M != -INFINITY) ? num / den : 0.f;
    }
    // every thread's read of the count lies before a barrier above (in both workgroups of a split head once the
    // second ticket has been drawn), so the counter can be handed over and cleared
    if (publish_count && threadIdx.x == 0 && (SPLIT == 1 || drawn == SPLIT - 1)) {
        publish_count[hq] = true_cnt;
        head_stat[hq] = true_cnt;
        head_count[hq * LVR_CNT_STRIDE] = 0;
        if constexpr (SPLIT > 1) ticket[hq] = 0;
    }
}

// Merge of the partial triples of one query head.  512 threads: thread (slice s, channel c) owns
// every fourth partial of channel c; its values are requested first, then the weights
// w_p = 2^(m_p - M) are computed into LDS, the slices are weighted, and the four slices are
// added through LDS.  With a count pointer the number of partials in use follows the sparse
// attention's split geometry; without one all P are merged (dense baseline).
constexpr int COMBINE_MAX_P = 256;

// `count` and `head_count` may be the same array (the decode step hands the internal counters to
// both), so neither is declared restrict, every thread reads the count BEFORE the kernel's first
// barrier and the counter is cleared only AFTER it.
__global__ void __launch_bounds__(512)
combine_kernel(const float *__restrict__ part_o, const float *__restrict__ part_ml, const int32_t *count, int64_t cap,
               float *__restrict__ out, int P, int count_stride, int32_t *head_count,
               int32_t *__restrict__ head_stat, int32_t *__restrict__ publish_count) {
    __shared__ float s_w[COMBINE_MAX_P];
    __shared__ float s_red[8];
    __shared__ float s_num[4][LVR_D];
    const int64_t hq = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int c = t & (LVR_D - 1), sl = t >> 7;
    const float *po = part_o + hq * P * LVR_D + c;
    // up to 16 partials per thread (all of them for P <= 64) and the (m, l) pairs are requested
    // first, together with the count, so that nothing waits for a second trip to memory; what
    // lies beyond the partials in use is stale and is masked once the count has arrived
    float pv[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = sl + 4 * i;
        pv[i] = (p < P) ? po[(int64_t)p * LVR_D] : 0.f;
    }
    const float m_raw = (t < P) ? part_ml[(hq * P + t) * 2] : -INFINITY;
    const float l_raw = (t < P) ? part_ml[(hq * P + t) * 2 + 1] : 0.f;
    int used = P;
    int32_t true_cnt = 0;
    if (count) {
        int64_t cnt = count[hq * count_stride];
        true_cnt = (int32_t)cnt;
        if (cnt > cap) cnt = cap;
        if (cnt < 0) cnt = 0;
        split_length(cnt, P, &used);
    }
    const float m = (t < used) ? m_raw : -INFINITY;
    const float l = (t < used) ? l_raw : 0.f;
    float mx = m;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if (lane == 0) s_red[wave] = mx;
    __syncthreads();
    // every thread's read of the count has completed (its value fed the shuffle above), so the
    // counter can be handed over and cleared for the next query
    if (count && publish_count && t == 0) {
        publish_count[hq] = true_cnt;
        head_stat[hq] = true_cnt;
        head_count[hq * LVR_CNT_STRIDE] = 0;
    }
    float M = s_red[0];
#pragma unroll
    for (int w = 1; w < 8; ++w) M = fmaxf(M, s_red[w]);
    __syncthreads();
    const float w_p = exp2_safe(m, M);
    if (t < COMBINE_MAX_P) s_w[t] = w_p;
    float dn = w_p * l;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) dn += __shfl_xor(dn, off, 64);
    if (lane == 0) s_red[wave] = dn;
    __syncthreads();
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) den += s_red[w];
    float num = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = sl + 4 * i;
        num += (p < used) ? s_w[p] * pv[i] : 0.f;
    }
#pragma unroll 4
    for (int p = sl + 64; p < used; p += 4) num += s_w[p] * po[(int64_t)p * LVR_D];
    s_num[sl][c] = num;
    __syncthreads();
    if (t < LVR_D) {
        const float tot = s_num[0][t] + s_num[1][t] + s_num[2][t] + s_num[3][t];
        out[hq * LVR_D + t] = (den > 0.f && M != -INFINITY) ? tot / den : 0.f;
    }
}

template <typename KT, int G>
__global__ void __launch_bounds__(256)
dense_partial_kernel(const void *__restrict__ K, const void *__restrict__ V, const float *__restrict__ q,
                     float *__restrict__ part_ml, float *__restrict__ part_o, int64_t cap_rows, int64_t n_total,
                     int P, int n_q_heads, int n_kv_heads, float qscale) {
    __shared__ float sm_m[4][G], sm_l[4][G];
    __shared__ float sm_o[4][G][LVR_D];
    const int bh = blockIdx.y, p = blockIdx.x;
    const int b = bh / n_kv_heads, kvh = bh % n_kv_heads;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = lane >> 4, li = lane & 15;
    const int64_t hq0 = (int64_t)b * n_q_heads + kvh * G;

    const int64_t R = (((n_total + P - 1) / P) + 15) & ~(int64_t)15;
    const int64_t start = (int64_t)p * R;
    const int64_t end = (start + R < n_total) ? start + R : n_total;

    float qv[G][8];
#pragma unroll
    for (int h = 0; h < G; ++h) {
        const float *qh = q + (hq0 + h) * LVR_D + li * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[h][e] = qh[e] * qscale;
    }
    const char *Kb = static_cast<const char *>(K) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);

    float m[G], l[G], acc[G][8];
#pragma unroll
    for (int h = 0; h < G; ++h) {
        m[h] = -INFINITY;
        l[h] = 0.f;
        lvr_zero8(acc[h]);
    }
    for (int64_t r0 = start + wave * 4; r0 < end; r0 += 16) {   // uniform over the wave
        const int64_t row = r0 + sub;
        const bool valid = row < end;
        const int64_t rc = valid ? row : 0;
        float kx[8], vx[8];
        lvr_load8<KT>(Kb, rc, li, kx);
        lvr_load8<KT>(Vb, rc, li, vx);
#pragma unroll
        for (int h = 0; h < G; ++h) {
            float d = 0.f;
#pragma unroll
            for (int c = 0; c < 8; ++c) d += qv[h][c] * kx[c];
            float s = lvr_row16_sum(d);
            s = valid ? s : -INFINITY;
            const float m_new = fmaxf(m[h], s);
            const float alpha = exp2_safe(m[h], m_new);
            const float w = exp2_safe(s, m_new);
            l[h] = l[h] * alpha + w;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[h][c] = acc[h][c] * alpha + w * vx[c];
            m[h] = m_new;
        }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
        float m_all = fmaxf(m[h], __shfl_xor(m[h], 16, 64));
        m_all = fmaxf(m_all, __shfl_xor(m_all, 32, 64));
        const float sc = exp2_safe(m[h], m_all);
        float lh = l[h] * sc;
        lh += __shfl_xor(lh, 16, 64);
        lh += __shfl_xor(lh, 32, 64);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float a = acc[h][c] * sc;
            a += __shfl_xor(a, 16, 64);
            a += __shfl_xor(a, 32, 64);
            if (sub == 0) sm_o[wave][h][li * 8 + c] = a;
        }
        if (lane == 0) {
            sm_m[wave][h] = m_all;
            sm_l[wave][h] = lh;
        }
    }
    __syncthreads();
    // 256 threads merge the four waves: thread -> (head pair, channel)
    for (int item = threadIdx.x; item < G * LVR_D; item += 256) {
        const int h = item / LVR_D, c = item % LVR_D;
        float M = fmaxf(fmaxf(sm_m[0][h], sm_m[1][h]), fmaxf(sm_m[2][h], sm_m[3][h]));
        float o = 0.f, lt = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float sc = exp2_safe(sm_m[w][h], M);
            o += sc * sm_o[w][h][c];
            lt += sc * sm_l[w][h];
        }
        part_o[((hq0 + h) * P + p) * LVR_D + c] = o;
        if (c == 0) {
            part_ml[((hq0 + h) * P + p) * 2] = M;
            part_ml[((hq0 + h) * P + p) * 2 + 1] = lt;
        }
    }
}

// Dense baseline for bf16 caches with the logits on the matrix cores.  A wave takes tiles of 16
// rows: K in MFMA operand layout (scores as in mfma_score.h, q pre-scaled by sigma*log2 e), V in
// row layout (lane (sub, li): row 4i+sub, channels 8li..8li+7).  The lanes that hold the scores
// keep the running maximum, turn the tile's scores into weights and hand them (and the rescale
// factor) to the V lanes through LDS; the weighted sum of V runs on the vector ALU.
template <int HB>
__global__ void __launch_bounds__(256)
dense_mfma_kernel(const void *__restrict__ K, const void *__restrict__ V, const float *__restrict__ q,
                  float *__restrict__ part_ml, float *__restrict__ part_o, int64_t cap_rows, int64_t n_total, int P,
                  int n_q_heads, int n_kv_heads, int G, float qscale) {
    constexpr int NH = HB * 4;
    __shared__ uint4 s_bq[HB][4][64];
    __shared__ float s_p[4][NH][4][4];      // [wave][head][row % 4][row / 4]
    __shared__ float s_alpha[4][NH];
    __shared__ float sm_m[4][NH], sm_l[4][NH];
    __shared__ float sm_o[4][NH][LVR_D];
    const int bh = blockIdx.y, p = blockIdx.x;
    const int b = bh / n_kv_heads, kvh = bh % n_kv_heads;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, kq = lane >> 4;     // MFMA roles
    const int sub = kq, li = n;                  // V roles
    const int64_t hq0 = (int64_t)b * n_q_heads + kvh * G;

    const int64_t R = (((n_total + P - 1) / P) + 15) & ~(int64_t)15;
    const int64_t start = (int64_t)p * R;
    const int64_t end = (start + R < n_total) ? start + R : n_total;

    lvr_bf16x8 bq[HB][4];
    lvr_build_q_frags_wg<HB>(q + hq0 * LVR_D, G, qscale, s_bq, bq);
    const bool rep = n >= 8 && n < 12;           // this lane holds scores of head hb*4 + n - 8
    const char *Kb = static_cast<const char *>(K) + (int64_t)bh * cap_rows * LVR_D * 2;
    const char *Vb = static_cast<const char *>(V) + (int64_t)bh * cap_rows * LVR_D * 2;

    float m_run[HB], l_run[HB], acc[NH][8];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
        m_run[hb] = -INFINITY;
        l_run[hb] = 0.f;
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) lvr_zero8(acc[h]);

    // the waves of the workgroups that share a compute unit take turns at the top priority (at equal priority the
    // oldest wave is served first and the workgroups dispatched last finish last), as in the sparse path's query kernel
    const int prio_phase = (int)((blockIdx.y * gridDim.x + blockIdx.x) >> 8);
    int turn = 0;
    for (int64_t r0 = start + wave * 16; r0 < end; r0 += 64) {   // uniform over the wave
        switch ((prio_phase + (turn++ >> 1)) & 3) {
            case 0: __builtin_amdgcn_s_setprio(0); break;
            case 1: __builtin_amdgcn_s_setprio(1); break;
            case 2: __builtin_amdgcn_s_setprio(2); break;
            default: __builtin_amdgcn_s_setprio(3); break;
        }
        uint4 av[4];
        lvr_raw8<lvr_bf16_t> vr[4];
        {
            int64_t row = r0 + n;
            if (row >= end) row = end - 1;
            lvr_load_a_frags(Kb, row, av);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int64_t row = r0 + 4 * i + sub;
            if (row >= end) row = end - 1;
            lvr_load_raw(Vb, row, li, vr[i]);
        }
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
            lvr_f32x4 s = lvr_score_tile(av, bq[hb]);
            float tmax = -INFINITY;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (r0 + 4 * kq + j >= end) s[j] = -INFINITY;
                tmax = fmaxf(tmax, s[j]);
            }
            tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
            const float m_new = fmaxf(m_run[hb], tmax);
            const float alpha = exp2_safe(m_run[hb], m_new);
            float psum = 0.f;
            float pj[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                pj[j] = exp2_safe(s[j], m_new);
                psum += pj[j];
            }
            l_run[hb] = l_run[hb] * alpha + psum;
            m_run[hb] = m_new;
            if (rep) {
                const int h = hb * 4 + n - 8;
#pragma unroll
                for (int j = 0; j < 4; ++j) s_p[wave][h][j][kq] = pj[j];
                if (kq == 0) s_alpha[wave][h] = alpha;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float vx[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) lvr_unpack(vr[i], vx[i]);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const float4 pw = *reinterpret_cast<const float4 *>(&s_p[wave][h][sub][0]);
            const float al = s_alpha[wave][h];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                acc[h][c] = acc[h][c] * al + pw.x * vx[0][c] + pw.y * vx[1][c] + pw.z * vx[2][c] + pw.w * vx[3][c];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_s_setprio(0);
    // per wave: add the four row subsets (same running maximum), collect l over the score lanes
#pragma unroll
    for (int h = 0; h < NH; ++h) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float a = acc[h][c];
            a += __shfl_xor(a, 16, 64);
            a += __shfl_xor(a, 32, 64);
            if (sub == 0) sm_o[wave][h][li * 8 + c] = a;
        }
    }
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
        float lh = l_run[hb];
        lh += __shfl_xor(lh, 16, 64);
        lh += __shfl_xor(lh, 32, 64);
        if (rep && kq == 0) {
            sm_m[wave][hb * 4 + n - 8] = m_run[hb];
            sm_l[wave][hb * 4 + n - 8] = lh;
        }
    }
    __syncthreads();
    for (int item = threadIdx.x; item < G * LVR_D; item += 256) {
        const int h = item / LVR_D, c = item % LVR_D;
        const float M = fmaxf(fmaxf(sm_m[0][h], sm_m[1][h]), fmaxf(sm_m[2][h], sm_m[3][h]));
        float o = 0.f, lt = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float sc = exp2_safe(sm_m[w][h], M);
            o += sc * sm_o[w][h][c];
            lt += sc * sm_l[w][h];
        }
        part_o[((hq0 + h) * P + p) * LVR_D + c] = o;
        if (c == 0) {
            part_ml[((hq0 + h) * P + p) * 2] = M;
            part_ml[((hq0 + h) * P + p) * 2 + 1] = lt;
        }
    }
}

template <typename KT>
hipError_t launch_dense_t(lvr_index *ix, const float *q, float *out, int P, hipStream_t st) {
    dim3 grid((unsigned)P, (unsigned)lvr_n_bh(ix));
    const float qscale = ix->sigma * LOG2E;
#define LVR_DENSE_CASE(GG)                                                                                     \
    case GG:                                                                                                   \
        hipLaunchKernelGGL((dense_partial_kernel<KT, GG>), grid, dim3(256), 0, st, ix->K, ix->V, q, ix->part_ml, \
                           ix->part_o, ix->cap_rows, ix->n_total, P, ix->cfg.n_q_heads, ix->cfg.n_kv_heads,    \
                           qscale);                                                                            \
        break;
    switch (ix->G) {
        LVR_DENSE_CASE(1)
        LVR_DENSE_CASE(2)
        LVR_DENSE_CASE(4)
        LVR_DENSE_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef LVR_DENSE_CASE
    return hipGetLastError();
}

}  // namespace

hipError_t lvr_launch_sparse_attention_wg(lvr_index *ix, const float *q, const int32_t *idx, const float *scores,
                                          const int32_t *count, int count_stride, int64_t cap, float *out,
                                          int32_t *publish_count, hipStream_t st) {
    const int n_bhq = lvr_n_bhq(ix);
    const float qscale = ix->sigma * LOG2E;
    // a pair of events handed in by the caller goes into the dispatch itself (they then read the kernel's own start and end)
    hipEvent_t ev0 = ix->launch_start, ev1 = ix->launch_stop;
#define LVR_AT_LAUNCH_N(KERNEL, GRID, THREADS, ...)                                                         \
    do {                                                                                                    \
        if (ev0) hipExtLaunchKernelGGL(KERNEL, GRID, dim3(THREADS), 0, st, ev0, ev1, 0, __VA_ARGS__);        \
        else hipLaunchKernelGGL(KERNEL, GRID, dim3(THREADS), 0, st, __VA_ARGS__);                           \
    } while (0)
#define LVR_AT_LAUNCH(KERNEL, GRID, ...) LVR_AT_LAUNCH_N(KERNEL, GRID, 1024, __VA_ARGS__)
#define LVR_WG_LAUNCH(KT)                                                                                                \
    LVR_AT_LAUNCH(sparse_attention_wg_kernel<KT>, dim3((unsigned)n_bhq), ix->K, ix->V, ix->pos_slot, q, idx, count,       \
                  count_stride, cap, out, ix->cap_rows, ix->n_total, ix->cfg.n_q_heads, ix->cfg.n_kv_heads, ix->G, qscale, \
                  lvr_head_count(ix), lvr_head_stat(ix), publish_count)
#define LVR_CARRY_LAUNCH(KT, WAVES)                                                                                      \
    LVR_AT_LAUNCH_N((sparse_attention_wg_carry_kernel<KT, WAVES>), dim3((unsigned)n_bhq), 64 * WAVES, count, idx, scores, \
                    ix->V, cap, count_stride, (int)ix->cap_rows, (int)ix->n_total, ix->G, ix->pos_slot, out, qscale,      \
                    lvr_head_count(ix), lvr_head_stat(ix), publish_count)
    // Lists that carry their scores.  With more heads than compute units a workgroup of eight waves serves a head: its waves
    // hold up to 64 rows each in flight (fp32: 32) as the sixteen of the wide form do, and two such workgroups share a compute
    // unit instead of queueing up behind each other (bf16, 512 heads of 655 keys: 126.5 us per step against 128.2 with sixteen
    // light waves that take a trip per 16 rows; 384 heads of 18 to 105 keys: 15.4 against 18.4, 34.2 against 37.2.  fp32, light
    // waves and eight: 288 heads of 20 to 100 keys 19.4 / 16.9 and 21.9 / 19.2, 2048 heads of 40 keys 168.1 / 158.0).
    const bool many_heads = n_bhq > 256;
    if (ix->cfg.kv_dtype == LVR_BF16) {
        // Up to 128 heads two workgroups can share a head (one per half of the channels) and every workgroup still
        // has a compute unit of its own.  That pays where a head's list is long (656 keys per head at 128k keys of
        // context: 9.1 against 9.7 us); short lists lose more to the extra barrier and the ticket than they gain
        // (3.6 keys per head: 7.6 against 6.9 us), and the list lengths are not known on the host, so the context
        // length stands in as it does for the launch form.
        if (scores && many_heads) LVR_CARRY_LAUNCH(lvr_bf16_t, 8);
        else if (scores && n_bhq <= 128 && publish_count && ix->n_total > 65536)
            LVR_AT_LAUNCH((sparse_attention_wg_carry_split_kernel<lvr_bf16_t, 2>), dim3((unsigned)n_bhq * 2),
                               count, idx, scores, ix->V, cap, count_stride, (int)ix->cap_rows, (int)ix->n_total, ix->G,
                               ix->pos_slot, out, qscale, lvr_head_count(ix), lvr_head_stat(ix), publish_count, lvr_head_ticket(ix));
        else if (scores) LVR_CARRY_LAUNCH(lvr_bf16_t, 16);
        else LVR_WG_LAUNCH(lvr_bf16_t);
    } else {
        if (scores && many_heads) LVR_CARRY_LAUNCH(lvr_f32_t, 8);
        else if (scores) LVR_CARRY_LAUNCH(lvr_f32_t, 16);
        else LVR_WG_LAUNCH(lvr_f32_t);
    }
#undef LVR_CARRY_LAUNCH
#undef LVR_WG_LAUNCH
#undef LVR_AT_LAUNCH
#undef LVR_AT_LAUNCH_N
    return hipGetLastError();
}

hipError_t lvr_launch_sparse_splits(lvr_index *ix, const float *q, const int32_t *idx, const int32_t *count, int count_stride,
                                    int64_t cap, float *out, int32_t *publish_count, hipStream_t st) {
    const int n_bhq = lvr_n_bhq(ix);
    // Every workgroup of a head costs a read of the count and a ticket whether the list reaches it or not, and the list lengths
    // are not known here, only the room for them.  Up to 2048 entries: 16 workgroups up to 16 heads, 8 up to 64, then 4 (80 / 330 / 1300 entries per
    // head, us: 32 bf16 heads 6.4 / 6.8 / 8.9 with 16 workgroups, 6.0 / 6.3 / 8.8 with 8; 64 fp32 heads 9.9 / 10.5 / 20.9 with 16, 8.2 / 8.8 / 18.9
    // with 8, 6.9 / 10.4 / 21.5 with 4; 128 bf16 heads 8.7 / 9.2 / 20.3 with 8, 6.6 / 9.0 / 18.2 with 4).  Where there is more room, two per
    // compute unit, with which the longest lists are read fastest (4000 / 16000 entries per head: 32 fp32 heads 27.1 / 123.3 with 8, 23.9 / 79.4
    // with 16, 25.9 / 79.4 with 32; 8 fp32 heads 14.5 / 43.6 with 16, 11.0 / 26.7 with 32, 10.6 / 23.4 with 64; 64 bf16 heads 23.0 / 61.3 with 8,
    // 23.7 / 66.4 with 16), and of short ones there 0.4 us slower (32 bf16 heads of 80 entries).
    int wgs = n_bhq <= 16 ? 16 : (n_bhq <= 64 ? 8 : 4);
    if (cap > 2048)
        while (wgs < SPLIT_WGS_MAX && 2 * wgs * n_bhq <= 512) wgs *= 2;
    if (wgs > ix->P) wgs = ix->P;   // the caller's number of splits is an upper bound
    const int P = wgs * SPLIT_WAVES;
    int word = 0;   // a word per number it counts modulo: an index meets two powers of two, or its P in the place of those above
    while ((1 << word) < wgs) ++word;
    int32_t *ticket = lvr_split_ticket(ix) + word;
    dim3 grid((unsigned)wgs, (unsigned)n_bhq);
#define LVR_SPLIT_LAUNCH(KT)                                                                                              \
    hipLaunchKernelGGL(sparse_attention_kernel<KT>, grid, dim3(64 * SPLIT_WAVES), 0, st, count, idx, q, ix->V, cap,         \
                       count_stride, P, (int)ix->cap_rows, (int)ix->n_total, ix->G, ix->sigma * LOG2E, ix->K,              \
                       ix->pos_slot, ix->part_ml, ix->part_o, ticket, out, lvr_head_count(ix),               \
                       lvr_head_stat(ix), publish_count)
    if (ix->cfg.kv_dtype == LVR_BF16) LVR_SPLIT_LAUNCH(lvr_bf16_t);
    else LVR_SPLIT_LAUNCH(lvr_f32_t);
#undef LVR_SPLIT_LAUNCH
    return hipGetLastError();
}

hipError_t lvr_launch_carried_splits(lvr_index *ix, const int32_t *idx, const float *scores, const int32_t *count, int count_stride,
                                     int64_t cap, hipStream_t st) {
    dim3 grid((unsigned)ix->P, (unsigned)lvr_n_bhq(ix));
#define LVR_SPLIT_LAUNCH(KT)                                                                                              \
    hipLaunchKernelGGL(carried_split_kernel<KT>, grid, dim3(64), 0, st, count, idx, scores, ix->V, cap, count_stride,      \
                       ix->P, (int)ix->cap_rows, (int)ix->n_total, ix->G, ix->sigma * LOG2E, ix->pos_slot, ix->part_ml,    \
                       ix->part_o)
    if (ix->cfg.kv_dtype == LVR_BF16) LVR_SPLIT_LAUNCH(lvr_bf16_t);
    else LVR_SPLIT_LAUNCH(lvr_f32_t);
#undef LVR_SPLIT_LAUNCH
    return hipGetLastError();
}

int lvr_dense_splits(const lvr_index *ix) {
    int64_t P = (ix->n_total + 63) / 64;
    if (P > ix->P_dense) P = ix->P_dense;
    if (P < 1) P = 1;
    return (int)P;
}

hipError_t lvr_launch_dense_partial(lvr_index *ix, const float *q, hipStream_t st) {
    const int P = lvr_dense_splits(ix);
    if (ix->cfg.kv_dtype == LVR_BF16 && ix->n_total > 0) {
        dim3 grid((unsigned)P, (unsigned)lvr_n_bh(ix));
        const float qscale = ix->sigma * LOG2E;
        if (ix->G <= 4)
            hipLaunchKernelGGL(dense_mfma_kernel<1>, grid, dim3(256), 0, st, ix->K, ix->V, q, ix->part_ml, ix->part_o,
                               ix->cap_rows, ix->n_total, P, ix->cfg.n_q_heads, ix->cfg.n_kv_heads, ix->G, qscale);
        else
            hipLaunchKernelGGL(dense_mfma_kernel<2>, grid, dim3(256), 0, st, ix->K, ix->V, q, ix->part_ml, ix->part_o,
                               ix->cap_rows, ix->n_total, P, ix->cfg.n_q_heads, ix->cfg.n_kv_heads, ix->G, qscale);
        return hipGetLastError();
    }
    return ix->cfg.kv_dtype == LVR_BF16 ? launch_dense_t<lvr_bf16_t>(ix, q, nullptr, P, st)
                                        : launch_dense_t<lvr_f32_t>(ix, q, nullptr, P, st);
}

hipError_t lvr_launch_combine(lvr_index *ix, float *out, int P, const int32_t *count, int count_stride, int64_t cap,
                              int32_t *publish_count, hipStream_t st) {
    const int n_bhq = lvr_n_bhq(ix);
    hipLaunchKernelGGL(combine_kernel, dim3((unsigned)n_bhq), dim3(512), 0, st, ix->part_o, ix->part_ml, count, cap, out, P,
                       count_stride, lvr_head_count(ix), lvr_head_stat(ix), publish_count);
    return hipGetLastError();
}
