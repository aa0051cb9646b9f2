// Fused range-query kernel for fp32 caches: bound test and exact check in one launch, on the vector ALU.
//
// The same two phases as the bf16 kernel (query_fused.hip).  A workgroup owns a segment of consecutive groups of one
// (sequence, KV head):
//   phase A  the bound of Eq. (2) per coordinate block, summed ("Query 2"): 16 lanes per centre, four centres per load of a
//            wave, the survivors' bits compacted into an LDS list;
//   phase B  the exact dot product of the surviving groups' key rows, 16 rows per wave and tile, two tiles in flight; positions
//            and scores of the qualifying keys go out through the emission queues (emitter.h), so that the attention that
//            follows reads V rows only.
// One extra workgroup per (sequence, KV head) scans the buffer rows (Sec. 4.3) and stores the rows of an append that rides in
// the launch.  The per-head counters must be zero when the kernel starts.
//
// Bound by the key rows: 512 bytes each, and at fp32's group sizes on keys without locality most balls survive.  What
// matters is therefore that the rows are spread over the device: segments are as small as one round of workgroups asks for, down to
// a trip of 16 groups.  With segments of 256 groups and a launch per stage the steps took 62.7 us at 8 x 16384 keys and
// 28.3 us at one head of 4096 keys; now 23.4 and 10.0 us.
#include "emitter.h"

namespace {

struct FusedF32Args {
    const void *K;
    void *V;
    const int32_t *slot_pos;
    const void *k_new, *v_new;   // rows appended by this launch ([batch][H_kv][m_new][d]), or NULL
    int m_new;                   // n_total already counts them
    int32_t *seg_count;          // survivors per segment, for statistics only
    lvr_emit_target emit;
    int64_t n_groups, max_groups, max_segs, cap_rows, n_indexed, n_total;
    int log2r, buffer_dense;
};

constexpr int F32_SEG_MAX = 1024;   // groups of a segment: 64 trips of 16 groups, lane `it` of a wave keeps the bits of trip `it`

template <int G>
__global__ void __launch_bounds__(256)
query_f32_kernel(const float *__restrict__ q_in, const void *__restrict__ centres, const float *__restrict__ tau_in,
                 const float *__restrict__ radii, const int n_groups, const int max_groups, const int seg_groups, const int n_segs,
                 const int S, const FusedF32Args a) {
    __shared__ int32_t s_queue[4][G][LVR_QCAP];
    __shared__ float s_qscore[4][G][LVR_QCAP];
    __shared__ uint16_t s_list[F32_SEG_MAX];   // surviving groups, as offsets from the segment's first group
    __shared__ int s_tot[4];
    __shared__ int s_wcnt[4][G], s_wbase[G];
    const int bh = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane >> 4, li = lane & 15;
    const int64_t hq0 = (int64_t)bh * G;
    const bool buffer_wg = (int)blockIdx.x >= n_segs;

    float qv[G][8], taue[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
        const float *qh = q_in + (hq0 + h) * LVR_D + li * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[h][e] = qh[e];
        taue[h] = lvr_effective_tau(tau_in[hq0 + h]);
    }

    int64_t rows;        // key rows phase B has to check
    int64_t seg_g0 = 0;  // first group of this workgroup's segment
    if (!buffer_wg) {
        // ---------------- phase A: bound test over this segment's centres ----------------
        seg_g0 = (int64_t)blockIdx.x * seg_groups;
        const char *Cb = static_cast<const char *>(centres) + (int64_t)bh * max_groups * LVR_D * 4;
        const float *Rb = radii + (int64_t)bh * max_groups * S;
        const int lanes_per_sub = 16 / S;
        float qn[G];   // lanes li < S: |pi_li q_h|, rounded up; the others zero
#pragma unroll
        for (int h = 0; h < G; ++h) {
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += qv[h][e] * qv[h][e];
            for (int off = 1; off < lanes_per_sub; off <<= 1) ss += __shfl_xor(ss, off, 64);
            const float mine = __shfl(ss, (lane & 48) + ((li < S) ? li * lanes_per_sub : li), 64);
            qn[h] = (li < S) ? sqrtf(mine) * (1.0f + 0x1p-20f) : 0.f;
        }
        const int trips = seg_groups >> 4;   // trip `it` of wave w: groups 16 it + 4 w .. + 3
        uint32_t mybits = 0;
        for (int it0 = 0; it0 < trips; it0 += 2) {
            if (seg_g0 + it0 * 16 >= n_groups) break;   // uniform
            lvr_raw8<lvr_f32_t> raw[2];
            float rad[2];
            int64_t g[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                g[u] = seg_g0 + (it0 + u) * 16 + wave * 4 + sub;
                const int64_t gc = g[u] < n_groups ? g[u] : n_groups - 1;
                lvr_load_raw(Cb, gc, li, raw[u]);
                rad[u] = Rb[gc * S + (li & (S - 1))];   // lanes li >= S multiply it by zero below
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float x[8];
                lvr_unpack(raw[u], x);
                bool alive = false;
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    float p = rad[u] * qn[h];
#pragma unroll
                    for (int e = 0; e < 8; ++e) p += qv[h][e] * x[e];
                    alive |= (lvr_row16_sum(p) >= taue[h]);
                }
                const uint64_t bal = __ballot(alive && g[u] < n_groups && it0 + u < trips && li == 0);
                const uint32_t mask4 = (uint32_t)(bal & 1u) | (uint32_t)((bal >> 15) & 2u) | (uint32_t)((bal >> 30) & 4u) |
                                       (uint32_t)((bal >> 45) & 8u);
                if (lane == it0 + u) mybits = mask4;
            }
        }
        const int cnt = __popc(mybits);
        const int incl = lvr_wave_inclusive_sum(cnt);
        if (lane == 63) s_tot[wave] = incl;
        __syncthreads();
        int o = incl - cnt, total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            o += (w < wave) ? s_tot[w] : 0;
            total += s_tot[w];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (mybits & (1u << k)) s_list[o++] = (uint16_t)(lane * 16 + wave * 4 + k);
        if (threadIdx.x == 0) a.seg_count[(int64_t)bh * a.max_segs + blockIdx.x] = total;
        __syncthreads();
        rows = (int64_t)total << a.log2r;
    } else {
        rows = a.n_total - a.n_indexed;
        if (a.m_new > 0) {   // append fused into the step (Sec. 4.3): the rows go to the arena tail before the buffer is scanned
            const int64_t pieces = (int64_t)a.m_new * 32;   // 16-byte pieces per matrix
            const uint4 *ks = static_cast<const uint4 *>(a.k_new) + (int64_t)bh * pieces;
            const uint4 *vs = static_cast<const uint4 *>(a.v_new) + (int64_t)bh * pieces;
            const int64_t row0 = (int64_t)bh * a.cap_rows + (a.n_total - a.m_new);
            uint4 *kd = static_cast<uint4 *>(const_cast<void *>(a.K)) + row0 * 32;
            uint4 *vd = static_cast<uint4 *>(a.V) + row0 * 32;
            for (int64_t i = threadIdx.x; i < 2 * pieces; i += 256) {
                if (i < pieces) kd[i] = ks[i];
                else vd[i - pieces] = vs[i - pieces];
            }
            __syncthreads();   // the new rows are in place for every wave of this workgroup
        }
    }

    // ---------------- phase B: exact check of the surviving rows ----------------
    const bool rep = li < G;
    float my_tau = INFINITY;
#pragma unroll
    for (int h = 0; h < G; ++h) my_tau = (li == h) ? taue[h] : my_tau;
    lvr_emitter<G, true> em;
    em.q = s_queue[wave];
    em.qs = s_qscore[wave];
    em.count = 0;
    em.rep_base = 0;
    em.hq_base = hq0;
    const char *Kb = static_cast<const char *>(a.K) + (int64_t)bh * a.cap_rows * LVR_D * 4;
    const int32_t *spos = a.slot_pos ? a.slot_pos + (int64_t)bh * a.cap_rows : nullptr;
    const int rmask = (1 << a.log2r) - 1;
    const int64_t tiles = (rows + 15) >> 4;
    for (int64_t t0 = wave; t0 < tiles; t0 += 8) {   // tiles t0 and t0 + 4; uniform over the wave
        int slot[2][4];
        lvr_raw8<lvr_f32_t> raw[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int64_t rowidx = (t0 + 4 * u) * 16 + i * 4 + sub;
                if (rowidx >= rows) rowidx = rows - 1;   // a repeat of the last row, dropped below
                slot[u][i] = buffer_wg ? (int)(a.n_indexed + rowidx)
                                       : (int)(((seg_g0 + s_list[rowidx >> a.log2r]) << a.log2r) + (rowidx & rmask));
                lvr_load_raw(Kb, slot[u][i], li, raw[u][i]);
            }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (t0 + 4 * u >= tiles) break;   // uniform
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float x[8];
                lvr_unpack(raw[u][i], x);
                float mine = 0.f;
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    float p = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) p += qv[h][e] * x[e];
                    const float s = lvr_row16_sum(p);
                    mine = (li == h) ? s : mine;
                }
                const bool valid = (t0 + 4 * u) * 16 + i * 4 + sub < rows;
                const bool pred = valid && rep && (mine >= my_tau || (buffer_wg && a.buffer_dense));
                em.push(a.emit, lane, rep, pred, slot[u][i], lane, spos, mine);   // the reporting lane holds the row's slot itself
            }
        }
    }
    // last flush: one lane per head reserves the workgroup's range in the head's list, every wave writes behind the waves
    // before it (a quarter of the atomics that end a launch)
    if (rep && sub == 0) s_wcnt[wave][li] = em.count;
    __syncthreads();
    if (wave == 0 && rep && sub == 0) {
        const int tot = s_wcnt[0][li] + s_wcnt[1][li] + s_wcnt[2][li] + s_wcnt[3][li];
        s_wbase[li] = lvr_reserve_last(a.emit, hq0 + li, tot, gridDim.x);
    }
    __syncthreads();
    int base = 0;
    if (rep && sub == 0) {
        const int c0 = s_wcnt[0][li], c1 = s_wcnt[1][li], c2 = s_wcnt[2][li];
        base = s_wbase[li] + (wave > 0 ? c0 : 0) + (wave > 1 ? c1 : 0) + (wave > 2 ? c2 : 0);
    }
    if (__ballot(em.count > 0)) em.write_out(a.emit, lane, spos, base);
}

}  // namespace

hipError_t lvr_launch_query_f32(lvr_index *ix, const float *q, const float *tau, int32_t *out_idx, int64_t cap,
                                hipStream_t st, const void *k_new, const void *v_new, int64_t m_new, int32_t *out_count) {
    if (ix->cfg.kv_dtype != LVR_F32) return hipErrorInvalidValue;
    FusedF32Args a;
    a.K = ix->K;
    a.V = ix->V;
    a.slot_pos = ix->slot_pos;
    a.k_new = k_new;
    a.v_new = v_new;
    a.m_new = (int)m_new;
    a.seg_count = lvr_seg_count(ix);
    a.emit.out_idx = out_idx;
    a.emit.head_count = lvr_head_count(ix);
    a.emit.overflow = lvr_overflow_flag(ix);
    a.emit.cap = cap;
    a.emit.out_score = ix->scores;
    a.emit.score_stride = ix->cap_rows;
    a.emit.out_count = out_count;
    a.emit.head_stat = lvr_head_stat(ix);
    a.n_groups = ix->n_indexed / ix->cfg.group_size;
    a.max_groups = ix->max_groups;
    a.max_segs = lvr_max_segs(ix->max_groups);
    a.cap_rows = ix->cap_rows;
    a.n_indexed = ix->n_indexed;
    a.n_total = ix->n_total + m_new;
    a.log2r = 0;
    while ((1 << a.log2r) < ix->cfg.group_size) ++a.log2r;
    a.buffer_dense = (ix->cfg.flags & LVR_ATTEND_BUFFER_DENSE) ? 1 : 0;
    const int n_bh = lvr_n_bh(ix);
    // segments of a multiple of 16 groups (a trip of the four waves); aim at the workgroups that are resident at once (three
    // per compute unit, two with eight heads: the registers of two tiles of rows and the query) less the buffers', so that
    // the launch is one round (8 x 16384 keys: 23.6 us per step against 25.2 with 1024, which ran as 768 + 264).  Counted in
    // whole segments per (sequence, KV head): the same total divided by the workgroups alone put 13 on each of 40, 520 on room
    // for 512 (five sequences of 16384 keys, 64 heads on 8: 133.5 us, 101.8 with twelve), and a long and a short one on each of 512
    // (4096 keys: 75.1 us on local keys, 56.9 with one).  What does not fit one round gets several, and four where already
    // a segment each is more than one.
    const int64_t buffers = a.n_total > ix->n_indexed ? n_bh : 0;
    // Rows behind the host link come no faster for more requests: 96 workgroups (8 x 4096 keys, all balls survive: 332 us per step,
    // 392 with 512, 361 with a launch per stage; 64 and 128: 333 and 360).
    const bool on_host = (ix->cfg.flags & LVR_KV_IN_HOST_MEMORY) != 0;
    const int64_t resident = on_host ? 96 : (ix->G == 8 ? 512 : 768);
    int64_t per_head = (a.n_groups + F32_SEG_MAX - 1) / F32_SEG_MAX;   // segments of a (sequence, KV head), at least
    if (ix->cfg.query_workgroups > 0) {
        per_head = ix->cfg.query_workgroups / n_bh;
    } else {
        int64_t rounds = (per_head * n_bh + buffers + resident - 1) / resident;
        if (n_bh + buffers > resident && rounds < 4 && !on_host) rounds = 4;
        if (rounds < 1) rounds = 1;
        per_head = (rounds * resident - buffers) / n_bh;
    }
    if (per_head < 1) per_head = 1;
    int64_t seg = (a.n_groups + per_head - 1) / per_head;
    seg = (seg + 15) & ~(int64_t)15;
    if (seg < LVR_MIN_SEG_GROUPS) seg = LVR_MIN_SEG_GROUPS;
    if (seg > F32_SEG_MAX) seg = F32_SEG_MAX;
    const int seg_groups = (int)seg, n_segs = (int)((a.n_groups + seg - 1) / seg);
    const int has_buffer = a.n_total > ix->n_indexed ? 1 : 0;
    ix->seg_groups = seg_groups;
    ix->n_segs = n_segs;
    if (n_segs + has_buffer == 0) return out_count ? lvr_launch_publish_counts(ix, out_count, st) : hipSuccess;
    const dim3 grid((unsigned)(n_segs + has_buffer), (unsigned)n_bh);
    switch (ix->G) {
        case 1: hipLaunchKernelGGL(query_f32_kernel<1>, grid, dim3(256), 0, st, q, ix->centres, tau, ix->radii, (int)a.n_groups, (int)a.max_groups, seg_groups, n_segs, ix->cfg.n_subspaces, a); break;
        case 2: hipLaunchKernelGGL(query_f32_kernel<2>, grid, dim3(256), 0, st, q, ix->centres, tau, ix->radii, (int)a.n_groups, (int)a.max_groups, seg_groups, n_segs, ix->cfg.n_subspaces, a); break;
        case 4: hipLaunchKernelGGL(query_f32_kernel<4>, grid, dim3(256), 0, st, q, ix->centres, tau, ix->radii, (int)a.n_groups, (int)a.max_groups, seg_groups, n_segs, ix->cfg.n_subspaces, a); break;
        case 8: hipLaunchKernelGGL(query_f32_kernel<8>, grid, dim3(256), 0, st, q, ix->centres, tau, ix->radii, (int)a.n_groups, (int)a.max_groups, seg_groups, n_segs, ix->cfg.n_subspaces, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
