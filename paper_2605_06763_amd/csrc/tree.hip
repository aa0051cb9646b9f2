// Grouping by a balanced axis-median tree (Sec. 4.1 "Grouping via balanced PCA trees", Alg. 2):
// starting from all keys, a node is split at the median of the coordinate axis of largest
// variance until a node holds r keys.  One tree over the full key is shared by all coordinate
// blocks, and the rows are stored regrouped, so the query kernels see the same layout as with
// contiguous grouping: group g = arena rows g*r .. g*r+r-1, plus a map slot -> token position.
//
// Level-synchronous construction.  The number of groups is padded to a power of two with
// virtual keys that compare greater than every real key; they drift to the right end, so the
// real keys always fill a prefix of full groups (for a power-of-two number of groups, which
// is what every workload here has, there is no padding and the splits are exactly Alg. 2's
// floor(m/2) medians).  At level L every node is an aligned run of n'/2^L entries of the
// current order; per level:
//   1. per node, variance of each of the 128 coordinates over its real keys -> axis of the
//      largest variance (first axis wins a tie);
//   2. the node is split at the median of (coordinate on that axis, position): the coordinate is
//      mapped to an order-preserving unsigned code, and equal coordinates are ordered by position
//      (Alg. 2 is silent; this is the rule the CPU reference uses).
// Only which entries go left matters above the last level, so nodes of more than 1024 entries are
// not sorted: a workgroup per node finds the median code by counting digits and moves the
// entries to the two halves in the order they had.  Every node's entries therefore stay in ascending
// position order, which is what breaks ties and keeps the padding at a node's end.  The levels of
// nodes of at most 1024 entries are finished by tree_small_kernel in one launch, a workgroup per
// node, an entry per thread; it sorts, so a finished group's rows are in the order of the last split.
//
// A build of 8 x 32768 bf16 keys in groups of four (five levels above 1024 entries, eight below) took
// 2.5 ms with one wave per SIMD on the statistics, a device-wide 64-bit radix sort per level and
// four waves per small node; this construction takes 0.33 ms (tree build and one step: 2321 -> 424 us).
#include <type_traits>

#include "lvr_internal.h"

namespace {

constexpr int PIECE = 1024;         // entries per partial-statistics piece of a large node
constexpr int TREE_WG_MAX = 1024;   // entries of a node that one workgroup finishes

struct TreeSrc {
    const char *K;             // source key rows
    int64_t sb, sh, st;        // element strides (batch, head, token)
    int elt, n_kv_heads;
    __device__ __forceinline__ const char *row(int bh, int64_t pos) const {
        const int b = bh / n_kv_heads, h = bh % n_kv_heads;
        return K + (b * sb + h * sh + pos * st) * elt;
    }
};

// entry i of (bh): low `pos_bits` bits of keys[bh*np + i] hold the position; >= n_real is padding
__device__ __forceinline__ int64_t key_pos(uint64_t k, int pos_bits) { return (int64_t)(k & ((1ull << pos_bits) - 1ull)); }

// lane owns channels 2*lane, 2*lane+1 of a row
template <int ELT>
__device__ __forceinline__ void lane_pair(const char *row, int lane, float &x0, float &x1) {
    if constexpr (ELT == 2) {
        const uint32_t w = reinterpret_cast<const uint32_t *>(row)[lane];
        x0 = __uint_as_float(w << 16);
        x1 = __uint_as_float(w & 0xffff0000u);
    } else {
        const float2 v = reinterpret_cast<const float2 *>(row)[lane];
        x0 = v.x;
        x1 = v.y;
    }
}

// order-preserving unsigned code of coordinate c of a row (16 or 32 bits); padding takes the largest code
template <int ELT>
__device__ __forceinline__ uint32_t coord_code(const char *row, int c) {
    if constexpr (ELT == 2) {
        uint32_t u = reinterpret_cast<const uint16_t *>(row)[c];
        if (u == 0x8000u) u = 0;   // -0 and +0 are the same coordinate
        return (u & 0x8000u) ? (~u & 0xffffu) : (u | 0x8000u);
    } else {
        uint32_t u = reinterpret_cast<const uint32_t *>(row)[c];
        if (u == 0x80000000u) u = 0;
        return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    }
}
template <int ELT>
constexpr uint32_t PAD_CODE = ELT == 2 ? 0xffffu : 0xffffffffu;

// one step of a wave maximum: the value DPP moves here, or this lane's own where nothing arrives
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
    const uint32_t l2 = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const uint32_t h2 = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    return fmax(v, __longlong_as_double((long long)(((uint64_t)h2 << 32) | l2)));
}

// argmax over 128 channel variances held as (v0, v1) per lane; lowest channel wins ties
// [c_lo, c_hi): the coordinates that may be chosen (a tree over one coordinate block looks at that block only)
__device__ __forceinline__ int wave_argmax(double v0, double v1, int lane, int c_lo, int c_hi) {
    if (2 * lane < c_lo || 2 * lane >= c_hi) v0 = -1.0;           // variances are >= 0
    if (2 * lane + 1 < c_lo || 2 * lane + 1 >= c_hi) v1 = -1.0;
    double m = fmax(v0, v1);
    m = dpp_max<0x111, 0xf>(m);   // row_shr:1, 2, 4, 8: lane 15 of a row holds the row's maximum
    m = dpp_max<0x112, 0xf>(m);
    m = dpp_max<0x114, 0xf>(m);
    m = dpp_max<0x118, 0xf>(m);
    m = dpp_max<0x142, 0xa>(m);   // row_bcast:15, row_bcast:31: lane 63 holds the wave's
    m = dpp_max<0x143, 0xc>(m);
    const uint64_t u = (uint64_t)__double_as_longlong(m);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
    const double best = __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    const uint64_t b0 = __ballot(v0 == best), b1 = __ballot(v1 == best);
    const int a0 = b0 ? 2 * __builtin_ctzll(b0) : 2 * 64, a1 = b1 ? 2 * __builtin_ctzll(b1) + 1 : 2 * 64;
    const int a = a0 < a1 ? a0 : a1;
    // Keys with NaN or overflowing coordinates: where no variance of the block is a number the masked coordinates' -1 is the
    // maximum and the first of them is taken (c_lo where nothing is masked); the split is then on that coordinate, the set a
    // query returns does not depend on it
    return a < 2 * 64 ? a : c_lo;
}

// Sums of the 64 consecutive entries whose positions the lanes hold, relative to the row (p0, p1): sixteen rows in flight.
// `real`: ballot of the lanes whose entry is no padding; `any`: a position that may be read in the place of padding.
template <int ELT>
__device__ __forceinline__ void sum_rows64(const TreeSrc &src, int bh, int lane, int mypos, uint64_t real, int any, float p0, float p1,
                                           double &s0, double &s1, double &q0, double &q1) {
    const char *base = src.row(bh, 0);
    const int64_t row_bytes = src.st * ELT;
    for (int j0 = 0; j0 < 64; j0 += 16) {
        if (!((real >> j0) & 1ull)) break;   // padding is at the end: nothing real follows (uniform)
        float x0[16], x1[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int pos = __builtin_amdgcn_readlane(mypos, j0 + u);
            const bool in = (real >> (j0 + u)) & 1ull;   // uniform
            lane_pair<ELT>(base + (int64_t)(in ? pos : any) * row_bytes, lane, x0[u], x1[u]);
        }
        if (((real >> j0) & 0xffffull) == 0xffffull) {   // uniform: no padding among them
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double d0 = (double)x0[u] - (double)p0, d1 = (double)x1[u] - (double)p1;
                s0 += d0; s1 += d1; q0 += d0 * d0; q1 += d1 * d1;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const bool in = (real >> (j0 + u)) & 1ull;
                const double d0 = in ? (double)x0[u] - (double)p0 : 0., d1 = in ? (double)x1[u] - (double)p1 : 0.;
                s0 += d0; s1 += d1; q0 += d0 * d0; q1 += d1 * d1;
            }
        }
    }
}

// Statistics of a piece of a large node: 16 waves, 64 entries each; sums are relative to the node's first key (the variance
// does not depend on the shift; the shift removes the cancellation).  order == NULL: entry i holds position i.
// Bound by the fp64 adds and the row reads about alike.
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_stats_piece_kernel(TreeSrc src, const uint32_t *__restrict__ order, double *__restrict__ partial, int64_t np,
                        int64_t n_real, int64_t m) {
    __shared__ double sm[16][256];
    __shared__ int sc[16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int bh = blockIdx.y;
    const int64_t piece = blockIdx.x;
    const int64_t node0 = (piece * PIECE / m) * m;
    const int64_t i = piece * PIECE + threadIdx.x;
    const uint32_t *ord = order + (int64_t)bh * np;
    const int mypos = order ? (int)ord[i] : (int)i;
    const int ppos = order ? (int)ord[node0] : (int)node0;   // first entry of the node; real unless the node is all padding
    const uint64_t real = __ballot(mypos < n_real);
    double s0 = 0., s1 = 0., q0 = 0., q1 = 0.;
    if (real) {   // uniform: then the node's first entry is real too
        float p0, p1;
        lane_pair<ELT>(src.row(bh, ppos), lane, p0, p1);
        sum_rows64<ELT>(src, bh, lane, mypos, real, ppos, p0, p1, s0, s1, q0, q1);
    }
    sm[wave][2 * lane] = s0; sm[wave][2 * lane + 1] = s1;
    sm[wave][128 + 2 * lane] = q0; sm[wave][128 + 2 * lane + 1] = q1;
    if (lane == 0) sc[wave] = __popcll(real);
    __syncthreads();
    const int t = threadIdx.x;
    double *out = partial + ((int64_t)bh * (np / PIECE) + piece) * 258;
    if (t < 256) {
        double a = 0.;
#pragma unroll
        for (int w = 0; w < 16; ++w) a += sm[w][t];
        out[t] = a;
    }
    if (t == 256) {
        int c = 0;
        for (int w = 0; w < 16; ++w) c += sc[w];
        out[256] = (double)c;
    }
}

// Adds the pieces of a node (eight slices of them side by side, 1024 threads) and picks the axis; every thread gets it.
__device__ __forceinline__ int node_axis(const double *__restrict__ partial, int bh, int64_t np, int64_t m, int64_t node, int c_lo, int c_hi) {
    __shared__ double sm[8][2][128];
    __shared__ double sc[8];
    __shared__ int s_axis;
    const int t = threadIdx.x, c = t & 127, sl = t >> 7;
    const int64_t pieces = m / PIECE;
    const double *pp = partial + ((int64_t)bh * (np / PIECE) + node * pieces) * 258;
    double s = 0.0, q = 0.0, cnt = 0.0;
#pragma unroll 4
    for (int64_t p = sl; p < pieces; p += 8) {
        s += pp[p * 258 + c];
        q += pp[p * 258 + 128 + c];
        cnt += pp[p * 258 + 256];
    }
    sm[sl][0][c] = s;
    sm[sl][1][c] = q;
    if (c == 0) sc[sl] = cnt;
    __syncthreads();
    if (t < 64) {
        double s0 = 0., s1 = 0., q0 = 0., q1 = 0., n = 0.;
        for (int k = 0; k < 8; ++k) {
            s0 += sm[k][0][2 * t]; s1 += sm[k][0][2 * t + 1];
            q0 += sm[k][1][2 * t]; q1 += sm[k][1][2 * t + 1];
            n += sc[k];
        }
        const double v0 = n > 0 ? (q0 - s0 * s0 / n) / n : 0., v1 = n > 0 ? (q1 - s1 * s1 / n) / n : 0.;
        const int a = wave_argmax(v0, v1, t, c_lo, c_hi);
        if (t == 0) s_axis = a;
    }
    __syncthreads();
    return s_axis;
}

// The axis of every node whose codes are fetched by a launch of their own.
__global__ void __launch_bounds__(1024)
tree_axis_kernel(const double *__restrict__ partial, int32_t *__restrict__ axis, int64_t np, int64_t m, int64_t n_nodes,
                 int c_lo, int c_hi) {
    const int a = node_axis(partial, blockIdx.y, np, m, blockIdx.x, c_lo, c_hi);
    if (threadIdx.x == 0) axis[(int64_t)blockIdx.y * n_nodes + blockIdx.x] = a;
}

// Code of every entry on its node's axis (nodes large enough that the whole device should fetch them).
template <int ELT>
__global__ void __launch_bounds__(256)
tree_codes_kernel(TreeSrc src, const uint32_t *__restrict__ order, uint32_t *__restrict__ codes, const int32_t *__restrict__ axis,
                  int64_t np, int64_t n_real, int64_t m, int64_t n_nodes) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;   // np is a multiple of 256 here
    const int bh = blockIdx.y;
    const int64_t at = (int64_t)bh * np + i;
    const int64_t pos = order ? (int64_t)order[at] : i;
    codes[at] = pos < n_real ? coord_code<ELT>(src.row(bh, pos), axis[(int64_t)bh * n_nodes + i / m]) : PAD_CODE<ELT>;
}

// Splits a node of m entries (a multiple of 2048) at its median: one workgroup per node, wave w takes the entries
// [w m/16, (w+1) m/16).  The code of the m/2-th smallest entry is found digit by digit (11 bits at a time: the leading
// digit of a bf16 code holds sign, exponent and two bits of the fraction, enough that the counters of one LDS pass are not
// all the same), then entries below it, and as many entries equal to it as the half still needs, in order, go left.
// STEPS: entries per thread that are held in registers with their codes (m <= 1024 STEPS); 0: any m, both re-read per pass.
// GATHER: the workgroup picks the axis from the partial statistics and fetches the codes from the rows itself (small nodes:
// there are many workgroups); else the codes are given.
// Bound by latency: the fetch of the entries, a pass over LDS counters per digit, the stores: 18 us for 8 nodes of 32768
// entries (22 with the codes read again in every pass), 20, 13 and 11 us for 32 to 128 nodes down to 2048 entries (with the
// axis in a launch of its own 27, 19 and 16).
template <int ELT, int STEPS, bool GATHER>
__global__ void __launch_bounds__(1024)
tree_split_kernel(TreeSrc src, const uint32_t *__restrict__ order, uint32_t *__restrict__ out, const uint32_t *__restrict__ codes,
                  const double *__restrict__ partial, int64_t np, int64_t n_real, int64_t m, int c_lo, int c_hi) {
    static_assert(!GATHER || STEPS > 0, "fetched codes are held in registers");
    __shared__ uint32_t s_hist[2048];
    __shared__ int s_tot[16], s_eq[16];
    __shared__ uint32_t s_digit;
    __shared__ int s_rank;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = blockIdx.y;
    const int64_t node0 = (int64_t)blockIdx.x * m, at0 = (int64_t)bh * np + node0;
    const int steps = (int)(m / 1024), first = wave * steps * 64 + lane;   // this thread's entries: first + 64 k, k < steps
    auto pos_of = [&](int i) { return order ? order[at0 + i] : (uint32_t)(node0 + i); };
    uint32_t code[STEPS ? STEPS : 1], entry[STEPS ? STEPS : 1];
    if constexpr (STEPS > 0) {
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
            if (k < steps) entry[k] = pos_of(first + 64 * k);   // uniform conditions throughout
        if constexpr (GATHER) {
            const int ax = node_axis(partial, bh, np, m, blockIdx.x, c_lo, c_hi);
#pragma unroll
            for (int k = 0; k < STEPS; ++k)
                if (k < steps) code[k] = entry[k] < n_real ? coord_code<ELT>(src.row(bh, entry[k]), ax) : PAD_CODE<ELT>;
        } else {
#pragma unroll
            for (int k = 0; k < STEPS; ++k)
                if (k < steps) code[k] = codes[at0 + first + 64 * k];
        }
    }
    // f(i, code, entry) for this thread's entries; the conditions are the same in every lane, so f may use ballots
    auto for_codes = [&](bool entries, auto f) {
        if constexpr (STEPS > 0) {
#pragma unroll
            for (int k = 0; k < STEPS; ++k)
                if (k < steps) f(first + 64 * k, code[k], entry[k]);
        } else {
            for (int b = 0; b < steps; b += 8) {   // eight at a time
                uint32_t c[8], p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (b + u < steps) {
                        c[u] = codes[at0 + first + 64 * (b + u)];
                        p[u] = entries ? pos_of(first + 64 * (b + u)) : 0u;
                    }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (b + u < steps) f(first + 64 * (b + u), c[u], p[u]);
            }
        }
    };
    int rank = (int)(m / 2);   // the entry looked for is the rank-th smallest (from 1) of those that share `known`
    uint32_t known = 0, known_mask = 0;
    constexpr int BITS = ELT * 8;
#pragma unroll
    for (int top = BITS; top > 0; top -= 11) {
        const int shift = top > 11 ? top - 11 : 0, width = top - shift;
        s_hist[t] = 0;
        s_hist[t + 1024] = 0;
        __syncthreads();
        for_codes(false, [&](int, uint32_t c, uint32_t) {
            if ((c & known_mask) == known) atomicAdd(&s_hist[(c >> shift) & ((1u << width) - 1u)], 1u);
        });
        __syncthreads();
        const int h0 = (int)s_hist[2 * t], h1 = (int)s_hist[2 * t + 1];
        const int incl = lvr_wave_inclusive_sum(h0 + h1);
        if (lane == 63) s_tot[wave] = incl;
        __syncthreads();
        int before = incl - (h0 + h1);
        for (int w = 0; w < wave; ++w) before += s_tot[w];
        if (before < rank && rank <= before + h0 + h1) {   // exactly one thread
            const bool second = rank > before + h0;
            s_digit = 2 * t + (second ? 1 : 0);
            s_rank = rank - before - (second ? h0 : 0);
        }
        __syncthreads();
        rank = s_rank;
        known |= s_digit << shift;
        known_mask |= ((1u << width) - 1u) << shift;
    }
    // `known` is the median code, `rank` (>= 1) the number of entries equal to it that go left
    int n_lt = 0, n_eq = 0;
    for_codes(false, [&](int, uint32_t c, uint32_t) {
        n_lt += (int)__popcll(__ballot(c < known));
        n_eq += (int)__popcll(__ballot(c == known));
    });
    if (lane == 0) {
        s_tot[wave] = n_lt;
        s_eq[wave] = n_eq;
    }
    __syncthreads();
    int eq_before = 0, left_at = 0;
    for (int w = 0; w < wave; ++w) {
        left_at += s_tot[w];
        eq_before += s_eq[w];
    }
    left_at += eq_before < rank ? eq_before : rank;
    int eq_left = rank - eq_before;   // equal entries this wave may still send left
    uint32_t *ob = out + at0;
    const uint64_t below = (1ull << lane) - 1ull;
    for_codes(true, [&](int i, uint32_t c, uint32_t pos) {
        const uint64_t eq = __ballot(c == known);
        // (the count as int: eq_left goes below zero once the half has all the equal entries it needs)
        const bool left = c < known || (c == known && (int)__popcll(eq & below) < eq_left);
        const uint64_t lefts = __ballot(left);
        const int lt = left_at + (int)__popcll(lefts & below);   // entries before this one that go left
        ob[left ? lt : (int)(m / 2) + i - lt] = pos;
        left_at += (int)__popcll(lefts);
        eq_left -= (int)__popcll(eq);
    });
}

// Rows into the arena in tree order, and the two position maps.  pos_base is added to the
// positions (a chunk's positions are relative to its first row).
__global__ void tree_gather_kernel(TreeSrc ksrc, TreeSrc vsrc, const uint64_t *__restrict__ keys, char *Kdst,
                                   char *Vdst, int32_t *slot_pos, int32_t *pos_slot, int64_t np, int64_t n_real,
                                   int pos_bits, int64_t cap_rows, int64_t row0, int row_bytes) {
    const int chunks = row_bytes / 16;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_real * chunks) return;
    const int bh = blockIdx.y;
    const int64_t slot = i / chunks;
    const int ch = (int)(i % chunks);
    const int64_t pos = key_pos(keys[(int64_t)bh * np + slot], pos_bits);
    const TreeSrc &s = blockIdx.z == 0 ? ksrc : vsrc;
    char *dst = blockIdx.z == 0 ? Kdst : Vdst;
    reinterpret_cast<uint4 *>(dst + ((int64_t)bh * cap_rows + row0 + slot) * row_bytes)[ch] =
        reinterpret_cast<const uint4 *>(s.row(bh, pos))[ch];
    if (blockIdx.z == 0 && ch == 0) {
        slot_pos[(int64_t)bh * cap_rows + row0 + slot] = (int32_t)(row0 + pos);
        pos_slot[(int64_t)bh * cap_rows + row0 + pos] = (int32_t)(row0 + slot);
    }
}

// All the remaining levels of a node of at most TREE_WG_MAX padded entries in ONE launch, an entry per thread.  Either the
// whole tree of a small input (a buffer chunk of B keys: order == NULL, one workgroup per (sequence, KV head)), or
// every node of the level at which the kernels above have brought the nodes down to TREE_WG_MAX entries (the node's
// entries are np consecutive ones of `order`, in ascending position order).  Per level: statistics (a wave per 64
// entries, sixteen rows in flight), the code on the axis, and a bitonic sort of [ code | index of the entry in the node's
// initial order ] inside every node, in registers where the exchange stays inside a wave.
// Bound by the fp64 adds of the statistics and the row reads from L2, eight passes over 256 KB per workgroup at 1024
// entries and groups of four.
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_small_kernel(TreeSrc src, const uint32_t *__restrict__ order, uint64_t *__restrict__ keys_out, int64_t np_total,
                  int np, int64_t n_real, int levels, int c_lo, int c_hi) {
    typedef typename std::conditional<ELT == 2, uint32_t, uint64_t>::type key_t;
    constexpr int ENT_BITS = 10;   // TREE_WG_MAX entries
    __shared__ key_t s_key[TREE_WG_MAX];
    __shared__ int32_t s_pos[TREE_WG_MAX];    // position of an entry
    __shared__ uint16_t s_ent[TREE_WG_MAX];   // the current order: entry in every place
    __shared__ int32_t s_axis[TREE_WG_MAX / 2];
    __shared__ double s_part[16][256];   // per wave: 128 sums, 128 sums of squares
    __shared__ int s_cnt[16];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = blockIdx.y;
    const int64_t base = (int64_t)bh * np_total + (int64_t)blockIdx.x * np;   // this node's entries
    const bool mine = t < np;
    if (mine) {
        s_pos[t] = order ? (int32_t)order[base + t] : t;
        s_ent[t] = (uint16_t)t;
    }
    __syncthreads();
    const char *rows = src.row(bh, 0);
    const int64_t row_bytes = src.st * ELT;
    for (int L = 0; L < levels; ++L) {
        const int m = np >> L;
        // 1. split axis of every node: sums relative to the node's first key (padding sorts last: it is real unless the
        // whole node is padding)
        const int mypos = mine ? s_pos[s_ent[t]] : 0x7fffffff;
        const uint64_t real = __ballot(mine && mypos < n_real);
        if (m >= 64) {
            double s0 = 0., s1 = 0., q0 = 0., q1 = 0.;
            if (real) {   // uniform
                const int ppos = s_pos[s_ent[wave * 64 / m * m]];
                float p0, p1;
                lane_pair<ELT>(rows + ppos * row_bytes, lane, p0, p1);
                sum_rows64<ELT>(src, bh, lane, mypos, real, ppos, p0, p1, s0, s1, q0, q1);
            }
            double *o = s_part[wave];
            o[2 * lane] = s0; o[2 * lane + 1] = s1;
            o[128 + 2 * lane] = q0; o[128 + 2 * lane + 1] = q1;
            if (lane == 0) s_cnt[wave] = __popcll(real);
            __syncthreads();
            if (wave < (1 << L)) {   // wave w adds the runs of node w in order
                const int runs = m / 64;
                s0 = s1 = q0 = q1 = 0.;
                int cnt = 0;
                for (int k = wave * runs; k < (wave + 1) * runs; ++k) {
                    s0 += s_part[k][2 * lane]; s1 += s_part[k][2 * lane + 1];
                    q0 += s_part[k][128 + 2 * lane]; q1 += s_part[k][128 + 2 * lane + 1];
                    cnt += s_cnt[k];
                }
                const double inv = cnt > 0 ? 1.0 / (double)cnt : 0.;
                const int arg = wave_argmax((q0 - s0 * s0 * inv) * inv, (q1 - s1 * s1 * inv) * inv, lane, c_lo, c_hi);
                if (lane == 0) s_axis[wave] = arg;
            }
        } else if (real) {   // several nodes per wave, one after the other; sixteen rows in flight whatever the node's size
            auto nodes = [&](auto rows_c) {   // rows_c = entries of a node within a batch of sixteen
                constexpr int RW = decltype(rows_c)::value;
                double s0 = 0., s1 = 0., q0 = 0., q1 = 0.;
                float p0 = 0.f, p1 = 0.f;
                int cnt = 0;
                const int some = __builtin_amdgcn_readlane(mypos, 0);   // real: the wave's first entry
                for (int j0 = 0; j0 < 64 && wave * 64 + j0 < np; j0 += 16) {
                    float x0[16], x1[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        const int pos = __builtin_amdgcn_readlane(mypos, j0 + u);
                        const bool in = (real >> (j0 + u)) & 1ull;
                        lane_pair<ELT>(rows + (int64_t)(in ? pos : some) * row_bytes, lane, x0[u], x1[u]);
                    }
#pragma unroll
                    for (int k = 0; k < 16 / RW; ++k) {
                        const int at = j0 + k * RW;   // first entry of this part of a node
                        if ((at & (m - 1)) == 0) {
                            p0 = x0[k * RW]; p1 = x1[k * RW];
                            s0 = s1 = q0 = q1 = 0.;
                            cnt = 0;
                        }
#pragma unroll
                        for (int u = 0; u < RW; ++u) {
                            const bool in = (real >> (at + u)) & 1ull;
                            const double d0 = in ? (double)x0[k * RW + u] - (double)p0 : 0.;
                            const double d1 = in ? (double)x1[k * RW + u] - (double)p1 : 0.;
                            s0 += d0; s1 += d1; q0 += d0 * d0; q1 += d1 * d1;
                            cnt += in ? 1 : 0;
                        }
                        if (((at + RW) & (m - 1)) == 0 && wave * 64 + at < np) {   // the node's last part
                            const double inv = cnt > 0 ? 1.0 / (double)cnt : 0.;
                            const int arg = wave_argmax((q0 - s0 * s0 * inv) * inv, (q1 - s1 * s1 * inv) * inv, lane, c_lo, c_hi);
                            if (lane == 0) s_axis[(wave * 64 + at) / m] = arg;
                        }
                    }
                }
            };
            if (m == 2) nodes(std::integral_constant<int, 2>{});
            else if (m == 4) nodes(std::integral_constant<int, 4>{});
            else if (m == 8) nodes(std::integral_constant<int, 8>{});
            else nodes(std::integral_constant<int, 16>{});
        }
        __syncthreads();
        // 2. this thread's entry: [ code on its node's axis | entry ]
        key_t key = ~(key_t)0;
        if (mine) {
            const uint32_t code = mypos < n_real ? coord_code<ELT>(rows + (int64_t)mypos * row_bytes, s_axis[t / m]) : PAD_CODE<ELT>;
            key = ((key_t)code << ENT_BITS) | (key_t)s_ent[t];
        }
        // 3. ascending bitonic sort inside every node (nodes are aligned runs of m = 2^x entries)
        for (int k = 2; k <= m; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                key_t other;
                if (j >= 64) {
                    __syncthreads();
                    s_key[t] = key;
                    __syncthreads();
                    other = s_key[t ^ j];
                } else {
                    other = __shfl_xor(key, j, 64);
                }
                const bool up = k == m || (t & k) == 0;   // the last merge of every node ascends
                const bool low = (t & j) == 0;
                key = (low == up) ? (key < other ? key : other) : (key < other ? other : key);
            }
        }
        if (mine) s_ent[t] = (uint16_t)(key & (key_t)(TREE_WG_MAX - 1));
        __syncthreads();
    }
    if (mine) keys_out[base + t] = (uint64_t)(uint32_t)s_pos[s_ent[t]];
}

int bits_for(int64_t v) {   // bits needed to hold values 0 .. v-1
    int b = 0;
    while (((int64_t)1 << b) < v) ++b;
    return b;
}

// The two work arrays: a = the order before and after a split (32-bit positions, two halves), b = the codes of a level
// (32 bits each), at the end the finished order as 64-bit keys.
template <int ELT>
hipError_t tree_order_t(lvr_index *ix, const TreeSrc &src, int64_t n_real, int64_t np, int levels, int c_lo, int c_hi,
                        hipStream_t st) {
    const int n_bh = lvr_n_bh(ix);
    uint32_t *cur = nullptr;   // the order at the start: entry i holds position i
    uint32_t *half[2] = {reinterpret_cast<uint32_t *>(ix->tree_keys_a),
                         reinterpret_cast<uint32_t *>(ix->tree_keys_a) + ix->tree_cap_keys};
    uint32_t *codes = reinterpret_cast<uint32_t *>(ix->tree_keys_b);
    int L = 0;
    for (; (np >> L) > TREE_WG_MAX; ++L) {   // np is a power of two: every node here holds a multiple of 2048 entries
        const int64_t n_nodes = (int64_t)1 << L, m = np >> L;
        hipLaunchKernelGGL(tree_stats_piece_kernel<ELT>, dim3((unsigned)(np / PIECE), (unsigned)n_bh), dim3(1024), 0, st, src,
                           cur, ix->tree_partial, np, n_real, m);
        uint32_t *next = half[L & 1];
        const dim3 nodes((unsigned)n_nodes, (unsigned)n_bh);
        // nodes of more than 8192 entries leave most of the device idle in the split launch (a workgroup fetches a
        // coordinate of 64 different rows at about one row per clock): there the codes are a launch of their own
        if (m > 8192) {
            hipLaunchKernelGGL(tree_axis_kernel, nodes, dim3(1024), 0, st, ix->tree_partial, ix->tree_axis, np, m, n_nodes, c_lo, c_hi);
            hipLaunchKernelGGL(tree_codes_kernel<ELT>, dim3((unsigned)(np / 256), (unsigned)n_bh), dim3(256), 0, st, src, cur,
                               codes, ix->tree_axis, np, n_real, m, n_nodes);
            if (m <= 32768)
                hipLaunchKernelGGL((tree_split_kernel<ELT, 32, false>), nodes, dim3(1024), 0, st, src, cur, next, codes,
                                   ix->tree_partial, np, n_real, m, c_lo, c_hi);
            else
                hipLaunchKernelGGL((tree_split_kernel<ELT, 0, false>), nodes, dim3(1024), 0, st, src, cur, next, codes,
                                   ix->tree_partial, np, n_real, m, c_lo, c_hi);
        } else {
            hipLaunchKernelGGL((tree_split_kernel<ELT, 8, true>), nodes, dim3(1024), 0, st, src, cur, next, codes,
                               ix->tree_partial, np, n_real, m, c_lo, c_hi);
        }
        cur = next;
    }
    const int64_t m0 = np >> L;   // entries of a node that one workgroup finishes
    const unsigned threads = m0 <= 64 ? 64u : (unsigned)m0;
    hipLaunchKernelGGL(tree_small_kernel<ELT>, dim3((unsigned)(np / m0), (unsigned)n_bh), dim3(threads), 0, st, src, cur,
                       ix->tree_keys_b, np, (int)m0, n_real, levels - L, c_lo, c_hi);
    return hipGetLastError();
}

}  // namespace

// Which inputs the tree takes: node number, coordinate code and position together have to fit 64 bits, and the work space the
// padded entries.  Only the second is a need of the kernels above, which keep codes and positions apart; the first is the
// limit of the entry points (LVR_E_UNSUPPORTED beyond it) since the construction sorted one 64-bit key per entry, and stands
// so that the same calls are refused.
bool lvr_tree_feasible(const lvr_index *ix, int64_t n_real) {
    if (n_real <= 0) return true;
    const int r = ix->cfg.group_size;
    const int n_bh = lvr_n_bh(ix);
    int64_t groups = n_real / r, gp = 1;
    while (gp < groups) gp <<= 1;
    const int64_t np = gp * r;
    const int pos_bits = bits_for(np);
    const int coord_bits = ix->elt == 2 ? 16 : 32;
    int levels = 0;
    while (((int64_t)1 << levels) < gp) ++levels;
    const int node_bits = bits_for((int64_t)n_bh << (levels > 0 ? levels - 1 : 0));
    return pos_bits + coord_bits + node_bits <= 64 && (int64_t)n_bh * np <= ix->tree_cap_keys;
}

// Orders n_real = groups*r keys (positions 0..n_real-1 of the given source rows) by the tree; perm->keys then holds, per
// (sequence, KV head), the position stored in every slot.  Returns hipErrorInvalidValue if lvr_tree_feasible says no.
hipError_t lvr_tree_order(lvr_index *ix, const void *Ksrc, const int64_t ks[3], int64_t n_real, hipStream_t st,
                          lvr_tree_perm *perm, int c_lo, int c_hi) {
    perm->keys = nullptr;
    if (n_real <= 0) return hipSuccess;
    if (!lvr_tree_feasible(ix, n_real)) return hipErrorInvalidValue;
    const int r = ix->cfg.group_size;
    int64_t groups = n_real / r, gp = 1;
    while (gp < groups) gp <<= 1;
    const int64_t np = gp * r;                         // padded entries per (sequence, KV head)
    int levels = 0;
    while (((int64_t)1 << levels) < gp) ++levels;       // nodes of r entries after `levels` splits
    const TreeSrc src{static_cast<const char *>(Ksrc), ks[0], ks[1], ks[2], (int)ix->elt, ix->cfg.n_kv_heads};
    const hipError_t e = ix->elt == 2 ? tree_order_t<2>(ix, src, n_real, np, levels, c_lo, c_hi, st)
                                      : tree_order_t<4>(ix, src, n_real, np, levels, c_lo, c_hi, st);
    if (e != hipSuccess) return e;
    perm->keys = ix->tree_keys_b;
    perm->np = np;
    perm->pos_bits = bits_for(np);
    return hipSuccess;
}

hipError_t lvr_tree_gather(lvr_index *ix, const void *Ksrc, const int64_t ks[3], const void *Vsrc, const int64_t vs[3],
                           const lvr_tree_perm *perm, int64_t n_real, int64_t row0, hipStream_t st) {
    if (n_real <= 0 || !perm->keys) return hipSuccess;
    const int n_bh = lvr_n_bh(ix);
    TreeSrc ksrc{static_cast<const char *>(Ksrc), ks[0], ks[1], ks[2], (int)ix->elt, ix->cfg.n_kv_heads};
    TreeSrc vsrc{static_cast<const char *>(Vsrc), vs[0], vs[1], vs[2], (int)ix->elt, ix->cfg.n_kv_heads};
    const int row_bytes = (int)(LVR_D * ix->elt);
    const int64_t total = n_real * (row_bytes / 16);
    hipLaunchKernelGGL(tree_gather_kernel, dim3((unsigned)((total + 255) / 256), (unsigned)n_bh, 2), dim3(256), 0, st,
                       ksrc, vsrc, perm->keys, static_cast<char *>(ix->K), static_cast<char *>(ix->V), ix->slot_pos,
                       ix->pos_slot, perm->np, n_real, perm->pos_bits, ix->cap_rows, row0, row_bytes);
    return hipGetLastError();
}

hipError_t lvr_tree_group(lvr_index *ix, const void *Ksrc, const int64_t ks[3], const void *Vsrc, const int64_t vs[3],
                          int64_t n_real, int64_t row0, hipStream_t st) {
    lvr_tree_perm perm;
    hipError_t e = lvr_tree_order(ix, Ksrc, ks, n_real, st, &perm);
    if (e != hipSuccess) return e;
    return lvr_tree_gather(ix, Ksrc, ks, Vsrc, vs, &perm, n_real, row0, st);
}
