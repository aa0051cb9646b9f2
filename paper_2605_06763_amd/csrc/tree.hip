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
// Only which entries go left matters above the last level, so nodes larger than tree_small_kernel takes (512 entries of bf16
// keys, 256 of fp32 ones) are not sorted: their workgroups find the median code by counting digits and move the
// entries to the two halves in the order they had.  Every node's entries therefore stay in ascending
// position order, which is what breaks ties and keeps the padding at a node's end.  The levels below are
// finished by tree_small_kernel in one launch, a workgroup per node, which sorts, so a finished group's rows are in the
// order of the last split.
//
// Variances come from sums and sums of squares in fp64, and only the left half of a node's rows is added up for the level below:
// the right half's sums are the node's less those, unless so little is left of them that the node's own rows are asked (unsure).
//
// A build of 8 x 32768 bf16 keys in groups of four and one step, us: 2321 with one wave per SIMD on the statistics, a device-wide radix
// sort per level and four waves per small node; 424 with a workgroup per node that splits, statistics over all rows in a launch per
// level, and small nodes of 1024 entries whose rows came from memory at every level; 302 without the question whether sums
// tell (unsure), 304 with it.  Builds alone, that form and this one: 2048 keys 176 / 81 (4 x 4 heads), 9000 keys 276 / 157 (2 heads), 32768
// fp32 keys 553 / 417, 131072 keys 1574 / 1245; one tree per coordinate block, S = 16, 32768 keys 5514 / 3761 (without the question,
// which costs a build 0.4 to 2.5 %, fp32 keys most).
#include <type_traits>

#include "lvr_internal.h"

namespace {

constexpr int PIECE = 1024;          // entries whose rows a workgroup adds up
// entries of a node whose workgroups each fetch the codes of all of it: every further time that all codes are fetched costs some 5 us (a line per
// coordinate: 33 MB for 8 x 32768 keys), a launch of its own with the fetch 8.8 us.  A level of 8 x 32768 keys, us: nodes of 4096 32.5 gathered by
// their four workgroups, 23.6 with the codes in a launch of their own; nodes of 2048 21.5 and 24
constexpr int GATHER_MAX = 2048;
template <int ELT>
constexpr int SMALL_NODE = ELT == 2 ? 512 : 256;   // entries of a node that one workgroup finishes: 128 KB of rows
template <int ELT>
using code_t = typename std::conditional<ELT == 2, uint16_t, uint32_t>::type;

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
using row_piece = typename std::conditional<ELT == 2, uint32_t, float2>::type;
template <int ELT>
__device__ __forceinline__ void unpack_pair(const row_piece<ELT> &w, float &x0, float &x1) {
    if constexpr (ELT == 2) {
        x0 = lvr_bf16_lo(w);
        x1 = lvr_bf16_hi(w);
    } else {
        x0 = w.x;
        x1 = w.y;
    }
}
template <int ELT>
__device__ __forceinline__ void lane_pair(const char *row, int lane, float &x0, float &x1) {
    unpack_pair<ELT>(reinterpret_cast<const row_piece<ELT> *>(row)[lane], x0, x1);
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

// Largest of a wave's values (lane 63 holds it, every lane gets it).
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    auto with = [&](auto ctrl, auto rows) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        v = v > o ? v : o;
    };
    with(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr:1, 2, 4, 8: lane 15 of a row
    with(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});   // holds the row's maximum
    with(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    with(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    with(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15, row_bcast:31
    with(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// argmax over 128 channel variances (>= 0) held as (v0, v1) per lane; lowest channel wins ties.
// [c_lo, c_hi): the coordinates that may be chosen (a tree over one coordinate block looks at that block only).
// Non-negative doubles are ordered as their bits are: the upper words decide, the lower ones only where those tie.  `top`: the largest's upper word.
__device__ __forceinline__ int wave_argmax(double v0, double v1, int lane, int c_lo, int c_hi, int &top) {
    const bool may0 = 2 * lane >= c_lo && 2 * lane < c_hi, may1 = 2 * lane + 1 >= c_lo && 2 * lane + 1 < c_hi;
    const uint64_t u0 = (uint64_t)__double_as_longlong(v0), u1 = (uint64_t)__double_as_longlong(v1);
    const uint32_t h0 = may0 ? (uint32_t)(u0 >> 32) + 1u : 0u, h1 = may1 ? (uint32_t)(u1 >> 32) + 1u : 0u;
    const uint32_t best = wave_max(h0 > h1 ? h0 : h1);
    top = (int)best - 1;
    uint64_t b0 = __ballot(h0 == best), b1 = __ballot(h1 == best);
    if ((int)__popcll(b0) + (int)__popcll(b1) > 1) {   // uniform
        const uint32_t l0 = h0 == best ? (uint32_t)u0 : 0u, l1 = h1 == best ? (uint32_t)u1 : 0u;
        const uint32_t low = wave_max(l0 > l1 ? l0 : l1);
        b0 = __ballot(h0 == best && (uint32_t)u0 == low);
        b1 = __ballot(h1 == best && (uint32_t)u1 == low);
    }
    const int a0 = b0 ? 2 * __builtin_ctzll(b0) : 2 * 64, a1 = b1 ? 2 * __builtin_ctzll(b1) + 1 : 2 * 64;
    return a0 < a1 ? a0 : a1;
}

// Variances of a node's 128 channels from its sums, times the square of the number of keys (the same factor for all of them):
// n q - s^2, with the rounding of the product carried along, so that sums that are exact (bf16 keys, whole numbers) give variances that
// are equal where they should be.  Never negative; what is no number counts as zero.
__device__ __forceinline__ double spread(double s, double q, double n) {
    const double p = s * s;
    return fmax(fma(n, q, -p) - fma(s, s, -p), 0.0);
}

// Upper word of the largest of a node's sums of squares over the coordinates that may be chosen (beyond every number where one of them
// is no number).
__device__ __forceinline__ int largest_square(double q0, double q1, int lane, int c_lo, int c_hi) {
    const bool may0 = 2 * lane >= c_lo && 2 * lane < c_hi, may1 = 2 * lane + 1 >= c_lo && 2 * lane + 1 < c_hi;
    const uint32_t h0 = may0 ? (uint32_t)((uint64_t)__double_as_longlong(q0) >> 32) & 0x7fffffffu : 0u;
    const uint32_t h1 = may1 ? (uint32_t)((uint64_t)__double_as_longlong(q1) >> 32) & 0x7fffffffu : 0u;
    return (int)wave_max(h0 > h1 ? h0 : h1);
}

// Whether the largest spread of a node of m = 2^log_m keys (its upper word: top) may be made of rounding errors.  They are some 2^-53 m times
// the sum of squares that the node's sums descend from, its own or, for differences, that of the last node above it whose rows were added up (`mag`:
// the upper word of the largest).  22 binades between spread and square leave the largest variance good to about 1e-9.  Keys whose mean is 16 times
// their deviation, seven right halves below the last rows added up, need 15 of them.  Where there are more, a key far off went left (its square, or
// its infinity, is still in the difference), all keys are the same, or the shift is far from all of them: then the
// node's own rows are added up, relative to its own first key.
__device__ __forceinline__ bool unsure(int top, int mag, int log_m) { return top < mag + ((log_m - 22) << 20); }

// What is taken off every coordinate before it is squared: nothing for bf16 keys, whose rows' sums are exact in fp64 wherever squares
// of the mean cancel (eight significant bits); for fp32 ones a value among the tree's keys.
struct Shift {
    double p0, p1;
};

// Sums relative to `from`, of n keys, as sums relative to `to`.
__device__ __forceinline__ void shift_sums(double &s, double &q, double n, double from, double to) {
    const double d = from - to;
    q += d * (2.0 * s + n * d);
    s += n * d;
}

// Adds the rows held in (x0, x1) to the sums.
template <int ELT, int N>
__device__ __forceinline__ void add_rows(const float (&x0)[N], const float (&x1)[N], const Shift &p, double &s0, double &s1, double &q0,
                                         double &q1) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
        double d0 = (double)x0[u], d1 = (double)x1[u];
        if constexpr (ELT == 4) {
            d0 -= p.p0;
            d1 -= p.p1;
        }
        s0 += d0; s1 += d1; q0 = fma(d0, d0, q0); q1 = fma(d1, d1, q1);
    }
}

// Sums of the up to 64 entries whose positions the lanes hold; the next sixteen rows are requested before sixteen are added up.
// `real`: ballot of the lanes whose entry is no padding, a prefix of them.
template <int ELT>
__device__ __forceinline__ void sum_rows64(const TreeSrc &src, int bh, int lane, int mypos, uint64_t real, const Shift &p, double &s0,
                                           double &s1, double &q0, double &q1) {
    const char *base = src.row(bh, 0);
    const int64_t row_bytes = src.st * ELT;
    const int n = (int)__popcll(real);
    row_piece<ELT> w[2][16];
    auto fetch = [&](int j0, row_piece<ELT>(&x)[16]) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int pos = __builtin_amdgcn_readlane(mypos, j0 + u);
            x[u] = reinterpret_cast<const row_piece<ELT> *>(base + (int64_t)(j0 + u < n ? pos : 0) * row_bytes)[lane];
        }
        __builtin_amdgcn_sched_barrier(0);   // requested here, not next to their use
    };
    auto add = [&](int j0, const row_piece<ELT>(&x)[16]) {
        float x0[16], x1[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) unpack_pair<ELT>(x[u], x0[u], x1[u]);
        if (j0 + 16 > n) {   // uniform: what is masked adds nothing
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                x0[u] = j0 + u < n ? x0[u] : (float)p.p0;   // (the shift is a key's coordinate: exact)
                x1[u] = j0 + u < n ? x1[u] : (float)p.p1;
            }
        }
        add_rows<ELT>(x0, x1, p, s0, s1, q0, q1);
    };
    if (n > 0) fetch(0, w[0]);   // uniform conditions throughout
#pragma unroll
    for (int j0 = 0; j0 < 64; j0 += 16) {
        if (j0 + 16 < 64 && n > j0 + 16) fetch(j0 + 16, w[(j0 / 16 + 1) & 1]);
        if (n > j0) add(j0, w[(j0 / 16) & 1]);
    }
}

// A row of keys as a shift, where there is one.
template <int ELT>
__device__ __forceinline__ Shift shift_of(const char *row, int lane) {
    float x0 = 0.f, x1 = 0.f;
    if constexpr (ELT == 4) lane_pair<ELT>(row, lane, x0, x1);
    return Shift{(double)x0, (double)x1};
}

// The shift of every node above the small ones: in every channel the middle one of the first, a middle and the last key's values,
// so that one key far from the others (often the first) does not move it.
template <int ELT>
__device__ __forceinline__ Shift tree_shift(const TreeSrc &src, int bh, int lane, int64_t n_real) {
    Shift p = {0.0, 0.0};
    if constexpr (ELT == 4) {
        float a0, a1, b0, b1, c0, c1;
        lane_pair<ELT>(src.row(bh, 0), lane, a0, a1);
        lane_pair<ELT>(src.row(bh, n_real >> 1), lane, b0, b1);
        lane_pair<ELT>(src.row(bh, n_real - 1), lane, c0, c1);
        p.p0 = (double)fmaxf(fminf(a0, b0), fminf(fmaxf(a0, b0), c0));   // (a NaN among them is passed over)
        p.p1 = (double)fmaxf(fminf(a1, b1), fminf(fmaxf(a1, b1), c1));
    }
    return p;
}

// The waves' sums of a workgroup, added in order and stored as 256 doubles: 128 sums, 128 sums of squares.
template <int NW>
__device__ __forceinline__ void store_partial(double (*sm)[256], int lane, int wave, int waves, double s0, double s1, double q0, double q1,
                                              double *out) {
    sm[wave][2 * lane] = s0; sm[wave][2 * lane + 1] = s1;
    sm[wave][128 + 2 * lane] = q0; sm[wave][128 + 2 * lane + 1] = q1;
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 256) {
        double a = 0.;
#pragma unroll
        for (int w = 0; w < NW; ++w) a += w < waves ? sm[w][t] : 0.;
        out[t] = a;
    }
}

// Sums of whole pieces of PIECE entries: the root, and the nodes below one that was split by a single workgroup.  order == NULL:
// entry i holds position i.  (Everywhere else the launch that splits a node adds up the rows that go left, see below.)
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_stats_piece_kernel(TreeSrc src, const uint32_t *__restrict__ order, double *__restrict__ partial, int64_t np, int64_t n_real) {
    __shared__ double sm[16][256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int bh = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t *ord = order + (int64_t)bh * np;
    const int mypos = order ? (int)ord[i] : (int)i;
    const uint64_t real = __ballot(mypos < n_real);
    double s0 = 0., s1 = 0., q0 = 0., q1 = 0.;
    if (real) sum_rows64<ELT>(src, bh, lane, mypos, real, tree_shift<ELT>(src, bh, lane, n_real), s0, s1, q0, q1);   // uniform
    store_partial<16>(sm, lane, wave, (int)(blockDim.x >> 6), s0, s1, q0, q1, partial + ((int64_t)bh * gridDim.x + blockIdx.x) * 256);
}

// The sums a level starts from.  `whole`: the pieces' sums cover their entries; else they cover the rows of the parents' level that
// went left, so a left node adds up its parent's pieces and a right one takes them off its parent's sums.
struct LevelSums {
    const double *pieces;   // [n_bh][pieces of the tree][256]
    const double *parent;   // [n_bh][nodes of the level above][256]
    double *own;            // [n_bh][nodes of this level][256], or NULL where no level below needs them (then there may be more nodes than room)
    const int *parent_mag;  // [n_bh][nodes of the level above]: what the rounding errors of their sums are measured by (unsure)
    int *own_mag;
    int64_t n_pieces;
    int whole;
};

// Sums of the n real entries of a node (`order`: theirs, or NULL where entry i holds position node0 + i), relative to p, by a workgroup of NT threads;
// threads 0 to 63 get those of their two channels.  Sixteen rows of every wave in flight.
template <int ELT, int NT>
__device__ __forceinline__ void own_sums(const TreeSrc &src, int bh, const uint32_t *__restrict__ order, int64_t node0, int64_t n, const Shift &p,
                                         double (&sm)[NT / 128][256], double &s0, double &s1, double &q0, double &q1) {
    constexpr int SL = NT / 128;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const char *base = src.row(bh, 0);
    const int64_t row_bytes = src.st * ELT;
    s0 = s1 = q0 = q1 = 0.;
    for (int64_t e0 = wave * 64; e0 < n; e0 += NT) {   // uniform over the wave
        const int rows = n - e0 < 64 ? (int)(n - e0) : 64;
        const int mypos = lane < rows ? (order ? (int)order[e0 + lane] : (int)(node0 + e0 + lane)) : 0;
        for (int j0 = 0; j0 < rows; j0 += 16) {
            row_piece<ELT> w[16];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                w[u] = reinterpret_cast<const row_piece<ELT> *>(base + (int64_t)__builtin_amdgcn_readlane(mypos, j0 + u < rows ? j0 + u : 0) * row_bytes)[lane];
            __builtin_amdgcn_sched_barrier(0);   // all of them requested before the first is used
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                float x0[1], x1[1];
                unpack_pair<ELT>(w[u], x0[0], x1[0]);
                if (j0 + u < rows) add_rows<ELT>(x0, x1, p, s0, s1, q0, q1);   // uniform
            }
        }
    }
    double *mine = sm[wave % SL];   // SL slices, twice as many waves
    __syncthreads();
    if (wave < SL) {
        mine[2 * lane] = s0; mine[2 * lane + 1] = s1;
        mine[128 + 2 * lane] = q0; mine[128 + 2 * lane + 1] = q1;
    }
    __syncthreads();
    if (wave >= SL) {
        mine[2 * lane] += s0; mine[2 * lane + 1] += s1;
        mine[128 + 2 * lane] += q0; mine[128 + 2 * lane + 1] += q1;
    }
    __syncthreads();
    if (t < 64) {
        s0 = s1 = q0 = q1 = 0.;
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            s0 += sm[k][2 * t]; s1 += sm[k][2 * t + 1];
            q0 += sm[k][128 + 2 * t]; q1 += sm[k][128 + 2 * t + 1];
        }
    }
}

// The axis of a node (every thread gets it); the first workgroup of a node also stores its sums for the level below.  NT threads.
// Where the sums do not tell (unsure), each of the node's workgroups adds up all of its rows: no launch and no trip more where they do.  Builds of
// 8 x 32768 bf16 keys, us: 270, with a key of -1e8 in every head 584 (its right-hand siblings ask, one node per level), all keys the same 700
// (every right half asks).  Statistics over all rows at every level: 388, 388 and 489; differences without the question: 268, 269 and 338,
// and in 73 of 126 builds with a key far off nodes that were not split on their widest axis.
template <int ELT, int NT>
__device__ __forceinline__ int node_axis(const LevelSums &a, const TreeSrc &src, const uint32_t *__restrict__ order, int bh, int64_t np, int64_t m,
                                         int64_t node, int64_t n_nodes, int64_t n_real, bool store, int c_lo, int c_hi) {
    constexpr int SL = NT / 128;   // slices of the pieces side by side
    __shared__ double sm[SL][256];
    __shared__ int s_axis;
    const int t = threadIdx.x, c = t & 127, sl = t >> 7;
    const int64_t up = a.whole ? m : 2 * m;   // entries the pieces to be added cover
    const int64_t count = up > PIECE ? up / PIECE : 1, first = (a.whole ? node : node >> 1) * count;
    const double *pp = a.pieces + ((int64_t)bh * a.n_pieces + first) * 256;
    const bool right = !a.whole && (node & 1);
    double e0 = 0., e1 = 0., f0 = 0., f1 = 0.;
    int mag = 0;
    if (right && t < 64) {
        mag = a.parent_mag[(int64_t)bh * (n_nodes >> 1) + (node >> 1)];
        const double *e = a.parent + ((int64_t)bh * (n_nodes >> 1) + (node >> 1)) * 256;
        e0 = e[2 * t]; e1 = e[2 * t + 1];
        f0 = e[128 + 2 * t]; f1 = e[128 + 2 * t + 1];
    }
    double s = 0.0, q = 0.0;
#pragma unroll 4
    for (int64_t p = sl; p < count; p += SL) {
        s += pp[p * 256 + c];
        q += pp[p * 256 + 128 + c];
    }
    sm[sl][c] = s;
    sm[sl][128 + c] = q;
    __syncthreads();
    int64_t n = n_real - node * m;   // real keys fill a prefix of the entries
    n = n < 0 ? 0 : (n > m ? m : n);
    auto finish = [&](double s0, double s1, double q0, double q1, int mag, int axis) {   // threads 0 to 63
        if (t == 0) s_axis = axis;
        if (!store || !a.own) return;
        double *o = a.own + ((int64_t)bh * n_nodes + node) * 256;
        o[2 * t] = s0; o[2 * t + 1] = s1;
        o[128 + 2 * t] = q0; o[128 + 2 * t + 1] = q1;
        if (t == 0) a.own_mag[(int64_t)bh * n_nodes + node] = mag;
    };
    if (t < 64) {
        double s0 = 0., s1 = 0., q0 = 0., q1 = 0.;
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            s0 += sm[k][2 * t]; s1 += sm[k][2 * t + 1];
            q0 += sm[k][128 + 2 * t]; q1 += sm[k][128 + 2 * t + 1];
        }
        if (right) {
            s0 = e0 - s0; s1 = e1 - s1;
            q0 = f0 - q0; q1 = f1 - q1;
        }
        int top;
        const int ax = wave_argmax(spread(s0, q0, (double)n), spread(s1, q1, (double)n), t, c_lo, c_hi, top);
        if (!right) mag = largest_square(q0, q1, t, c_lo, c_hi);
        // (one key has no axis; sums of bf16 rows are as good as sums relative to one of them)
        const bool ask = n > 1 && (ELT == 4 || right) && unsure(top, mag, __builtin_ctzll(m));
        finish(s0, s1, q0, q1, mag, ask ? -1 : ax);
    }
    __syncthreads();
    int axis = s_axis;
    if (axis < 0) {   // uniform
        const uint32_t *ord = order ? order + (int64_t)bh * np + node * m : nullptr;
        const int lane = t & 63;
        const Shift p = shift_of<ELT>(src.row(bh, ord ? (int64_t)ord[0] : node * m), lane);
        double s0, s1, q0, q1;
        own_sums<ELT, NT>(src, bh, ord, node * m, n, p, sm, s0, s1, q0, q1);
        if (t < 64) {
            int top;
            const int ax = wave_argmax(spread(s0, q0, (double)n), spread(s1, q1, (double)n), t, c_lo, c_hi, top);
            if constexpr (ELT == 4) {
                const Shift to = tree_shift<ELT>(src, bh, lane, n_real);
                shift_sums(s0, q0, (double)n, p.p0, to.p0);
                shift_sums(s1, q1, (double)n, p.p1, to.p1);
            }
            finish(s0, s1, q0, q1, largest_square(q0, q1, t, c_lo, c_hi), ax);
        }
        __syncthreads();
        axis = s_axis;
    }
    return axis;
}

// The axis of every node that a single workgroup splits.
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_axis_kernel(TreeSrc src, const uint32_t *__restrict__ order, LevelSums sums, int32_t *__restrict__ axis, int64_t np, int64_t m, int64_t n_nodes,
                 int64_t n_real, int c_lo, int c_hi) {
    const int a = node_axis<ELT, 1024>(sums, src, order, blockIdx.y, np, m, blockIdx.x, n_nodes, n_real, false, c_lo, c_hi);
    if (threadIdx.x == 0) axis[(int64_t)blockIdx.y * n_nodes + blockIdx.x] = a;
}

// Code of every entry on its node's axis, and how often each value of a code's upper eight bits occurs in every piece, for nodes
// so large that the whole device should fetch the coordinates (a workgroup fetches a coordinate of 64 different rows at
// about one row per clock).  axis == NULL: the workgroup picks it from the sums itself.
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_codes_kernel(TreeSrc src, const uint32_t *__restrict__ order, code_t<ELT> *__restrict__ codes, uint32_t *__restrict__ hist,
                  const int32_t *__restrict__ axis, LevelSums sums, int64_t np, int64_t n_real, int64_t m, int64_t n_nodes, int c_lo, int c_hi) {
    __shared__ uint32_t s_hist[256];
    const int t = threadIdx.x, bh = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * PIECE + t, at = (int64_t)bh * np + i;
    const int64_t node = i / m;   // the same in every thread
    if (t < 256) s_hist[t] = 0;
    const int64_t pos = order ? (int64_t)order[at] : i;
    const int ax = axis ? axis[(int64_t)bh * n_nodes + node]
                        : node_axis<ELT, 1024>(sums, src, order, bh, np, m, node, n_nodes, n_real, (int64_t)blockIdx.x * PIECE == node * m, c_lo, c_hi);
    const uint32_t c = pos < n_real ? coord_code<ELT>(src.row(bh, pos), ax) : PAD_CODE<ELT>;
    codes[at] = (code_t<ELT>)c;
    if (axis) return;   // uniform
    atomicAdd(&s_hist[c >> (ELT * 8 - 8)], 1u);   // (cleared before the barriers of node_axis)
    __syncthreads();
    if (t < 256) hist[((int64_t)bh * (np / PIECE) + blockIdx.x) * 256 + t] = s_hist[t];
}

// One digit of the search for the code of a node's median: s_hist holds how often each of 2048 values of the digit occurs among the
// entries looked at, `rank` (from 1) counts among them.  Returns the digit and leaves the rank among the entries that have it.
template <int NT>
__device__ __forceinline__ uint32_t pick_digit(uint32_t (&s_hist)[2048], int lane, int wave, int &rank) {
    constexpr int BPT = 2048 / NT;   // values per thread
    __shared__ int s_tot[NT / 64], s_rank;
    __shared__ uint32_t s_digit;
    const int t = threadIdx.x;
    int h[BPT], sum = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
        h[j] = (int)s_hist[BPT * t + j];
        sum += h[j];
    }
    const int incl = lvr_wave_inclusive_sum(sum);
    if (lane == 63) s_tot[wave] = incl;
    __syncthreads();
    int before = incl - sum;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) before += w < wave ? s_tot[w] : 0;
    if (before < rank && rank <= before + sum) {   // exactly one thread
#pragma unroll
        for (int j = 0; j < BPT; ++j) {
            if (before < rank && rank <= before + h[j]) {
                s_digit = (uint32_t)(BPT * t + j);
                s_rank = rank - before;
            }
            before += h[j];
        }
    }
    __syncthreads();
    rank = s_rank;
    return s_digit;
}

// Splits nodes of m entries (NT to 32768) at their median, a workgroup of NT threads per NT entries.  Every workgroup of a node
// finds the node's median code for itself, from all the node's codes (digit by digit, in registers and LDS counters),
// and then sends its own entries left or right: entries below the median, and as many equal to it as the half still needs, in
// order, go left.  The rows that go left are added up on the way (part_out, unless NULL): a level's statistics take half of the rows, and
// no launch of their own.
// GATHER: the codes are fetched from the rows of the whole node by each of its workgroups, and the axis is picked from the sums
// (nodes of up to STEPS workgroups, where that costs less than a launch); else codes and the counts of their upper eight bits
// come from tree_codes_kernel.
// Bound by a chain of short stretches (8 x 32768 keys, nodes of 16384, from timestamps): codes 0.9 us, two digits 2.5 and 2.1, the partition 1.9,
// the rows 5 (2.8 of them fp64 instructions), the sums' way out 3; a workgroup per 1024 entries, so one round of the device.
template <int ELT, int STEPS, bool GATHER, int NT>
__global__ void __launch_bounds__(NT)
tree_split_kernel(TreeSrc src, const uint32_t *__restrict__ order, uint32_t *__restrict__ out, const code_t<ELT> *__restrict__ codes,
                  const uint32_t *__restrict__ hist, LevelSums sums, double *__restrict__ part_out, int64_t np, int64_t n_real, int64_t m,
                  int64_t n_nodes, int c_lo, int c_hi) {
    constexpr int NW = NT / 64, BITS = ELT * 8;
    __shared__ uint32_t s_hist[2048];
    __shared__ int s_lt[NW], s_eq[NW], s_plt[NW], s_peq[NW];   // entries below / equal to the median: the workgroup's own, those of the workgroups before it
    __shared__ uint32_t s_left[NT];
    __shared__ double s_part[NW][256];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = blockIdx.y;
    const int parts = (int)(m / NT);   // workgroups of a node
    const int node = (int)blockIdx.x / parts, mine = (int)blockIdx.x % parts;
    const int64_t node0 = (int64_t)node * m, at0 = (int64_t)bh * np + node0;
    auto pos_of = [&](int i) { return order ? order[at0 + i] : (uint32_t)(node0 + i); };
    uint32_t code[STEPS], entry = 0, own = 0;   // code[k]: entry k NT + t of the node
    if constexpr (GATHER) {
        uint32_t e[STEPS];
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
            if (k < parts) e[k] = pos_of(k * NT + t);   // uniform conditions throughout
        const int ax = node_axis<ELT, NT>(sums, src, order, bh, np, m, node, n_nodes, n_real, mine == 0, c_lo, c_hi);
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
            if (k < parts) {
                code[k] = e[k] < n_real ? coord_code<ELT>(src.row(bh, e[k]), ax) : PAD_CODE<ELT>;
                if (k == mine) entry = e[k];
            }
    } else {
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
            if (k < parts) code[k] = codes[at0 + k * NT + t];
        entry = pos_of(mine * NT + t);
    }
    int rank = (int)(m / 2);   // the entry looked for is the rank-th smallest (from 1) of those that share `known`
    uint32_t known = 0, known_mask = 0;
    int top = BITS;   // bits not known yet
    if constexpr (!GATHER) {
        static_assert(GATHER || NT == 1024, "four slices of 256 counts");
        const uint32_t *h = hist + ((int64_t)bh * (np / PIECE) + (int64_t)node * parts) * 256;
        uint32_t n = 0;
#pragma unroll 8
        for (int p = t >> 8; p < parts; p += 4) n += h[p * 256 + (t & 255)];
        s_hist[t] = 0;
        s_hist[t + 1024] = 0;
        __syncthreads();
        if (n) atomicAdd(&s_hist[t & 255], n);
        __syncthreads();
        top -= 8;
        known = pick_digit<NT>(s_hist, lane, wave, rank) << top;
        known_mask = 0xffu << top;
    }
    while (top > 0) {
        const int width = top > 11 ? 11 : top, shift = top - width;
        for (int i = t; i < 2048; i += NT) s_hist[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
            if (k < parts && (code[k] & known_mask) == known) atomicAdd(&s_hist[(code[k] >> shift) & ((1u << width) - 1u)], 1u);
        __syncthreads();
        known |= pick_digit<NT>(s_hist, lane, wave, rank) << shift;
        known_mask |= ((1u << width) - 1u) << shift;
        top = shift;
    }
    // `known` is the median code, `rank` (>= 1) the number of entries equal to it that go left
    int plt = 0, peq = 0;
#pragma unroll
    for (int k = 0; k < STEPS; ++k)
        if (k < parts) {
            if (k < mine) {
                plt += (int)__popcll(__ballot(code[k] < known));
                peq += (int)__popcll(__ballot(code[k] == known));
            } else if (k == mine) own = code[k];
        }
    const uint64_t lts = __ballot(own < known), eqs = __ballot(own == known);
    if (lane == 0) {
        s_plt[wave] = plt;
        s_peq[wave] = peq;
        s_lt[wave] = (int)__popcll(lts);
        s_eq[wave] = (int)__popcll(eqs);
    }
    __syncthreads();
    int lt0 = 0, eq0 = 0, lt_w = 0, eq_w = 0, lt_all = 0, eq_all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        lt0 += s_plt[w];
        eq0 += s_peq[w];
        lt_w += w < wave ? s_lt[w] : 0;
        eq_w += w < wave ? s_eq[w] : 0;
        lt_all += s_lt[w];
        eq_all += s_eq[w];
    }
    auto lefts_before = [&](int lt, int eq) { return lt + (eq < rank ? eq : rank); };
    const int left0 = lefts_before(lt0, eq0);                                  // entries of the node before this workgroup's that go left
    const int n_left = lefts_before(lt0 + lt_all, eq0 + eq_all) - left0;       // of this workgroup's
    const uint64_t below = (1ull << lane) - 1ull;
    const int eq_before = eq0 + eq_w + (int)__popcll(eqs & below);
    const int lt = lefts_before(lt0 + lt_w + (int)__popcll(lts & below), eq_before);   // entries before this one that go left
    const bool left = own < known || (own == known && eq_before < rank);
    out[at0 + (left ? lt : (int)(m / 2) + mine * NT + t - lt)] = entry;
    if (!part_out) return;   // uniform
    if (left) s_left[lt - left0] = entry;
    __syncthreads();
    const int share = ((n_left + NW - 1) / NW + 15) & ~15;   // rows of a wave, at most 64
    const int idx = wave * share + lane;
    const int mypos = (lane < share && idx < n_left) ? (int)s_left[idx] : 0x7fffffff;
    const uint64_t real = __ballot(mypos < n_real);
    double s0 = 0., s1 = 0., q0 = 0., q1 = 0.;
    if (real) sum_rows64<ELT>(src, bh, lane, mypos, real, tree_shift<ELT>(src, bh, lane, n_real), s0, s1, q0, q1);   // uniform
    store_partial<NW>(s_part, lane, wave, NW, s0, s1, q0, q1, part_out + ((int64_t)bh * sums.n_pieces + blockIdx.x) * 256);
}

// Splits a node of more than 32768 entries: one workgroup per node, wave w takes the entries [w m/16, (w+1) m/16), eight codes per
// thread in flight, the codes read again for every digit.
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_split_large_kernel(const uint32_t *__restrict__ order, uint32_t *__restrict__ out, const code_t<ELT> *__restrict__ codes, int64_t np,
                        int64_t m) {
    __shared__ uint32_t s_hist[2048];
    __shared__ int s_lt[16], s_eq[16];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = blockIdx.y;
    const int64_t node0 = (int64_t)blockIdx.x * m, at0 = (int64_t)bh * np + node0;
    const int steps = (int)(m / 1024), first = wave * steps * 64 + lane;   // this thread's entries: first + 64 k, k < steps
    auto pos_of = [&](int i) { return order ? order[at0 + i] : (uint32_t)(node0 + i); };
    // f(i, code, entry) for this thread's entries; the conditions are the same in every lane, so f may use ballots
    auto for_codes = [&](bool entries, auto f) {
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
    };
    int rank = (int)(m / 2);
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
        known |= pick_digit<1024>(s_hist, lane, wave, rank) << shift;
        known_mask |= ((1u << width) - 1u) << shift;
    }
    int n_lt = 0, n_eq = 0;
    for_codes(false, [&](int, uint32_t c, uint32_t) {
        n_lt += (int)__popcll(__ballot(c < known));
        n_eq += (int)__popcll(__ballot(c == known));
    });
    if (lane == 0) {
        s_lt[wave] = n_lt;
        s_eq[wave] = n_eq;
    }
    __syncthreads();
    int eq_before = 0, left_at = 0;
    for (int w = 0; w < wave; ++w) {
        left_at += s_lt[w];
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

// Rows into the arena in tree order, and with the key rows the two position maps (row0 is added to the
// positions: a chunk's positions are relative to its first row).  blockIdx.z = 0: keys, 1: values; z0 is added to it.
__global__ void tree_gather_kernel(TreeSrc ksrc, TreeSrc vsrc, const uint64_t *__restrict__ keys, char *Kdst,
                                   char *Vdst, int32_t *slot_pos, int32_t *pos_slot, int64_t np, int64_t n_real,
                                   int pos_bits, int64_t cap_rows, int64_t row0, int row_bytes, int z0) {
    const int chunks = row_bytes / 16;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_real * chunks) return;
    const int bh = blockIdx.y;
    const int64_t slot = i / chunks;
    const int ch = (int)(i % chunks);
    const int64_t pos = key_pos(keys[(int64_t)bh * np + slot], pos_bits);
    const bool keys_too = blockIdx.z + z0 == 0;
    const TreeSrc &s = keys_too ? ksrc : vsrc;
    char *dst = keys_too ? Kdst : Vdst;
    reinterpret_cast<uint4 *>(dst + ((int64_t)bh * cap_rows + row0 + slot) * row_bytes)[ch] =
        reinterpret_cast<const uint4 *>(s.row(bh, pos))[ch];
    if (keys_too && ch == 0) {
        slot_pos[(int64_t)bh * cap_rows + row0 + slot] = (int32_t)(row0 + pos);
        pos_slot[(int64_t)bh * cap_rows + row0 + pos] = (int32_t)(row0 + slot);
    }
}

// Lanes whose number has the bit J.
template <int J>
constexpr uint64_t LANES = J == 1 ? 0xaaaaaaaaaaaaaaaaull : J == 2 ? 0xccccccccccccccccull : J == 4 ? 0xf0f0f0f0f0f0f0f0ull
                         : J == 8 ? 0xff00ff00ff00ff00ull : J == 16 ? 0xffff0000ffff0000ull : 0xffffffff00000000ull;

// One compare-exchange of a bitonic sort with the lane J away; the lanes of `flip` stand in a descending run.  Data-parallel moves up
// to J = 8, row and half swaps beyond (these put the two values of a pair side by side), so no step makes a trip through LDS.
template <int J>
__device__ __forceinline__ uint32_t exchanged(uint32_t key, uint64_t flip) {
    auto dpp = [](uint32_t x, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xf, 0xf, true); };
    uint32_t a = key, b;
    if constexpr (J == 1) b = dpp(key, std::integral_constant<int, 0xB1>{});        // quad_perm [1,0,3,2]
    else if constexpr (J == 2) b = dpp(key, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
    else if constexpr (J == 4)                                                      // 7 - i within 8, then 3 - i within 4
        b = dpp(dpp(key, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{});
    else if constexpr (J == 8) b = dpp(key, std::integral_constant<int, 0x128>{});  // row_ror:8
    else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(key, key, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(key, key, false, false);
        a = r[0];
        b = r[1];
    }
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    return __builtin_amdgcn_inverse_ballot_w64(~LANES<J> ^ flip) ? lo : hi;
}
template <int J>
__device__ __forceinline__ uint64_t exchanged(uint64_t key, uint64_t flip) {
    auto word = [](uint32_t v, uint32_t &a, uint32_t &b) {   // the pair's two values, in either order but the same one for both words
        auto dpp = [](uint32_t x, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xf, 0xf, true); };
        a = v;
        if constexpr (J == 1) b = dpp(v, std::integral_constant<int, 0xB1>{});
        else if constexpr (J == 2) b = dpp(v, std::integral_constant<int, 0x4E>{});
        else if constexpr (J == 4) b = dpp(dpp(v, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{});
        else if constexpr (J == 8) b = dpp(v, std::integral_constant<int, 0x128>{});
        else if constexpr (J == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            a = r[0];
            b = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            a = r[0];
            b = r[1];
        }
    };
    uint32_t a0, a1, b0, b1;
    word((uint32_t)key, a0, b0);
    word((uint32_t)(key >> 32), a1, b1);
    const uint64_t a = ((uint64_t)a1 << 32) | a0, b = ((uint64_t)b1 << 32) | b0;
    const bool less = a < b;
    return (__builtin_amdgcn_inverse_ballot_w64(~LANES<J> ^ flip) == less) ? a : b;
}

// The merge of runs of K entries as far as it stays inside a wave.
template <int K, typename KEY>
__device__ __forceinline__ KEY merged(KEY key, uint64_t flip) {
    if constexpr (K >= 64) key = exchanged<32>(key, flip);
    if constexpr (K >= 32) key = exchanged<16>(key, flip);
    if constexpr (K >= 16) key = exchanged<8>(key, flip);
    if constexpr (K >= 8) key = exchanged<4>(key, flip);
    if constexpr (K >= 4) key = exchanged<2>(key, flip);
    return exchanged<1>(key, flip);
}

// The merges of up to 32 entries of a sort of every aligned run of m (a merge of m entries ends in ascending order, the ones
// before it alternate).  The upper half of a wave may repeat the lower.
template <typename KEY>
__device__ __forceinline__ KEY sort_in_wave(KEY key, int m) {
    key = merged<2>(key, m == 2 ? 0ull : LANES<2>);
    if (m > 2) key = merged<4>(key, m == 4 ? 0ull : LANES<4>);   // uniform
    if (m > 4) key = merged<8>(key, m == 8 ? 0ull : LANES<8>);
    if (m > 8) key = merged<16>(key, m == 16 ? 0ull : LANES<16>);
    if (m > 16) key = merged<32>(key, m == 32 ? 0ull : LANES<32>);
    return key;
}

// Where a finished node's rows go in the same launch (K == NULL: only the order is wanted).
struct TreeRows {
    char *K;
    int32_t *slot_pos, *pos_slot;
    int64_t cap_rows, row0;
};

// All the remaining levels of a node of np <= SMALL_NODE padded entries in one launch, a workgroup per node.  Either the whole
// tree of a small input (a buffer chunk of B keys: order == NULL, one workgroup per (sequence, KV head)), or every node of
// the level at which the kernels above have brought the nodes down to that size (the node's entries are np consecutive ones of
// `order`, in ascending position order).
// The node's rows are fetched once, 128 KB that stay in LDS: all levels read them there, and the finished node's key rows go to the
// arena from there.  A wave per 32 entries.  Per level a wave adds up 16 rows: nodes of 32 entries and more share the rows of the left
// child out among the waves of the parent, the sums meet in LDS, and the right child's sums are the parent's less the left child's (a wave holds
// its own node's in registers); below that a node belongs to one wave and no barrier is left.  Nodes of 64 and more are sorted by
// [ code | index of the entry in the node's initial order ], an entry per thread, exchanged through LDS only between waves.
// Bound by instructions: 8 per row and two channels (conversion, add, multiply-add in fp64), then the searches for the largest
// variance and the exchanges.  A round of one workgroup per compute unit takes 36 us (8 x 32768 keys are two): 7.4 to fetch the rows, 3.2 for the first
// sums, 3.3 to 4.3 per level of 512 to 64 entries, 8 for the levels of one wave, 2 for the rows' way out; 77 us in all.  (Nodes of 1024 entries
// whose rows were fetched from memory at every level: 160 us, and 19 more to gather the key rows.)
template <int ELT>
__global__ void __launch_bounds__(1024)
tree_small_kernel(TreeSrc src, const uint32_t *__restrict__ order, uint64_t *__restrict__ keys_out, int64_t np_total,
                  int np, int64_t n_real, int levels, int c_lo, int c_hi, TreeRows dst) {
    typedef typename std::conditional<ELT == 2, uint32_t, uint64_t>::type key_t;
    constexpr int NODE = SMALL_NODE<ELT>, ROW = LVR_D * ELT, PIECES = ROW / 16;
    constexpr int ENT_BITS = ELT == 2 ? 9 : 8;
    static_assert((1 << ENT_BITS) == NODE, "an entry's index fills its bits of a key");
    __shared__ __align__(16) char s_rows[NODE * ROW];
    __shared__ double2 s_part[NODE / 64][2][64];   // sums of a pair of waves: lane's two channels, their squares
    __shared__ key_t s_key[2][NODE];
    __shared__ int32_t s_pos[NODE];      // position of an entry
    __shared__ uint16_t s_ent[NODE];     // the current order: entry in every place
    __shared__ int32_t s_axis[NODE / 64];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), waves = (int)(blockDim.x >> 6);
    const int bh = blockIdx.y;
    const int64_t node0 = (int64_t)blockIdx.x * np, base = (int64_t)bh * np_total + node0;
    const int nr = n_real - node0 < np ? (int)(n_real - node0) : np;   // real entries: a prefix of the node's
    if (nr <= 0) return;   // uniform: all padding, which nothing reads
    auto pos_of = [&](int e) { return order ? (int)order[base + e] : (int)(node0 + e); };
    const char *rows = src.row(bh, 0);
    const int64_t row_bytes = src.st * ELT;
    const int held = np < 32 ? 32 : np;   // rows a wave may look at: those past nr add nothing to any sum
    {
        const int c = t % PIECES, step = (int)blockDim.x / PIECES;
        for (int e0 = t / PIECES; e0 < held; e0 += 8 * step) {
            uint4 w[8];
            int p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int e = e0 + u * step;
                p[u] = pos_of(e < nr ? e : 0);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = reinterpret_cast<const uint4 *>(rows + (int64_t)p[u] * row_bytes)[c];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int e = e0 + u * step;
                // padding: zeros for bf16, the first row (the shift of the sums) for fp32
                if (e < held) reinterpret_cast<uint4 *>(s_rows + e * ROW)[c] = (e < nr || ELT == 4) ? w[u] : make_uint4(0, 0, 0, 0);
            }
        }
    }
    if (t < held) {
        s_ent[t] = (uint16_t)t;
        s_pos[t] = t < np ? pos_of(t) : 0;
    }
    __syncthreads();
    Shift shift = {0.0, 0.0};
    if constexpr (ELT == 4) {
        float x0, x1;
        lane_pair<ELT>(s_rows, lane, x0, x1);
        shift.p0 = (double)x0;
        shift.p1 = (double)x1;
    }
    double s0, s1, q0, q1;   // sums of this wave's node
    int mag;                 // and what their rounding errors are measured by
    // sums of N rows: the entries that lanes `first` .. `first` + N - 1 hold in `ent`
    auto sum = [&](auto n_c, int ent, int first, double &a0, double &a1, double &b0, double &b1) {
        constexpr int N = decltype(n_c)::value;
        float x0[N], x1[N];
#pragma unroll
        for (int u = 0; u < N; ++u) lane_pair<ELT>(s_rows + __builtin_amdgcn_readlane(ent, first + u) * ROW, lane, x0[u], x1[u]);
        a0 = a1 = b0 = b1 = 0.;
        add_rows<ELT>(x0, x1, shift, a0, a1, b0, b1);
    };
    typedef std::integral_constant<int, 16> N16;
    typedef std::integral_constant<int, 8> N8;
    typedef std::integral_constant<int, 4> N4;
    typedef std::integral_constant<int, 2> N2;
    // the sums of `group` consecutive waves (a power of two, at least 2), the same in each of them
    auto add_waves = [&](int group, double &a0, double &a1, double &b0, double &b1) {
        double2(&pair)[2][64] = s_part[wave >> 1];
        if (wave & 1) {
            pair[0][lane] = make_double2(a0, a1);
            pair[1][lane] = make_double2(b0, b1);
        }
        __syncthreads();
        if (!(wave & 1)) {
            const double2 a = pair[0][lane], b = pair[1][lane];
            pair[0][lane] = make_double2(a0 + a.x, a1 + a.y);
            pair[1][lane] = make_double2(b0 + b.x, b1 + b.y);
        }
        __syncthreads();
        const int first = (wave & ~(group - 1)) >> 1;
        a0 = a1 = b0 = b1 = 0.;
        for (int i = 0; i < group >> 1; ++i) {
            const double2 a = s_part[first + i][0][lane], b = s_part[first + i][1][lane];
            a0 += a.x; a1 += a.y; b0 += b.x; b1 += b.y;
        }
    };
    int ent = s_ent[wave * 32 + (lane & 31)];
    auto real_of = [&](int first, int m) { return nr <= first ? 0. : (nr - first < m ? (double)(nr - first) : (double)m); };
    // Axis of the node at entries [first, first + 2^log_m) of the order, from its sums; `difference`: they are one.  Where they do not
    // tell, they are taken again from the node's real rows, relative to its first: add(shift, ...) adds those up.
    auto axis_of = [&](double &a0, double &a1, double &b0, double &b1, int first, int log_m, bool difference, int first_ent, auto add) {
        const double n = real_of(first, 1 << log_m);
        int top;
        int ax = wave_argmax(spread(a0, b0, n), spread(a1, b1, n), lane, c_lo, c_hi, top);
        if (n > 1. && (ELT == 4 || difference) && unsure(top, mag, log_m)) {   // uniform over the wave
            const Shift p = shift_of<ELT>(s_rows + first_ent * ROW, lane);
            a0 = a1 = b0 = b1 = 0.;
            add(p, (int)n);
            ax = wave_argmax(spread(a0, b0, n), spread(a1, b1, n), lane, c_lo, c_hi, top);
            if constexpr (ELT == 4) {
                shift_sums(a0, b0, n, p.p0, shift.p0);
                shift_sums(a1, b1, n, p.p1, shift.p1);
            }
            if (log_m >= 5) mag = largest_square(b0, b1, lane, c_lo, c_hi);   // (the wave's only node)
        }
        return ax;
    };
    // n rows: the entries that lanes `at` .. hold in `e`
    auto add_some = [&](int e, int at, int n, const Shift &p, double &a0, double &a1, double &b0, double &b1) {
        for (int j0 = 0; j0 < n; j0 += 4) {
            float x0[4], x1[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                lane_pair<ELT>(s_rows + __builtin_amdgcn_readlane(e, at + (j0 + u < n ? j0 + u : 0)) * ROW, lane, x0[u], x1[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float y0[1] = {x0[u]}, y1[1] = {x1[u]};
                if (j0 + u < n) add_rows<ELT>(y0, y1, p, a0, a1, b0, b1);   // uniform
            }
        }
    };
    // the axis of a node of 32 entries or less that lanes `at` .. of `ent` hold
    auto axis_in_wave = [&](double &a0, double &a1, double &b0, double &b1, int at, int log_m, bool difference) {
        return axis_of(a0, a1, b0, b1, wave * 32 + at, log_m, difference, __builtin_amdgcn_readlane(ent, at),
                       [&](const Shift &p, int n) { add_some(ent, at, n, p, a0, a1, b0, b1); });
    };
    auto code_of = [&](int e, int axis) { return e < nr ? coord_code<ELT>(s_rows + e * ROW, axis) : PAD_CODE<ELT>; };
    const int groups_of = np >> levels;   // entries of a finished node
    int m = np;
    {
        double a0, a1, b0, b1;
        sum(N16{}, ent, 0, s0, s1, q0, q1);
        sum(N16{}, ent, 16, a0, a1, b0, b1);
        s0 += a0; s1 += a1; q0 += b0; q1 += b1;
    }
    if (waves > 1) add_waves(waves, s0, s1, q0, q1);
    mag = largest_square(q0, q1, lane, c_lo, c_hi);
    for (; m >= 64 && m > groups_of; m >>= 1) {   // uniform
        if (m < np) {   // the sums of this wave's node out of its parent's
            const int group = m / 16, parent = wave & ~(group - 1);   // the parent's waves
            const int e = s_ent[parent * 32 + (wave - parent) * 16 + (lane & 15)];
            double a0, a1, b0, b1;
            sum(N16{}, e, 0, a0, a1, b0, b1);
            add_waves(group, a0, a1, b0, b1);
            const bool right = (wave & (group >> 1)) != 0;
            s0 = right ? s0 - a0 : a0; s1 = right ? s1 - a1 : a1;
            q0 = right ? q0 - b0 : b0; q1 = right ? q1 - b1 : b1;
        }
        const int place = wave * 32 & ~(m - 1);
        const bool difference = m < np && (place & m) != 0;
        const int ax = axis_of(s0, s1, q0, q1, place, __builtin_ctz(m), difference, s_ent[place], [&](const Shift &p, int n) {
            for (int j = 0; j < n; j += 32) add_some(s_ent[place + j + (lane & 31)], 0, n - j < 32 ? n - j : 32, p, s0, s1, q0, q1);
        });
        if (lane == 0 && (wave & (m / 32 - 1)) == 0) s_axis[wave / (m / 32)] = ax;
        __syncthreads();
        const bool sorts = wave * 64 < np;   // an entry per thread: the waves that hold one
        key_t key = ~(key_t)0;
        if (sorts) {
            const int e = s_ent[t];
            key = ((key_t)code_of(e, s_axis[t / m]) << ENT_BITS) | (key_t)e;
        }
        int buf = 0;
        if (sorts) key = sort_in_wave(key, m);
        for (int k = 64; k <= m; k <<= 1) {
            const bool up = k == m || (wave * 64 & k) == 0;   // the same in the whole wave
            for (int j = k >> 1; j >= 64; j >>= 1) {
                if (sorts) s_key[buf][t] = key;
                __syncthreads();
                if (sorts) {
                    const key_t other = s_key[buf][t ^ j];
                    key = ((wave * 64 & j) == 0) == up ? (key < other ? key : other) : (key < other ? other : key);
                }
                buf ^= 1;
            }
            if (sorts) key = merged<64>(key, up ? 0ull : ~0ull);
        }
        if (sorts) s_ent[t] = (uint16_t)(key & (key_t)(NODE - 1));
        __syncthreads();
    }
    if (m > groups_of) {   // uniform: nodes of 32 entries and less, each of one wave
        const int i = lane & 31, place = wave * 32;
        if (np > 32) {   // this wave's node of 32 out of the node of 64 it shares with its neighbour
            const int e = s_ent[(wave & ~1) * 32 + (wave & 1) * 16 + (lane & 15)];
            double a0, a1, b0, b1;
            sum(N16{}, e, 0, a0, a1, b0, b1);
            add_waves(2, a0, a1, b0, b1);
            const bool right = (wave & 1) != 0;
            s0 = right ? s0 - a0 : a0; s1 = right ? s1 - a1 : a1;
            q0 = right ? q0 - b0 : b0; q1 = right ? q1 - b1 : b1;
            ent = s_ent[place + i];
        }
        auto split = [&](int axis, int size) {
            const key_t key = ((key_t)code_of(ent, axis) << ENT_BITS) | (key_t)ent;
            ent = (int)(sort_in_wave(key, size) & (key_t)(NODE - 1));
        };
        if (m == 32) {
            split(axis_in_wave(s0, s1, q0, q1, 0, 5, np > 32 && (wave & 1)), 32);
            m = 16;
        }
        double a[2][4];   // the nodes of 16 (where the whole tree is smaller than 32 entries the second is empty)
        if (m > groups_of) {
            sum(N16{}, ent, 0, a[0][0], a[0][1], a[0][2], a[0][3]);
            a[1][0] = s0 - a[0][0]; a[1][1] = s1 - a[0][1]; a[1][2] = q0 - a[0][2]; a[1][3] = q1 - a[0][3];
            if (m == 16) {
                const int x0 = axis_in_wave(a[0][0], a[0][1], a[0][2], a[0][3], 0, 4, false);
                const int x1 = axis_in_wave(a[1][0], a[1][1], a[1][2], a[1][3], 16, 4, true);
                split((i & 16) ? x1 : x0, 16);
                m = 8;
            }
        }
        if (m > groups_of) {
            int axis = 0;
            if (m == 8) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    double b[4];
                    sum(N8{}, ent, 16 * h, b[0], b[1], b[2], b[3]);
                    double d[4] = {a[h][0] - b[0], a[h][1] - b[1], a[h][2] - b[2], a[h][3] - b[3]};
                    const int x0 = axis_in_wave(b[0], b[1], b[2], b[3], 16 * h, 3, false);
                    const int x1 = axis_in_wave(d[0], d[1], d[2], d[3], 16 * h + 8, 3, true);
                    if ((i >> 4) == h) axis = (i & 8) ? x1 : x0;
                }
                split(axis, 8);
                m = 4;
            }
        }
        if (m == 4 && m > groups_of) {
            int axis = 0;
            for (int h = 0; h < 8; ++h) {
                double b[4];
                sum(N4{}, ent, 4 * h, b[0], b[1], b[2], b[3]);
                const int x = axis_in_wave(b[0], b[1], b[2], b[3], 4 * h, 2, false);
                if ((i >> 2) == h) axis = x;
            }
            split(axis, 4);
            m = 2;
        }
        if (m == 2 && m > groups_of) {
            int axis = 0;
            for (int h = 0; h < 16; ++h) {
                double b[4];
                sum(N2{}, ent, 2 * h, b[0], b[1], b[2], b[3]);
                const int x = axis_in_wave(b[0], b[1], b[2], b[3], 2 * h, 1, false);
                if ((i >> 1) == h) axis = x;
            }
            split(axis, 2);
        }
        if (lane < 32) s_ent[place + i] = (uint16_t)ent;
        __syncthreads();
    }
    if (t < np) keys_out[base + t] = (uint64_t)(uint32_t)s_pos[s_ent[t]];
    if (!dst.K) return;   // uniform
    const int64_t slot0 = (int64_t)bh * dst.cap_rows + dst.row0 + node0;
    for (int x = t; x < nr * PIECES; x += (int)blockDim.x) {
        const int j = x / PIECES, c = x % PIECES;
        reinterpret_cast<uint4 *>(dst.K + (slot0 + j) * ROW)[c] = reinterpret_cast<const uint4 *>(s_rows + s_ent[j] * ROW)[c];
    }
    if (t < nr) {
        const int pos = s_pos[s_ent[t]];
        dst.slot_pos[slot0 + t] = (int32_t)(dst.row0 + pos);
        dst.pos_slot[(int64_t)bh * dst.cap_rows + dst.row0 + pos] = (int32_t)(dst.row0 + node0 + t);
    }
}

int bits_for(int64_t v) {   // bits needed to hold values 0 .. v-1
    int b = 0;
    while (((int64_t)1 << b) < v) ++b;
    return b;
}

// The two work arrays: a = the order before and after a split (32-bit positions, two halves), b = the codes of a level and, behind
// room for 32-bit codes, the counts of their upper eight bits, at the end the finished order as 64-bit keys.
template <int ELT>
hipError_t tree_order_t(lvr_index *ix, const TreeSrc &src, int64_t n_real, int64_t np, int levels, int c_lo, int c_hi,
                        hipStream_t st, const TreeRows &dst) {
    const int n_bh = lvr_n_bh(ix);
    uint32_t *cur = nullptr;   // the order at the start: entry i holds position i
    uint32_t *half[2] = {reinterpret_cast<uint32_t *>(ix->tree_keys_a),
                         reinterpret_cast<uint32_t *>(ix->tree_keys_a) + ix->tree_cap_keys};
    code_t<ELT> *codes = reinterpret_cast<code_t<ELT> *>(ix->tree_keys_b);
    uint32_t *hist = reinterpret_cast<uint32_t *>(ix->tree_keys_b) + ix->tree_cap_keys;
    // sums of pieces and of nodes, of two levels each
    const int64_t n_pieces = np > PIECE ? np / PIECE : 1;
    double *pieces[2], *node_sums[2];
    // What the rounding errors of a node's sums are measured by, of two levels, in the upper half of the room for a group's axis each: what has an
    // axis there, nodes of more than 32768 entries, stays in the lower half, and two words per piece are at most a 32nd of the groups wherever
    // there is a node to split here.  (Behind the sums, which fill 2 MB for 8 x 32768 keys, they made that allocation 2 KB larger, and a program
    // that sets up one such index after the other took 1.3 ms for each instead of 1.0.)
    int *node_mag[2];
    for (int i = 0; i < 2; ++i) {
        node_mag[i] = ix->tree_axis + n_bh * ((int64_t)1 << levels) / 2 + i * n_bh * n_pieces;
        pieces[i] = ix->tree_partial + (int64_t)i * n_bh * n_pieces * 256;
        node_sums[i] = ix->tree_partial + (int64_t)(2 + i) * n_bh * n_pieces * 256;
    }
    int whole = 1;   // the next level's pieces are added up by a launch of their own
    int L = 0;
    for (; (np >> L) > SMALL_NODE<ELT>; ++L) {   // np is a power of two
        const int64_t n_nodes = (int64_t)1 << L, m = np >> L;
        const bool last = m / 2 <= SMALL_NODE<ELT>;   // small nodes take their own sums
        // (fp32: the last level's nodes of 512 entries are twice as many as there are pieces)
        LevelSums sums{pieces[L & 1], node_sums[(L & 1) ^ 1], last ? nullptr : node_sums[L & 1], node_mag[(L & 1) ^ 1], node_mag[L & 1], n_pieces, whole};
        if (whole)
            hipLaunchKernelGGL(tree_stats_piece_kernel<ELT>, dim3((unsigned)n_pieces, (unsigned)n_bh),
                               dim3(np < PIECE ? (unsigned)np : (unsigned)PIECE), 0, st, src, cur, pieces[L & 1], np, n_real);
        uint32_t *next = half[L & 1];
        double *part_out = last ? nullptr : pieces[(L & 1) ^ 1];
        const dim3 per_piece((unsigned)n_pieces, (unsigned)n_bh), per_node((unsigned)n_nodes, (unsigned)n_bh);
#define LVR_SPLIT_LAUNCH(STEPS, GATHER, NT)                                                                                        \
    hipLaunchKernelGGL((tree_split_kernel<ELT, STEPS, GATHER, NT>), dim3((unsigned)(np / NT), (unsigned)n_bh), dim3(NT), 0, st, src, \
                       cur, next, codes, hist, sums, part_out, np, n_real, m, n_nodes, c_lo, c_hi)
        if (m > 32768) {   // more codes than the threads of a workgroup hold
            hipLaunchKernelGGL(tree_axis_kernel<ELT>, per_node, dim3(1024), 0, st, src, cur, sums, ix->tree_axis, np, m, n_nodes, n_real, c_lo, c_hi);
            hipLaunchKernelGGL(tree_codes_kernel<ELT>, per_piece, dim3(1024), 0, st, src, cur, codes, hist, ix->tree_axis, sums, np, n_real,
                               m, n_nodes, c_lo, c_hi);
            hipLaunchKernelGGL(tree_split_large_kernel<ELT>, per_node, dim3(1024), 0, st, cur, next, codes, np, m);
            whole = 1;
        } else {
            if (m > GATHER_MAX) {
                hipLaunchKernelGGL(tree_codes_kernel<ELT>, per_piece, dim3(1024), 0, st, src, cur, codes, hist, (const int32_t *)nullptr, sums,
                                   np, n_real, m, n_nodes, c_lo, c_hi);
                LVR_SPLIT_LAUNCH(32, false, 1024);
            } else if (m >= 1024) LVR_SPLIT_LAUNCH(GATHER_MAX / 1024, true, 1024);
            else LVR_SPLIT_LAUNCH(1, true, 512);   // fp32: nodes of 512
            whole = 0;
        }
#undef LVR_SPLIT_LAUNCH
        cur = next;
    }
    const int64_t m0 = np >> L;   // entries of a node that one workgroup finishes
    const unsigned threads = m0 <= 32 ? 64u : (unsigned)(2 * m0);
    hipLaunchKernelGGL(tree_small_kernel<ELT>, dim3((unsigned)(np / m0), (unsigned)n_bh), dim3(threads), 0, st, src, cur,
                       ix->tree_keys_b, np, (int)m0, n_real, levels - L, c_lo, c_hi, dst);
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

namespace {

hipError_t tree_order(lvr_index *ix, const void *Ksrc, const int64_t ks[3], int64_t n_real, hipStream_t st, lvr_tree_perm *perm, int c_lo,
                      int c_hi, const TreeRows &dst) {
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
    const hipError_t e = ix->elt == 2 ? tree_order_t<2>(ix, src, n_real, np, levels, c_lo, c_hi, st, dst)
                                      : tree_order_t<4>(ix, src, n_real, np, levels, c_lo, c_hi, st, dst);
    if (e != hipSuccess) return e;
    perm->keys = ix->tree_keys_b;
    perm->np = np;
    perm->pos_bits = bits_for(np);
    return hipSuccess;
}

// Rows `from` keys (z0 = 0) or values (z0 = 1) on into the arena, in the order of perm.
hipError_t gather_rows(lvr_index *ix, const void *Ksrc, const int64_t ks[3], const void *Vsrc, const int64_t vs[3], const lvr_tree_perm *perm,
                       int64_t n_real, int64_t row0, hipStream_t st, int z0) {
    if (n_real <= 0 || !perm->keys) return hipSuccess;
    const int n_bh = lvr_n_bh(ix);
    TreeSrc ksrc{static_cast<const char *>(Ksrc), ks[0], ks[1], ks[2], (int)ix->elt, ix->cfg.n_kv_heads};
    TreeSrc vsrc{static_cast<const char *>(Vsrc), vs[0], vs[1], vs[2], (int)ix->elt, ix->cfg.n_kv_heads};
    const int row_bytes = (int)(LVR_D * ix->elt);
    const int64_t total = n_real * (row_bytes / 16);
    hipLaunchKernelGGL(tree_gather_kernel, dim3((unsigned)((total + 255) / 256), (unsigned)n_bh, 2u - z0), dim3(256), 0, st,
                       ksrc, vsrc, perm->keys, static_cast<char *>(ix->K), static_cast<char *>(ix->V), ix->slot_pos,
                       ix->pos_slot, perm->np, n_real, perm->pos_bits, ix->cap_rows, row0, row_bytes, z0);
    return hipGetLastError();
}

}  // namespace

// Orders n_real = groups*r keys (positions 0..n_real-1 of the given source rows) by the tree; perm->keys then holds, per
// (sequence, KV head), the position stored in every slot.  Returns hipErrorInvalidValue if lvr_tree_feasible says no.
hipError_t lvr_tree_order(lvr_index *ix, const void *Ksrc, const int64_t ks[3], int64_t n_real, hipStream_t st,
                          lvr_tree_perm *perm, int c_lo, int c_hi) {
    return tree_order(ix, Ksrc, ks, n_real, st, perm, c_lo, c_hi, TreeRows{nullptr, nullptr, nullptr, 0, 0});
}

hipError_t lvr_tree_gather(lvr_index *ix, const void *Ksrc, const int64_t ks[3], const void *Vsrc, const int64_t vs[3],
                           const lvr_tree_perm *perm, int64_t n_real, int64_t row0, hipStream_t st) {
    return gather_rows(ix, Ksrc, ks, Vsrc, vs, perm, n_real, row0, st, 0);
}

// Order and rows at once: the launch that finishes the order writes the key rows and the position maps.
hipError_t lvr_tree_group(lvr_index *ix, const void *Ksrc, const int64_t ks[3], const void *Vsrc, const int64_t vs[3],
                          int64_t n_real, int64_t row0, hipStream_t st) {
    lvr_tree_perm perm;
    hipError_t e = tree_order(ix, Ksrc, ks, n_real, st, &perm, 0, LVR_D,
                              TreeRows{static_cast<char *>(ix->K), ix->slot_pos, ix->pos_slot, ix->cap_rows, row0});
    if (e != hipSuccess) return e;
    return gather_rows(ix, Ksrc, ks, Vsrc, vs, &perm, n_real, row0, st, 1);
}
