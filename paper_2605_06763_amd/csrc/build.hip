// Index construction kernels: copy K/V rows into the arena and compute, for every group of r
// consecutive arena rows, the ball of Sec. 4.1 "Ball enclosing" / Eq. (1) in each of the S
// coordinate blocks: centre = mean of the members, radius = largest member distance.
//
// Zero false negatives under rounding: the centre is stored in the cache's own format
// (bf16 or fp32), the radius is measured against the centre AS STORED, in fp32, and then
// widened to  rho * (1 + 2^-12) + 2^-12 * |centre_s|  (+1 ulp).  The widening exceeds every
// fp32 rounding error of the bound <q,c> + sum_s rho_s |pi_s q| evaluated at query time
// (at most ~(d+S) 2^-24 of the sum of term magnitudes), so a computed bound never falls
// below the exact score of a member.
#include <type_traits>

#include "lvr_internal.h"

namespace {

typedef uint32_t lvr_u32x4 __attribute__((ext_vector_type(4)));

// One side of a copy of rows into the arena: arbitrary source strides (in elements) for (batch, head, token).
struct CopySide {
    const char *src;
    char *dst;
    int64_t sb, sh, st;
    int64_t first;   // rows below this one are left alone (someone else writes them)
};

// Where a build kernel takes the member rows from: the arena (base == NULL), or the caller's K with
// its element strides, in which case the kernel also writes the rows into the arena (the copy of K
// and the pass over the groups are then one read of K instead of two).
struct BuildSrc {
    const char *base;
    int64_t sb, sh, st;
    int n_kv_heads;
};

// Rows that nothing reads again soon are streamed past the caches, but only where they would push out more than they are
// worth: a copy that fits the caches is faster through them.  `rows` rows of n_bh (sequence, KV head) pairs, each read and
// written once; with bf16 centres, groups of four: 37 MB of values 17.3 us against 18.9 streamed (build of 8 x 9001 keys), 67 MB
// 54.4 against 48.7 (8 x 32768), 268 MB 208 against 199.  An append's rows are read again by the next launch.
constexpr int64_t STREAM_BYTES = 48 << 20;
inline bool streamed(int64_t rows, int n_bh, size_t row_bytes) { return rows * n_bh * (int64_t)row_bytes >= STREAM_BYTES; }

// Block `block` (256 threads) of the copy of rows [c.first, rows), 2^SH 16-byte pieces each, to arena row dst_row0 on.  All of
// a thread's pieces are in flight before the first is stored.
template <int SH, int PIECES, bool STREAM>
__device__ __forceinline__ void copy_block(const CopySide &c, int bh, int n_kv_heads, int64_t cap_rows, int64_t dst_row0, int64_t rows,
                                           int64_t block) {
    constexpr int ELT = SH == 4 ? 2 : 4;
    const char *src = c.src + ((int64_t)(bh / n_kv_heads) * c.sb + (int64_t)(bh % n_kv_heads) * c.sh) * ELT;
    char *dst = c.dst + (((int64_t)bh * cap_rows + dst_row0) << (SH + 4));
    const int64_t first = (c.first << SH) + block * (256 * PIECES) + threadIdx.x, end = rows << SH;
    lvr_u32x4 w[PIECES];
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        const int64_t i = first + 256 * u;
        if (i < end) {
            const lvr_u32x4 *from = reinterpret_cast<const lvr_u32x4 *>(src + (i >> SH) * c.st * ELT) + (i & ((1 << SH) - 1));
            if constexpr (STREAM) w[u] = __builtin_nontemporal_load(from);
            else w[u] = *from;
        }
    }
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        const int64_t i = first + 256 * u;
        if (i < end) {
            lvr_u32x4 *to = reinterpret_cast<lvr_u32x4 *>(dst) + i;
            if constexpr (STREAM) __builtin_nontemporal_store(w[u], to);
            else *to = w[u];
        }
    }
}

// One piece per thread where the copy is a launch of its own (four: 17.6 against 17.3 us at 8 x 9001 keys, 208 against 201 at
// 8 x 131072); four, streamed, where it rides behind another step's few workgroups, as the 6-bit build streams the key rows
// (build and one step at 8 x 131072 keys: 262 us streamed, 277 with ordinary accesses; the four pieces 237).
constexpr int COPY_PIECES = 1, STEP_PIECES = 4;
inline unsigned copy_blocks(int64_t rows, int sh, int pieces) {
    return (unsigned)(((rows << sh) + 256 * pieces - 1) / (256 * pieces));
}

// Values in the first v_blocks blocks, keys in the rest, so an append is one launch.
template <int SH, bool STREAM>
__global__ void __launch_bounds__(256)
copy_rows_kernel(CopySide k, CopySide v, int n_kv_heads, int64_t cap_rows, int64_t dst_row0, int64_t rows, unsigned v_blocks) {
    if (blockIdx.x < v_blocks) copy_block<SH, COPY_PIECES, STREAM>(v, blockIdx.y, n_kv_heads, cap_rows, dst_row0, rows, blockIdx.x);
    else copy_block<SH, COPY_PIECES, STREAM>(k, blockIdx.y, n_kv_heads, cap_rows, dst_row0, rows, blockIdx.x - v_blocks);
}

__device__ __forceinline__ float seg_sum(float v, int lanes_per_sub) {
    for (int off = 1; off < lanes_per_sub; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// fp32 -> OCP e4m3 code (1 sign, 4 exponent bits of bias 7, 3 mantissa bits; subnormals below 2^-6),
// round to nearest even, magnitudes above the largest finite value (448) saturate to it.
__device__ __forceinline__ uint32_t f32_to_e4m3(float x) {
    const uint32_t sign = (__float_as_uint(x) >> 24) & 0x80u;
    float a = fabsf(x);
    if (!(a < 448.f)) a = 448.f;
    if (a < 0x1p-6f) return sign | (uint32_t)(int)rintf(a * 512.f);   // 0..8; 8 is the smallest normal
    uint32_t u = __float_as_uint(a);
    u += 0x7ffffu + ((u >> 20) & 1u);
    uint32_t code = (((u >> 23) - 120u) << 3) | ((u >> 20) & 7u);
    if (code > 0x7eu) code = 0x7eu;
    return sign | code;
}

typedef __attribute__((__vector_size__(2 * sizeof(float)))) float lvr_f32x2;

// Value of one e4m3 code (never the NaN code: the encoder above does not produce it).
__device__ __forceinline__ float e4m3_value(uint32_t code) {
    const lvr_f32x2 d = __builtin_amdgcn_cvt_pk_f32_fp8((int)(code & 0xffu), false);
    return d[0];
}

// fp32 -> e4m3 code rounded towards +inf (up = true) or -inf (up = false): the nearest code, moved one
// step in the wanted direction when it fell on the wrong side.  Codes are sign-magnitude, so a step
// up is magnitude + 1 for positive and magnitude - 1 for negative values, with -0 -> smallest positive.
// At the ends (+-448) the code stays; the caller accounts for what it cannot enclose.
__device__ __forceinline__ uint32_t f32_to_e4m3_directed(float x, bool up) {
    uint32_t c = f32_to_e4m3(x);
    const float d = e4m3_value(c);
    const uint32_t mag = c & 0x7fu;
    const bool neg = (c & 0x80u) != 0;
    if (up && d < x) {
        if (neg) c = mag == 0 ? 0x01u : (0x80u | (mag - 1u));
        else if (mag < 0x7eu) c = mag + 1u;
    } else if (!up && d > x) {
        if (!neg) c = mag == 0 ? 0x81u : (mag - 1u);
        else if (mag < 0x7eu) c = 0x80u | (mag + 1u);
    }
    return c;
}

typedef __attribute__((__vector_size__(6 * sizeof(uint32_t)))) uint32_t lvr_u32x6;
typedef __attribute__((__vector_size__(32 * sizeof(float)))) float lvr_f32x32;

// CF = 1: the centre is stored as 128 e4m3 codes in the order the matrix-core operand wants them
// (byte kq*32 + kk*8 + j holds coordinate kk*32 + kq*8 + j); only for bf16 caches.
// (6-bit codes have a kernel of their own below.)
template <typename KT, int CF = 0>
__global__ void __launch_bounds__(256)
build_groups_kernel(void *__restrict__ K, void *__restrict__ centres, float *__restrict__ radii,
                    int64_t cap_rows, int64_t max_groups, int64_t g0, int64_t g1, int r, int S, const BuildSrc src) {
    const int bh = blockIdx.y;
    const int li = threadIdx.x & 15;
    int64_t g = g0 + (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const bool valid = g < g1;
    if (!valid) g = g0;   // keep every lane busy so the shuffles below see defined data
    char *Kb = static_cast<char *>(K) + (int64_t)bh * cap_rows * LVR_D * sizeof(KT);
    const bool from_src = src.base != nullptr;   // uniform
    const char *Sb = from_src ? src.base + ((int64_t)(bh / src.n_kv_heads) * src.sb + (int64_t)(bh % src.n_kv_heads) * src.sh) * (int64_t)sizeof(KT)
                              : Kb;
    const int64_t row_stride = from_src ? src.st * (int64_t)sizeof(KT) : (int64_t)LVR_D * (int64_t)sizeof(KT);

    float c[8];
    lvr_zero8(c);
    // groups of up to four rows stay in registers between the two passes over the members
    lvr_raw8<KT> keep[4];
    const bool kept = r <= 4;   // uniform
    if (kept) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (m < r) lvr_load_raw(Sb + (g * r + m) * row_stride, 0, li, keep[m]);
#pragma unroll
        for (int m = 0; m < 4; ++m) {       // members in ascending row order
            if (m < r) {
                float x[8];
                if (from_src && valid) lvr_store_raw(Kb, g * r + m, li, keep[m]);   // the arena's copy of the row
                lvr_unpack(keep[m], x);
#pragma unroll
                for (int e = 0; e < 8; ++e) c[e] += x[e];
            }
        }
    } else {
        for (int m = 0; m < r; ++m) {
            float x[8];
            lvr_raw8<KT> raw;
            lvr_load_raw(Sb + (g * r + m) * row_stride, 0, li, raw);
            if (from_src && valid) lvr_store_raw(Kb, g * r + m, li, raw);
            lvr_unpack(raw, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) c[e] += x[e];
        }
    }
    const float inv = 1.0f / (float)r;
#pragma unroll
    for (int e = 0; e < 8; ++e) c[e] *= inv;
    constexpr bool CF8 = CF == 1;
    char *Cb = static_cast<char *>(centres) + ((int64_t)bh * max_groups + g) * (LVR_D * (CF8 ? 1 : sizeof(KT)));
    if constexpr (CF8) {
        uint32_t code[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) code[e] = f32_to_e4m3(c[e]);
        const uint32_t w0 = code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);
        const uint32_t w1 = code[4] | (code[5] << 8) | (code[6] << 16) | (code[7] << 24);
        // from here on: the centre as stored (decoded by the same instruction the query kernel uses)
        const lvr_f32x2 d0 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w0, false), d1 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w0, true);
        const lvr_f32x2 d2 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w1, false), d3 = __builtin_amdgcn_cvt_pk_f32_fp8((int)w1, true);
        c[0] = d0[0]; c[1] = d0[1]; c[2] = d1[0]; c[3] = d1[1];
        c[4] = d2[0]; c[5] = d2[1]; c[6] = d3[0]; c[7] = d3[1];
        if (valid) *reinterpret_cast<uint2 *>(Cb + (li & 3) * 32 + (li >> 2) * 8) = make_uint2(w0, w1);
    } else if constexpr (std::is_same<KT, lvr_bf16_t>::value) {
        uint32_t b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            b[e] = lvr_f32_to_bf16_bits(c[e]);
            c[e] = __uint_as_float(b[e] << 16);   // from here on: the centre as stored
        }
        if (valid)
            reinterpret_cast<uint4 *>(Cb)[li] =
                make_uint4(b[0] | (b[1] << 16), b[2] | (b[3] << 16), b[4] | (b[5] << 16), b[6] | (b[7] << 16));
    } else {
        if (valid) {
            reinterpret_cast<float4 *>(Cb)[2 * li] = make_float4(c[0], c[1], c[2], c[3]);
            reinterpret_cast<float4 *>(Cb)[2 * li + 1] = make_float4(c[4], c[5], c[6], c[7]);
        }
    }

    const int lanes_per_sub = 16 / S;
    float cn2 = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) cn2 += c[e] * c[e];
    cn2 = seg_sum(cn2, lanes_per_sub);

    float max_d2 = 0.f;
    auto distance = [&](const float (&x)[8]) {
        float d2 = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float t = x[e] - c[e];
            d2 += t * t;
        }
        d2 = seg_sum(d2, lanes_per_sub);
        max_d2 = fmaxf(max_d2, d2);
    };
    if (kept) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (m < r) {            // uniform: every lane takes part in the reduction
                float x[8];
                lvr_unpack(keep[m], x);
                distance(x);
            }
        }
    } else {
        for (int m = 0; m < r; ++m) {
            float x[8];
            lvr_load8<KT>(Sb + (g * r + m) * row_stride, 0, li, x);
            distance(x);
        }
    }
    float rho = sqrtf(max_d2) * (1.0f + 0x1p-12f) + sqrtf(cn2) * 0x1p-12f;
    rho = __uint_as_float(__float_as_uint(rho) + 1u);    // one ulp up (rho >= 0)
    if constexpr (CF != 0) {
        // The radii go out in the form the query's radius step reads them: four bf16 per group (8 bytes),
        // slot s = rho_s rounded UP to bf16's eight significant bits (looser by at most 2^-7 rho_s, never
        // tighter), slots S..3 zero.
        uint32_t slot[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) slot[k] = 0;
        const int lane = threadIdx.x & 63, base = lane & ~15;
        for (int sidx = 0; sidx < S; ++sidx) {   // S <= 4
            const float rs = __shfl(rho, base + sidx * lanes_per_sub, 64);
            uint32_t up = __float_as_uint(rs);
            if (up & 0xffffu) up = (up & 0xffff0000u) + 0x10000u;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k == sidx) slot[k] = up >> 16;
        }
        if (valid && li == 0)
            reinterpret_cast<uint2 *>(radii)[(int64_t)bh * max_groups + g] =
                make_uint2(slot[0] | (slot[1] << 16), slot[2] | (slot[3] << 16));
    } else {
        if (valid && (li % lanes_per_sub) == 0) radii[((int64_t)bh * max_groups + g) * S + li / lanes_per_sub] = rho;
    }
}

// Balls with 6-bit centres, the default index.  A centre is stored as 128 e2m3 codes of 6 bits in the order the matrix-core
// operand wants them (bits 6 (kk*8 + j) .. of the 24 bytes at kq*24 hold coordinate kk*32 + kq*8 + j), times one power-of-two
// scale per kq: the 32 coordinates of a scale block are the ones a lane of the query kernel holds.  The scale is the smallest
// power of two that brings the block's largest magnitude to at most 7.5; its biased exponent byte goes into the group's
// record in `radii` (byte kq of the third word).  `chan`: LVR_CHAN_STRIDE bytes per (sequence, KV head), at LVR_D the factors
// 2^e_c; the index describes the keys with coordinate c divided by 2^e_c: centre, codes and radii are all formed in that space
// (an exact rescaling: powers of two), and the query multiplies q_c by 2^e_c, which leaves every dot product as it was.
//
// Four lanes per group, lane b of the quad holding the 32
// coordinates 32 kk + 8 b + e of scale block b in registers: the block's largest magnitude, its codes (one conversion
// instruction there, one back) and its share of every distance need no other lane, and what the coordinate blocks of Eq. (1)
// add up over the quad is two lane exchanges per radius.  A wave stores 16 groups' codes as 1536 consecutive bytes.
// R = group size up to four (the members stay in registers between the two passes); R = 0: any r, members read twice.
// Bound by memory: K in, K out and 108 bytes per group (650 MB for 8 heads of 131072 keys).  With 16 lanes per group, a software encoder
// and a four-step exchange per reduction the vector ALU took longer than the traffic, 223 us; with four lanes 113-119 us.  Now 106 us: a lane's
// pieces of a row are 64 bytes apart, so what a wave stored at once were halves of lines, and the codes and records partial ones (420 MB
// written for 381 MB).  Rows (group sizes up to four), codes and records go through LDS and leave in whole lines.  Builds, us, before and after: 8 x 32768 keys
// 59.5 / 53.9, 128 x 32768 843 / 793, 8 x 131072 in groups of 1 (token-major), 2, 4: 221 / 209, 208 / 193, 206 / 185.
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float lvr_f32x16;

__device__ __forceinline__ float quad_sum(float v) {
    v += lvr_dpp<0xB1>(v);   // lane ^ 1
    v += lvr_dpp<0x4E>(v);   // lane ^ 2
    return v;
}

template <int R, int S>
__global__ void __launch_bounds__(256)
build_groups6_kernel(void *__restrict__ K, void *__restrict__ centres, float *__restrict__ radii, int64_t cap_rows,
                     int64_t max_groups, int64_t g0, int64_t g1, int r, const BuildSrc src, const int8_t *__restrict__ chan) {
    constexpr int KEEP = R ? R : 1;
    __shared__ uint4 s_codes[64 * 6];    // 96 bytes of codes per group
    __shared__ uint32_t s_rec[64 * 3];   // 12 bytes of radii and scales
    constexpr bool STAGED = R != 0;      // the rows stay until the whole workgroup writes them
    __shared__ uint4 s_row[STAGED ? 64 * R * 16 : 1];
    const int bh = blockIdx.y;
    const int b = threadIdx.x & 3;
    int64_t g = g0 + (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2);
    const bool valid = g < g1;
    if (!valid) g = g0;   // keep every lane busy so the exchanges below see defined data
    char *Kb = static_cast<char *>(K) + (int64_t)bh * cap_rows * LVR_D * 2;
    const bool from_src = src.base != nullptr;   // uniform
    const char *Sb = from_src ? src.base + ((int64_t)(bh / src.n_kv_heads) * src.sb + (int64_t)(bh % src.n_kv_heads) * src.sh) * 2 : Kb;
    const int64_t row_stride = from_src ? src.st * 2 : (int64_t)LVR_D * 2;
    const int members = R ? R : r;
    uint4 raw[KEEP][4];
    auto fetch = [&](int m, uint4 (&w)[4]) {   // this lane's four pieces of member m
        const uint4 *p = reinterpret_cast<const uint4 *>(Sb + (g * members + m) * row_stride) + b;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) w[kk] = p[kk * 4];
    };
    auto keep_row = [&](int m, const uint4 (&w)[4]) {   // the arena's copy of the row
        if constexpr (STAGED) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) s_row[((threadIdx.x >> 2) * R + m) * 16 + b + kk * 4] = w[kk];
            return;
        }
        uint4 *p = reinterpret_cast<uint4 *>(Kb + (g * members + m) * (LVR_D * 2)) + b;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            __builtin_nontemporal_store(__builtin_bit_cast(lvr_u32x4, w[kk]), reinterpret_cast<lvr_u32x4 *>(p + kk * 4));
        }
    };
    auto value = [](const uint4 &w, int e) {
        const uint32_t u = e < 2 ? w.x : (e < 4 ? w.y : (e < 6 ? w.z : w.w));
        return (e & 1) ? lvr_bf16_hi(u) : lvr_bf16_lo(u);
    };
    if constexpr (R != 0) {
#pragma unroll
        for (int m = 0; m < R; ++m) fetch(m, raw[m]);
    }
    // 2^-e_c of this lane's coordinates, from the factors 2^e_c: the exponent field of the reciprocal of a power of two
    float chs[32];
    {
        const float4 *cf = reinterpret_cast<const float4 *>(chan + (int64_t)bh * LVR_CHAN_STRIDE + LVR_D) + b * 2;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const float4 x = cf[kk * 8], y = cf[kk * 8 + 1];
            const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) chs[kk * 8 + e] = __uint_as_float((254u << 23) - __float_as_uint(f[e]));
        }
    }
    float c[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) c[i] = 0.f;
    auto add_member = [&](const uint4 (&w)[4]) {   // members in ascending row order
#pragma unroll
        for (int i = 0; i < 32; ++i) c[i] += value(w[i / 8], i % 8);
    };
    if constexpr (R != 0) {
#pragma unroll
        for (int m = 0; m < R; ++m) {
            if (from_src && valid) keep_row(m, raw[m]);
            add_member(raw[m]);
        }
    } else {
        for (int m = 0; m < members; ++m) {
            fetch(m, raw[0]);
            if (from_src && valid) keep_row(m, raw[0]);
            add_member(raw[0]);
        }
    }
    const float inv = 1.0f / (float)members;   // a power of two: exact
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        c[i] = c[i] * inv * chs[i];
        amax = fmaxf(amax, fabsf(c[i]));
    }
    // smallest E with amax <= 7.5 * 2^E; held to [-100, 120] so that scale and every decoded value are normal numbers (a
    // block beyond that saturates or rounds to zero; the radius measures it)
    int p;
    const float f = frexpf(amax, &p);   // amax = f * 2^p, f in [0.5, 1)
    int E = (amax > 0.f) ? (f <= 0.9375f ? p - 3 : p - 2) : -100;
    E = E < -100 ? -100 : (E > 120 ? 120 : E);
    const float scale = __uint_as_float((uint32_t)(E + 127) << 23);
    lvr_f32x16 even, odd;   // the conversion interleaves its two operands: code 2i from the first, 2i + 1 from the second
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        even[i] = c[2 * i];
        odd[i] = c[2 * i + 1];
    }
    const lvr_u32x6 code = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(even, odd, scale);
    // from here on: the centre as stored (decoded by the conversion the query kernel uses, in its fp32 form)
    const lvr_f32x32 dec = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(code, scale);
    {
        uint2 *dst = reinterpret_cast<uint2 *>(s_codes) + (threadIdx.x >> 2) * 12 + b * 3;
        dst[0] = make_uint2(code[0], code[1]);
        dst[1] = make_uint2(code[2], code[3]);
        dst[2] = make_uint2(code[4], code[5]);
    }
    constexpr int SPAN = 32 / S;   // this lane's coordinates of one coordinate block are consecutive: 4/S steps of 8
    float cn2[S], max_d2[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < SPAN; ++i) t += dec[s * SPAN + i] * dec[s * SPAN + i];
        cn2[s] = quad_sum(t);
        max_d2[s] = 0.f;
    }
    auto distance = [&](const uint4 (&w)[4]) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            float d2 = 0.f;
#pragma unroll
            for (int i = s * SPAN; i < (s + 1) * SPAN; ++i) {
                const float t = value(w[i / 8], i % 8) * chs[i] - dec[i];
                d2 += t * t;
            }
            max_d2[s] = fmaxf(max_d2[s], quad_sum(d2));
        }
    };
    if constexpr (R != 0) {
#pragma unroll
        for (int m = 0; m < R; ++m) distance(raw[m]);
    } else {
        for (int m = 0; m < members; ++m) {
            fetch(m, raw[0]);
            distance(raw[0]);
        }
    }
    // lane b forms radius b of the record (slots S..3 are zero): widened as above, then rounded UP to bf16
    float d2 = max_d2[0], n2 = cn2[0];
#pragma unroll
    for (int s = 1; s < S; ++s) {
        d2 = b == s ? max_d2[s] : d2;
        n2 = b == s ? cn2[s] : n2;
    }
    float rho = sqrtf(d2) * (1.0f + 0x1p-12f) + sqrtf(n2) * 0x1p-12f;
    uint32_t up = __float_as_uint(rho) + 1u;   // one ulp up (rho >= 0)
    if (up & 0xffffu) up = (up & 0xffff0000u) + 0x10000u;
    const uint32_t mine = b < S ? up >> 16 : 0u;
    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xf, 0xf, false);   // lane ^ 1
    uint32_t scales = (uint32_t)(E + 127) << (8 * b);
    scales |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)scales, 0xB1, 0xf, 0xf, false);
    scales |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)scales, 0x4E, 0xf, 0xf, false);
    if (b != 3)   // 12-byte record: two words of radii (lanes 0 and 2 hold them), then the scale bytes
        s_rec[(threadIdx.x >> 2) * 3 + (b == 0 ? 0 : (b == 2 ? 1 : 2))] = b == 1 ? scales : mine | (next << 16);
    __syncthreads();
    const int64_t first = g0 + (int64_t)blockIdx.x * 64;
    const int groups = g1 - first < 64 ? (int)(g1 - first) : 64;
    if constexpr (STAGED) {
        if (from_src) {
            lvr_u32x4 *rows = reinterpret_cast<lvr_u32x4 *>(Kb + first * R * (LVR_D * 2));
#pragma unroll
            for (int u = 0; u < 4 * R; ++u) {
                const int i = threadIdx.x + 256 * u;
                if (i < groups * R * 16) __builtin_nontemporal_store(__builtin_bit_cast(lvr_u32x4, s_row[i]), rows + i);
            }
        }
    }
    uint4 *out = reinterpret_cast<uint4 *>(static_cast<char *>(centres) + ((int64_t)bh * max_groups + first) * (LVR_D * 3 / 4));
    for (int i = threadIdx.x; i < groups * 6; i += 256) out[i] = s_codes[i];
    uint32_t *rec = reinterpret_cast<uint32_t *>(radii) + ((int64_t)bh * max_groups + first) * 3;
    if ((int)threadIdx.x < groups * 3) rec[threadIdx.x] = s_rec[threadIdx.x];
}

// Axis-aligned box of every group (appendix "Ablation on Index Design", Def. 1): per coordinate the
// largest and the smallest member value, stored as two rows (upper corner, lower corner).  The
// corners are member values, so bf16 storage is exact.  The one float per group in `radii` is a
// rounding allowance for the bound  sum_c (q+_c hi_c + q-_c lo_c)  evaluated in fp32 over 256
// terms: 2^-15 * |a|_2 with a_c = max(|lo_c|, |hi_c|); times |q|_2 it exceeds the rounding error
// by Cauchy-Schwarz, so a computed bound never falls below a member's exact score.
// CF8: the corners are stored as e4m3 codes in matrix-operand order, the upper corner rounded up and
// the lower corner rounded down, so the stored box contains the exact one.  A member beyond +-448
// cannot be enclosed by a code; what sticks out (e_c per coordinate) is added to the allowance as
// |e|_2, which times |q|_2 exceeds sum_c |q_c| e_c.
template <bool CF8>
__global__ void __launch_bounds__(256)
build_boxes_kernel(void *__restrict__ K, void *__restrict__ corners, float *__restrict__ allowance,
                   int64_t cap_rows, int64_t max_groups, int64_t g0, int64_t g1, int r, const BuildSrc src) {
    const int bh = blockIdx.y;
    const int li = threadIdx.x & 15;
    int64_t g = g0 + (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const bool valid = g < g1;
    if (!valid) g = g0;
    char *Kb = static_cast<char *>(K) + (int64_t)bh * cap_rows * LVR_D * 2;
    const bool from_src = src.base != nullptr;   // uniform
    const char *Sb = from_src ? src.base + ((int64_t)(bh / src.n_kv_heads) * src.sb + (int64_t)(bh % src.n_kv_heads) * src.sh) * 2 : Kb;
    const int64_t row_stride = from_src ? src.st * 2 : (int64_t)LVR_D * 2;
    float lo[8], hi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lo[e] = INFINITY;
        hi[e] = -INFINITY;
    }
    for (int m = 0; m < r; ++m) {
        float x[8];
        lvr_raw8<lvr_bf16_t> raw;
        lvr_load_raw(Sb + (g * r + m) * row_stride, 0, li, raw);
        if (from_src && valid) lvr_store_raw(Kb, g * r + m, li, raw);   // the arena's copy of the row
        lvr_unpack(raw, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            lo[e] = fminf(lo[e], x[e]);
            hi[e] = fmaxf(hi[e], x[e]);
        }
    }
    float a2 = 0.f;
    if constexpr (CF8) {
        uint32_t ch[8], cl[8];
        float e2 = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            ch[e] = f32_to_e4m3_directed(hi[e], true);
            cl[e] = f32_to_e4m3_directed(lo[e], false);
            const float hd = e4m3_value(ch[e]), ld = e4m3_value(cl[e]);
            const float out = fmaxf(fmaxf(hi[e] - hd, ld - lo[e]), 0.f);   // non-zero only beyond +-448
            e2 += out * out;
            const float a = fmaxf(fabsf(ld), fabsf(hd));
            a2 += a * a;
        }
        a2 = seg_sum(a2, 16);
        e2 = seg_sum(e2, 16);
        if (valid) {
            char *dst = static_cast<char *>(corners) + ((int64_t)bh * max_groups + g) * 2 * LVR_D;
            const int at = (li & 3) * 32 + (li >> 2) * 8;
            *reinterpret_cast<uint2 *>(dst + at) = make_uint2(ch[0] | (ch[1] << 8) | (ch[2] << 16) | (ch[3] << 24),
                                                              ch[4] | (ch[5] << 8) | (ch[6] << 16) | (ch[7] << 24));
            *reinterpret_cast<uint2 *>(dst + LVR_D + at) = make_uint2(cl[0] | (cl[1] << 8) | (cl[2] << 16) | (cl[3] << 24),
                                                                      cl[4] | (cl[5] << 8) | (cl[6] << 16) | (cl[7] << 24));
            if (li == 0) {
                float al = sqrtf(a2) * 0x1p-15f + sqrtf(e2) * (1.0f + 0x1p-20f);
                allowance[(int64_t)bh * max_groups + g] = __uint_as_float(__float_as_uint(al) + 1u);
            }
        }
        return;
    }
    uint32_t bh_[8], bl_[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float a = fmaxf(fabsf(lo[e]), fabsf(hi[e]));
        a2 += a * a;
        bh_[e] = __float_as_uint(hi[e]) >> 16;   // exact: the values are bf16 already
        bl_[e] = __float_as_uint(lo[e]) >> 16;
    }
    a2 = seg_sum(a2, 16);
    if (valid) {
        uint4 *dst = reinterpret_cast<uint4 *>(static_cast<char *>(corners) +
                                               ((int64_t)bh * max_groups + g) * 2 * LVR_D * 2);
        dst[li] = make_uint4(bh_[0] | (bh_[1] << 16), bh_[2] | (bh_[3] << 16), bh_[4] | (bh_[5] << 16),
                             bh_[6] | (bh_[7] << 16));
        dst[16 + li] = make_uint4(bl_[0] | (bl_[1] << 16), bl_[2] | (bl_[3] << 16), bl_[4] | (bl_[5] << 16),
                                  bl_[6] | (bl_[7] << 16));
        if (li == 0) {
            float al = sqrtf(a2) * 0x1p-15f;
            allowance[(int64_t)bh * max_groups + g] = __uint_as_float(__float_as_uint(al) + 1u);
        }
    }
}

// Identity position map for rows [row0, row0+rows) (used when rows are stored in arrival order
// but a map is kept, i.e. the buffer of a regrouped arena).
__global__ void iota_rows_kernel(int32_t *slot_pos, int32_t *pos_slot, int64_t cap_rows, int64_t row0, int64_t rows) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows) return;
    int64_t o = (int64_t)blockIdx.y * cap_rows + row0 + i;
    slot_pos[o] = (int32_t)(row0 + i);
    pos_slot[o] = (int32_t)(row0 + i);
}

}  // namespace

hipError_t lvr_launch_copy_kv(lvr_index *ix, const void *K, const int64_t ks[3], const void *V, const int64_t vs[3],
                              int64_t dst_row0, int64_t rows, hipStream_t st, int64_t k_first) {
    if (rows <= 0) return hipSuccess;
    // k_first > 0: the leading key rows are written by the build kernel that reads them from the caller's K
    CopySide k{static_cast<const char *>(K), static_cast<char *>(ix->K), ks[0], ks[1], ks[2], k_first};
    CopySide v{static_cast<const char *>(V), static_cast<char *>(ix->V), vs[0], vs[1], vs[2], 0};
    const int sh = ix->elt == 2 ? 4 : 5;
    const unsigned v_blocks = copy_blocks(rows, sh, COPY_PIECES);
    // an append's rows are read again by the next launch; of a build, only the values come this way (and the ungrouped tail)
    const bool stream = k_first > 0 && streamed(rows, lvr_n_bh(ix), LVR_D * ix->elt);
    const dim3 grid(v_blocks + copy_blocks(rows - k_first, sh, COPY_PIECES), (unsigned)lvr_n_bh(ix));
#define LVR_COPY_LAUNCH(SH, STREAM)                                                                                      \
    hipLaunchKernelGGL((copy_rows_kernel<SH, STREAM>), grid, dim3(256), 0, st, k, v, ix->cfg.n_kv_heads, ix->cap_rows,    \
                       dst_row0, rows, v_blocks)
    if (sh == 4) {
        if (stream) LVR_COPY_LAUNCH(4, true);
        else LVR_COPY_LAUNCH(4, false);
    } else {
        if (stream) LVR_COPY_LAUNCH(5, true);
        else LVR_COPY_LAUNCH(5, false);
    }
#undef LVR_COPY_LAUNCH
    return hipGetLastError();
}

hipError_t lvr_launch_build_groups(lvr_index *ix, int64_t g0, int64_t g1, hipStream_t st, const void *K_src,
                                   const int64_t *ks) {
    if (g1 <= g0) return hipSuccess;
    dim3 grid((unsigned)((g1 - g0 + 15) / 16), (unsigned)lvr_n_bh(ix));
    // K_src: the groups' rows come from the caller's K (element strides ks) and are copied into the arena on the way
    BuildSrc src{static_cast<const char *>(K_src), K_src ? ks[0] : 0, K_src ? ks[1] : 0, K_src ? ks[2] : 0, ix->cfg.n_kv_heads};
    if (ix->box) {
        if (ix->cf8)
            hipLaunchKernelGGL(build_boxes_kernel<true>, grid, dim3(256), 0, st, ix->K, ix->centres, ix->radii, ix->cap_rows,
                               ix->max_groups, g0, g1, ix->cfg.group_size, src);
        else
            hipLaunchKernelGGL(build_boxes_kernel<false>, grid, dim3(256), 0, st, ix->K, ix->centres, ix->radii, ix->cap_rows,
                               ix->max_groups, g0, g1, ix->cfg.group_size, src);
        return hipGetLastError();
    }
    if (ix->cf6) {
        grid.x = (unsigned)((g1 - g0 + 63) / 64);   // four lanes per group
        const int r = ix->cfg.group_size;
#define LVR_B6_LAUNCH(R, S)                                                                                               \
    hipLaunchKernelGGL((build_groups6_kernel<R, S>), grid, dim3(256), 0, st, ix->K, ix->centres, ix->radii, ix->cap_rows, \
                       ix->max_groups, g0, g1, r, src, lvr_chan_exp(ix))
#define LVR_B6_ANY(S)                 \
    do {                              \
        if (r == 1) LVR_B6_LAUNCH(1, S);      \
        else if (r == 2) LVR_B6_LAUNCH(2, S); \
        else if (r == 4) LVR_B6_LAUNCH(4, S); \
        else LVR_B6_LAUNCH(0, S);             \
    } while (0)
        if (ix->cfg.n_subspaces == 1) LVR_B6_ANY(1);
        else if (ix->cfg.n_subspaces == 2) LVR_B6_ANY(2);
        else LVR_B6_ANY(4);
#undef LVR_B6_ANY
#undef LVR_B6_LAUNCH
    } else if (ix->cf8)
        hipLaunchKernelGGL((build_groups_kernel<lvr_bf16_t, 1>), grid, dim3(256), 0, st, ix->K, ix->centres, ix->radii,
                           ix->cap_rows, ix->max_groups, g0, g1, ix->cfg.group_size, ix->cfg.n_subspaces, src);
    else if (ix->cfg.kv_dtype == LVR_BF16)
        hipLaunchKernelGGL(build_groups_kernel<lvr_bf16_t>, grid, dim3(256), 0, st, ix->K, ix->centres, ix->radii,
                           ix->cap_rows, ix->max_groups, g0, g1, ix->cfg.group_size, ix->cfg.n_subspaces, src);
    else
        hipLaunchKernelGGL(build_groups_kernel<lvr_f32_t>, grid, dim3(256), 0, st, ix->K, ix->centres, ix->radii,
                           ix->cap_rows, ix->max_groups, g0, g1, ix->cfg.group_size, ix->cfg.n_subspaces, src);
    return hipGetLastError();
}

namespace {

// Channel exponents of a (sequence, KV head): with L_c = log2(rms of coordinate c) over a sample of the rows,
// e_c = round(L_c - o), held to [-8, 8]; a coordinate that is zero throughout keeps e_c = 0.  The offset o (the same for
// all 128 channels, so it only moves the block scales) is the circular mean of the fractional parts of L_c: channels of
// about the same size then sit in the middle of one rounding interval and get the same exponent, instead of being split
// by a boundary that happens to fall among them.  Any exponents give a correct index (the radii are measured in the
// rescaled space against the centres as stored there); these make the coordinates of a key comparable in size, so that
// the 32 coordinates that share a scale in the 6-bit code are not drowned by one large channel.
//
// Up to CHAN_SPLITS workgroups per (sequence, KV head) add up squares, 16 lanes per row with
// 16-byte loads, four rows of every lane in flight; a sample of 4096 rows is one round trip to memory for 64 workgroups.  The last of
// them to end adds the workgroups' sums in order (the exponents do not depend on timing) and forms the exponents: the sums are
// stored and read with device scope, and a workgroup takes its ticket once its own are in memory.  What is left is the latency of one launch and its
// trips, so where V has to be copied as well (contiguous groups) the copy rides behind the sums of each (sequence, KV head).
// As one workgroup per (sequence, KV head) with a 2-byte load and an add per row the sums alone took 826 us.  With sums and exponents in
// launches of their own, half of the copy behind each, and now, builds, us: 8 x 1500 keys 14.2 / 12.3, 8 x 9001 25.0 / 22.3, 8 x 32768
// 53.9 / 51.3, 8 x 131072 198 / 194.  A workgroup has a fixed cost (the sums' way out, the ticket, three barriers), so with 64 of them for every one
// of many (sequence, KV head) the sums were no longer bound by memory (256 x 4096 rows 81 us alone, 64 with 16 each; a read of them 45)
// and builds were slower than before the single launch: 128 x 32768 791 -> 807.  2048 workgroups, eight per compute unit and so one round,
// and at least 16 per (sequence, KV head), from 64 each: 64 x 32768 404 / 400, 128 x 32768 820 / 806, 256 x 16384 863 / 844, 256 x 4096 in groups of four
// 221 / 204, 512 x 4096 515 / 495; at least 8: 804, 849, 208, 498; 4096 workgroups: 808, 842, 204, 496, but 64 x 32768 405.
constexpr int CHAN_SPLITS = 64;

struct ChannelArgs {
    const char *K;
    int64_t sb, sh, st;       // element strides
    int64_t rows, step;       // sampled rows, every step-th of the caller's
    int n_kv_heads, splits;   // workgroups per (sequence, KV head) that add up squares
    float *part;              // [n_bh][splits][128]
    int8_t *chan_exp;
    int32_t *ticket;          // zero between launches, ticket_stride apart per (sequence, KV head)
    int ticket_stride;
};

// Returns whether this workgroup is the last of its (sequence, KV head) to end: all sums are then in memory.
__device__ __forceinline__ bool channel_sums(const ChannelArgs &a, int bh, int split) {   // 256 threads
    __shared__ float s_sum[4][LVR_D];
    __shared__ int s_arrived;
    const int64_t rows = a.rows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15;
    const char *base = a.K + ((int64_t)(bh / a.n_kv_heads) * a.sb + (int64_t)(bh % a.n_kv_heads) * a.sh) * 2;
    const int64_t share = (rows + a.splits - 1) / a.splits;   // sampled rows of this workgroup
    const int64_t first = split * share, end = first + share < rows ? first + share : rows;
    float ss[8];
    lvr_zero8(ss);
    for (int64_t i0 = first + (threadIdx.x >> 4); i0 < end; i0 += 64) {
        lvr_raw8<lvr_bf16_t> raw[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + 16 * u;
            lvr_load_raw(base + (i < end ? i : i0) * a.step * a.st * 2, 0, li, raw[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float x[8];
            lvr_unpack(raw[u], x);
            const bool in = i0 + 16 * u < end;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss[e] += in ? x[e] * x[e] : 0.f;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        ss[e] += __shfl_xor(ss[e], 16, 64);
        ss[e] += __shfl_xor(ss[e], 32, 64);
        if (lane < 16) s_sum[wave][li * 8 + e] = ss[e];
    }
    __syncthreads();
    if (threadIdx.x < LVR_D) {
        const int c = threadIdx.x;
        __hip_atomic_store(&a.part[((int64_t)bh * a.splits + split) * LVR_D + c], (s_sum[0][c] + s_sum[1][c]) + (s_sum[2][c] + s_sum[3][c]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's sums have reached the memory all compute units share
    __syncthreads();
    int32_t *ticket = &a.ticket[(int64_t)bh * a.ticket_stride];
    if (threadIdx.x == 0) s_arrived = atomicAdd(ticket, 1);
    __syncthreads();
    if (s_arrived != a.splits - 1) return false;
    if (threadIdx.x == 0) *ticket = 0;
    return true;
}

__device__ __forceinline__ void channel_exponents(const ChannelArgs &a, int bh) {   // 256 threads, the upper half repeats the lower
    __shared__ float s_dir[2][2];
    const int c = threadIdx.x & (LVR_D - 1), wave = (threadIdx.x >> 6) & 1;
    const float *p = a.part + (int64_t)bh * a.splits * LVR_D + c;
    float ss = 0.f;
#pragma unroll 16
    for (int k = 0; k < a.splits; ++k) ss += __hip_atomic_load(&p[(int64_t)k * LVR_D], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float ms = ss / (float)(a.rows > 0 ? a.rows : 1);
    const bool live = ms > 0.f && ms < INFINITY;
    const float L = live ? 0.5f * log2f(ms) : 0.f;
    constexpr float kTwoPi = 6.283185307179586f;
    // the sum over the channels of the directions of L_c's fractional part, in the same order in every thread: one offset
    float sc = live ? cosf(kTwoPi * L) : 0.f, sn = live ? sinf(kTwoPi * L) : 0.f;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        sc += __shfl_xor(sc, off, 64);
        sn += __shfl_xor(sn, off, 64);
    }
    if (threadIdx.x < LVR_D && (c & 63) == 0) {
        s_dir[wave][0] = sc;
        s_dir[wave][1] = sn;
    }
    __syncthreads();
    sc = s_dir[0][0] + s_dir[1][0];
    sn = s_dir[0][1] + s_dir[1][1];
    const float o = (sc != 0.f || sn != 0.f) ? atan2f(sn, sc) / kTwoPi : 0.f;
    int e = 0;
    if (live) {
        e = (int)rintf(L - o);
        e = e < -8 ? -8 : (e > 8 ? 8 : e);
    }
    if (threadIdx.x < LVR_D) {
        int8_t *mine = a.chan_exp + (int64_t)bh * LVR_CHAN_STRIDE;
        mine[c] = (int8_t)e;
        reinterpret_cast<float *>(mine + LVR_D)[c] = __uint_as_float((uint32_t)(127 + e) << 23);
    }
}

// Sums and exponents, and behind those of each (sequence, KV head) the copy of its values' rows [0, rows) and keys' rows [k.first, rows)
// (v_blocks = 0 and an empty key range: no copy).
__global__ void __launch_bounds__(256)
channel_step_kernel(ChannelArgs a, CopySide k, CopySide v, int64_t cap_rows, int64_t rows, unsigned v_blocks) {
    const unsigned lead = (unsigned)a.splits;
    if (blockIdx.x < lead) {
        if (channel_sums(a, blockIdx.y, blockIdx.x)) channel_exponents(a, blockIdx.y);
    } else if (blockIdx.x - lead < v_blocks) copy_block<4, STEP_PIECES, true>(v, blockIdx.y, a.n_kv_heads, cap_rows, 0, rows, blockIdx.x - lead);
    else copy_block<4, STEP_PIECES, true>(k, blockIdx.y, a.n_kv_heads, cap_rows, 0, rows, blockIdx.x - lead - v_blocks);
}

}  // namespace

// The workgroups' sums go through the attention's partial-output buffer (G * Pmax * 128 floats per (sequence, KV head),
// Pmax >= 4), which no launch in flight on the same stream still needs once these run.
// V != NULL: the launch also copies all n value rows and the key rows from k_first on.
hipError_t lvr_launch_channel_scales(lvr_index *ix, const void *K, const int64_t ks[3], int64_t n, hipStream_t st, const void *V,
                                     const int64_t *vs, int64_t k_first) {
    if (!ix->chan_scaled || n <= 0) return hipSuccess;
    ChannelArgs a;
    a.K = static_cast<const char *>(K);
    a.sb = ks[0];
    a.sh = ks[1];
    a.st = ks[2];
    a.step = (n + 4095) / 4096;   // at most 4096 rows are looked at
    a.rows = (n + a.step - 1) / a.step;
    a.n_kv_heads = ix->cfg.n_kv_heads;
    const int room = ix->G * (ix->P > ix->P_dense ? ix->P : ix->P_dense);
    a.splits = (int)((a.rows + 63) / 64);     // 64 rows: four per lane quarter of a workgroup
    if (a.splits > CHAN_SPLITS) a.splits = CHAN_SPLITS;
    const int n_bh = lvr_n_bh(ix), most = n_bh >= 128 ? 16 : 2048 / n_bh;   // 2048 workgroups, at least 16 per (sequence, KV head)
    if (a.splits > most) {
        const int64_t each = (a.rows + 64 * most - 1) / (64 * most) * 64;   // whole rounds of 64 rows
        a.splits = (int)((a.rows + each - 1) / each);
    }
    if (a.splits > room) a.splits = room;
    a.part = ix->part_o;
    a.chan_exp = lvr_chan_exp(ix);
    a.ticket = lvr_channel_ticket(ix);
    a.ticket_stride = ix->G * LVR_CNT_STRIDE;
    CopySide k{a.K, static_cast<char *>(ix->K), ks[0], ks[1], ks[2], V ? k_first : n};
    CopySide v{static_cast<const char *>(V), static_cast<char *>(ix->V), V ? vs[0] : 0, V ? vs[1] : 0, V ? vs[2] : 0, 0};
    const unsigned v_blocks = V ? copy_blocks(n, 4, STEP_PIECES) : 0;
    hipLaunchKernelGGL(channel_step_kernel, dim3((unsigned)a.splits + v_blocks + copy_blocks(n - k.first, 4, STEP_PIECES), (unsigned)n_bh),
                       dim3(256), 0, st, a, k, v, ix->cap_rows, n, v_blocks);
    return hipGetLastError();
}

hipError_t lvr_launch_iota_rows(lvr_index *ix, int64_t row0, int64_t rows, hipStream_t st) {
    if (rows <= 0 || !ix->slot_pos) return hipSuccess;
    dim3 grid((unsigned)((rows + 255) / 256), (unsigned)lvr_n_bh(ix));
    hipLaunchKernelGGL(iota_rows_kernel, grid, dim3(256), 0, st, ix->slot_pos, ix->pos_slot, ix->cap_rows, row0, rows);
    return hipGetLastError();
}
