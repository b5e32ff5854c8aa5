// Backward passes of the lattice operations (Sec. "Implementation": the
// network is trained end to end, so each operation needs the gradient of a
// loss with respect to its inputs).  Every forward here is linear in the
// quantity differentiated, so each gradient is the transposed map:
//
//   slice  f_p = sum_k b_pk y_{v_k}      ->  dy_v = sum_{(p,k): v_k = v} b_pk df_p
//          (Eq. splat applied to df: the splat's pair-list gather, splat.hip)
//   splat  x_v = sum_p b_pv f_p          ->  df_p = sum_k b_pk dx_{v_k}
//          (Eq. slice applied to dx: the slice kernel, slice.hip; the
//          normalised splat divides dx_v by w_v first)
//   conv   y_v = sum_t x_{nbr(v,t)} W_t^T
//          dx_u = sum over (v, t) with nbr(v,t) = u of g_v W_t
//          dW_t = sum_v g_v^T x_{nbr(v,t)}
//
// Input gradient.  The 1-hop ring is symmetric (Sec. "Permutohedral
// Lattice": the neighbours sit at +-n_j): tap 1+j of v is u exactly when tap
// d+2+j of u is v, and tap 0 is the vertex itself.  So dx_u = sum_s
// g_{nbr(u,s)} W_{flip(s)}, a forward convolution of g with the weights
// W'[i][s][o] = W[o][flip(s)][i].  k_flip_weights builds W' and the forward
// conv kernels (conv.hip) run it: no scatter, no atomics.
//
// Weight gradient.  For each tap, dW_t [C_out x C_in] is a product whose
// reduction runs over the V vertices: A = g^T (rows of g, contiguous) and
// B = the gathered rows x_{nbr(v,t)}.  k_conv_wgrad_taps (bf16 MFMA, three taps
// a workgroup) covers channel counts that are multiples of 4 with aligned
// rows, in bf16 and in fp32 on fp32 rows; k_conv_wgrad the rest: each workgroup
// one tap, one 64 x 64 tile of (output, input) channels and one chunk of the
// vertices (chunk c of nch covers rows [c V / nch, (c+1) V / nch), V read on
// the device).  Per step of 32 vertices it stages the 32 g rows and the 32
// gathered x rows in LDS as fp32 and four wavefronts each accumulate a
// 32 x 32 block with v_mfma_f32_32x32x2f32 (K = the vertex index).  Each
// chunk writes its tile to a partial buffer; k_wgrad_reduce adds the nch
// partials in a fixed order, so the result does not depend on scheduling.
// The bias gradient (sum_v g_v) is summed from the same g rows by the
// workgroups of tap 0 and the first input tile.
#include "internal.h"

namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kBlock = 256;
constexpr int kTile = 64;   // output and input channels per tile
constexpr int kStep = 32;   // vertices per K step
constexpr int kRowsPer = kStep / (kBlock / 16);  // rows each loader thread stages per step
constexpr int kWgPerCu = 4;  // weight-gradient workgroups per CU the chunk count aims at
// (32-row steps at four workgroups per CU measured best over 64 and 128 rows
// at two to eight workgroups per CU, on 64x64, 64x128 and 128x128 shapes)

// fp32 -> bf16 -> fp32, round to nearest with ties to even (NaN stays NaN).
__device__ __forceinline__ float round_bf16(float f) {
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return __uint_as_float(u | 0x00400000u);
    return __uint_as_float((u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u);
}

// LDS tile [kStep][kTile] fp32.  Column c of an odd row sits at c ^ 32: the
// two 32-lane halves of an MFMA operand read (rows k and k+1, same columns)
// then fall on different banks.
__device__ __forceinline__ int swz(int k, int c) { return k * kTile + (c ^ ((k & 1) << 5)); }

// Four consecutive channels [c, c+4) of row `row` (fp32 or bf16 storage),
// zero past C.  VEC: C % 4 == 0 and the rows are 16-byte (fp32) or 8-byte
// (bf16) aligned.
template <bool BF16, bool VEC>
__device__ __forceinline__ float4 load4(const void *base, int64_t row, int C, int c) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (VEC) {
        if (c >= C) return r;
        if (BF16) {
            const uint2 u = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(base) + row * C + c);
            r.x = __uint_as_float(u.x << 16);
            r.y = __uint_as_float(u.x & 0xffff0000u);
            r.z = __uint_as_float(u.y << 16);
            r.w = __uint_as_float(u.y & 0xffff0000u);
        } else {
            r = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(base) + row * C + c);
        }
        return r;
    }
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = 0.f;
        if (c + e < C) {
            if (BF16)
                v[e] = __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(base)[row * C + c + e] << 16);
            else
                v[e] = reinterpret_cast<const float *>(base)[row * C + c + e];
        }
    }
    return make_float4(v[0], v[1], v[2], v[3]);
}

template <bool G_BF16, bool X_BF16, bool ROUND, bool VEC>
__global__ __launch_bounds__(kBlock) void k_conv_wgrad(const void *__restrict__ g, int C_out,
                                                       const void *__restrict__ x, int C_in, int T,
                                                       const int32_t *__restrict__ nbr,
                                                       const int32_t *__restrict__ counters, int nch,
                                                       float *__restrict__ partial, float *__restrict__ pbias) {
    __shared__ float gs[kStep * kTile];
    __shared__ float xs[kStep * kTile];
    __shared__ float bred[kBlock / 16][kTile];

    const int64_t V = counters[CNT_V];
    const int chunk = blockIdx.x;
    const int t = blockIdx.y;
    const int tiles_i = (C_in + kTile - 1) / kTile;
    const int o0 = (blockIdx.z / tiles_i) * kTile;
    const int i0 = (blockIdx.z % tiles_i) * kTile;
    const int64_t lo = V * chunk / nch;
    const int64_t hi = V * (chunk + 1) / nch;
    const bool do_bias = pbias != nullptr && t == 0 && i0 == 0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int h = lane >> 5;            // MFMA K index of this lane
    const int ow = (wave >> 1) * 32;    // this wave's 32 x 32 block
    const int iw = (wave & 1) * 32;
    // Loader mapping: thread owns channel chunk c4 (4 channels) of rows
    // r0, r0+16, r0+32, ... of the step.
    const int c4 = (tid & 15) * 4;
    const int r0 = tid >> 4;

    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    float bsum[4] = {0.f, 0.f, 0.f, 0.f};

    // The neighbour indices of a step are loaded one step before its rows,
    // so that a row gather never waits on its own index load.
    float4 ga[kRowsPer], xa[kRowsPer];
    int32_t ua[kRowsPer];
    auto load_index = [&](int64_t k0) {
#pragma unroll
        for (int j = 0; j < kRowsPer; ++j) {
            const int64_t v = k0 + r0 + 16 * j;
            ua[j] = v < hi ? nbr[v * T + t] : -1;
        }
    };
    auto load_step = [&](int64_t k0) {
#pragma unroll
        for (int j = 0; j < kRowsPer; ++j) {
            const int64_t v = k0 + r0 + 16 * j;
            ga[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            xa[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (v < hi) ga[j] = load4<G_BF16, VEC>(g, v, C_out, o0 + c4);
            if (ua[j] >= 0) xa[j] = load4<X_BF16, VEC>(x, ua[j], C_in, i0 + c4);
        }
    };
    if (lo < hi) {
        load_index(lo);
        load_step(lo);
        load_index(lo + kStep);
    }
    for (int64_t k0 = lo; k0 < hi; k0 += kStep) {
        // registers -> LDS (rounded to bf16 for a bf16 computation)
#pragma unroll
        for (int j = 0; j < kRowsPer; ++j) {
            const int k = r0 + 16 * j;
            float4 a = ga[j], b = xa[j];
            if (do_bias) {
                bsum[0] += a.x;
                bsum[1] += a.y;
                bsum[2] += a.z;
                bsum[3] += a.w;
            }
            // (rows stored as bf16 are already rounded)
            if (ROUND && !G_BF16) a = make_float4(round_bf16(a.x), round_bf16(a.y), round_bf16(a.z), round_bf16(a.w));
            if (ROUND && !X_BF16) b = make_float4(round_bf16(b.x), round_bf16(b.y), round_bf16(b.z), round_bf16(b.w));
            *reinterpret_cast<float4 *>(&gs[swz(k, c4)]) = a;
            *reinterpret_cast<float4 *>(&xs[swz(k, c4)]) = b;
        }
        __syncthreads();
        if (k0 + kStep < hi) {  // next step's loads in flight during the MFMAs
            load_step(k0 + kStep);
            load_index(k0 + 2 * kStep);
        }
#pragma unroll 8
        for (int s = 0; s < kStep / 2; ++s) {
            const int k = 2 * s + h;
            const float a = gs[swz(k, ow + (lane & 31))];
            const float b = xs[swz(k, iw + (lane & 31))];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
        }
        __syncthreads();
    }

    // Partial tile of this chunk: register r of lane l holds row
    // 8 (r / 4) + 4 (l / 32) + r % 4 (output channel), column l % 32 (input channel).
    const int64_t tapstride = C_in;
    float *dst = partial + (int64_t)chunk * C_out * T * C_in;
    const int ic = i0 + iw + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int oc = o0 + ow + 8 * (r >> 2) + 4 * h + (r & 3);
        if (oc < C_out && ic < C_in) dst[((int64_t)oc * T + t) * tapstride + ic] = acc[r];
    }
    if (do_bias) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bred[r0][c4 + e] = bsum[e];
        __syncthreads();
        if (tid < kTile) {
            float s = 0.f;
            for (int q = 0; q < kBlock / 16; ++q) s += bred[q][tid];
            if (o0 + tid < C_out) pbias[(int64_t)chunk * C_out + o0 + tid] = s;
        }
    }
}

// The weight gradient on bf16 MFMA (v_mfma_f32_32x32x16_bf16), for channel
// counts that are multiples of 4 and aligned rows: bf16 products (CM 1), or
// fp32 ones as the six largest products of three-term splits (CM 3, see
// split3).  Lane l supplies A[l % 32][8 (l / 32) + 0..7] and B[8 (l / 32) +
// 0..7][l % 32], eight consecutive K = vertex values.  So the step's rows are
// staged transposed in LDS, channel-major with the 32 vertices of the step
// contiguous: each thread loads two consecutive rows of four channels, packs
// the pair of each channel into one word (per plane) and stores it at
// [channel][vertex pair].  At a pitch of 17 words those writes fall on 64
// different banks.
//
// What bounds it is the latency of a step's gathers, not their bytes: a
// workgroup takes kTaps taps of its chunk, so that a step's g rows are loaded
// and staged once for three products, with two steps' rows in flight and two
// workgroups per CU (a tap per workgroup, one step ahead and four per CU kept
// fewer loads in flight and read g nine times).  With its reduction, us, T = 9,
// that kernel -> this one (fp32: fp32 MFMA 32x32x2 -> the split): V = 293 290: bf16
// 64 -> 64 121 -> 80, 128 -> 128 425 -> 277, from fp32 rows 205 -> 125, 753 -> 457, fp32
// 267 -> 160, 966 -> 632; V = 68 199: 37 -> 31, 107 -> 76, 56 -> 41, 170 -> 110, 73 -> 51,
// 235 -> 154; V = 5 752: 18.5 -> 16.2, 23.1 -> 24.5, 20.9 -> 17.2, 29.0 -> 27.5, 23.3 ->
// 20.7, 36.5 -> 34.7.  The largest, bf16 128 -> 128, runs at 312 TFLOP/s of the
// 2 400 the matrix cores reach: the transposing stores to LDS and the gathers'
// latency.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_t u32x4_a4_t __attribute__((aligned(4)));

constexpr int kTStep = 32;   // vertices per step (two MFMA K-steps of 16)
constexpr int kTRow = 68;    // LDS bytes per channel row: 32 bf16 + 4 bytes of padding
constexpr int kTaps = 3;     // taps per workgroup

// Four consecutive channels of a row as loaded: bf16 bits, or fp32, which
// goes through the split or is rounded to bf16 (to nearest even) only when its
// step is staged: a conversion here would wait for the load.
template <bool BF16>
struct Row4;
template <>
struct Row4<true> {
    uint2 u;
    __device__ __forceinline__ void load(const void *base, int64_t row, int C, int c) {
        u = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(base) + row * C + c);
    }
    __device__ __forceinline__ void zero() { u = make_uint2(0u, 0u); }
    // channel e of this row and of the next, the bf16 pair of one LDS word
    __device__ __forceinline__ uint32_t pair(const Row4 &next, int e) const {
        const int sh = (e & 1) * 16;
        return (((e < 2 ? u.x : u.y) >> sh) & 0xffffu) | (((e < 2 ? next.u.x : next.u.y) >> sh) << 16);
    }
};
template <>
struct Row4<false> {
    float f[4];
    __device__ __forceinline__ void load(const void *base, int64_t row, int C, int c) {
        const float4 t = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(base) + row * C + c);
        f[0] = t.x;
        f[1] = t.y;
        f[2] = t.z;
        f[3] = t.w;
    }
    __device__ __forceinline__ void zero() { f[0] = f[1] = f[2] = f[3] = 0.f; }
    __device__ __forceinline__ uint32_t pair(const Row4 &next, int e) const { return pack_bf16(f[e], next.f[e]); }
};

// Chunks that a launch uses for V vertices, at most `most`.  The host knows
// only the lattice's bound; the kernel and the reduction both take this count,
// so that a lattice far below its bound does not write and sum partials of a
// step or two.  It trades a chunk's serial steps against its partial, which
// grows with the tiles:
//   * about `per` steps a chunk, 6 for bf16 over several tiles, else 3, and no
//     fewer than `low` chunks while there are steps for them, 48 of one tile
//     and 16 of several.  In multiples of 16: the reduction's four groups load
//     four partials at a time.
//   * One tile, or two in bf16: no more than `one`, a workgroup per CU, before
//     a chunk has 2.75 (fp32) or 4.5 steps with two per CU: a second workgroup on
//     some CUs only makes those the last to end.
// us, T = 9, one-tap kernel | three taps, at least 2 tiles steps a chunk and 8
// chunks | this rule: bf16 64 -> 64 V = 3 000 17.9 | 14.3 | 14.2, 11 000 19.7 | 24.4
// | 19.1, 25 000 24.1 | 24.4 | 24.2; 96 -> 96 3 000 16.0 | 20.7 | 16.7, 7 000 20.9 | 23.5
// | 21.7; fp32 64 -> 64 3 000 20.0 | 18.4 | 16.9, 7 000 23.3 | 25.5 | 22.1; 96 -> 96
// 2 000 18.9 | 26.6 | 20.1, 3 000 22.1 | 34.5 | 23.3.  Where the one-tap kernel was
// still better: fp32 16 -> 16 below V = 8 000 by up to 1.6 us (3 000 12.2 | 15.4 |
// 13.8), bf16 of several tiles up to V = 11 000 by 3 to 8%.
struct ChunkRule {
    int most, per, low, one;
    int64_t two_from;  // steps from which more than `one` are used
    __device__ __forceinline__ int used(int64_t V) const {
        const int64_t steps = (V + kTStep - 1) / kTStep;
        int64_t n = (steps / per + 8) / 16 * 16;
        const int64_t least = steps < low ? steps : low;
        if (n < least) n = least;
        if (n > one && steps < two_from) n = one;
        if (n > most) n = most;
        return (int)(n < 1 ? 1 : n);
    }
};

ChunkRule chunk_rule(int nch, int tiles, bool bf16) {
    const bool single = tiles == 1;
    ChunkRule r;
    r.most = nch;
    r.per = bf16 && !single ? 6 : 3;
    r.low = single ? 48 : 16;
    r.one = (single || (bf16 && tiles == 2)) && nch >= 32 ? nch / 2 / 8 * 8 : nch;
    r.two_from = (int64_t)nch * (bf16 ? 18 : 11) / 4;
    return r;
}

template <int CM, bool G_BF16, bool X_BF16>
__global__ __launch_bounds__(kBlock, 2) void k_conv_wgrad_taps(const void *__restrict__ g, int C_out,
                                                               const void *__restrict__ x, int C_in, int T,
                                                               const int32_t *__restrict__ nbr,
                                                               const int32_t *__restrict__ counters, ChunkRule rule,
                                                               float *__restrict__ partial,
                                                               float *__restrict__ pbias) {
    constexpr int Z = CM == 3 ? 3 : 1;               // planes
    constexpr int PLANE = kTile * kTRow;
    __shared__ __attribute__((aligned(16))) char gs[Z * PLANE];
    __shared__ __attribute__((aligned(16))) char xs[kTaps * Z * PLANE];
    __shared__ float bred[kBlock / 16][kTile];

    // the workgroups that are used come first in the order of the grid, so
    // that they spread evenly over the CUs
    const int64_t V = counters[CNT_V];
    const int nch = rule.used(V), groups = gridDim.y;
    const int id = blockIdx.x + gridDim.x * (blockIdx.y + groups * blockIdx.z);
    if (id >= nch * groups * (int)gridDim.z) return;
    const int chunk = id % nch, tile = id / nch / groups;
    const int t0 = id / nch % groups * kTaps;
    const int tiles_i = (C_in + kTile - 1) / kTile;
    const int o0 = tile / tiles_i * kTile;
    const int i0 = tile % tiles_i * kTile;
    const int64_t lo = V * chunk / nch;
    const int64_t hi = V * (chunk + 1) / nch;
    const bool do_bias = pbias != nullptr && t0 == 0 && i0 == 0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int h = lane >> 5;
    const int ow = (wave >> 1) * 32;
    const int iw = (wave & 1) * 32;
    // Loader mapping: channel chunk c4 (4 channels), rows 2 rp and 2 rp + 1 of the step.
    const int c4 = (tid & 15) * 4;
    const int rp = tid >> 4;
    const bool g_in = o0 + c4 < C_out, x_in = i0 + c4 < C_in;

    f32x16_t acc[kTaps];
#pragma unroll
    for (int k = 0; k < kTaps; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] = 0.f;
    float bsum[4] = {0.f, 0.f, 0.f, 0.f};

    // the rows of two steps (slot: step mod 2), and the next step's indices
    Row4<G_BF16> ga[2][2];
    Row4<X_BF16> xa[2][kTaps][2];
    int32_t un[kTaps][2];
    auto load_index = [&](int64_t k0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t v = k0 + 2 * rp + j;
#pragma unroll
            for (int k = 0; k < kTaps; ++k) un[k][j] = v < hi && t0 + k < T ? nbr[v * T + t0 + k] : -1;
        }
    };
    auto load_step = [&](int64_t k0, int s) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t v = k0 + 2 * rp + j;
            if (v < hi && g_in) ga[s][j].load(g, v, C_out, o0 + c4);
            else ga[s][j].zero();
#pragma unroll
            for (int k = 0; k < kTaps; ++k)
                if (un[k][j] >= 0 && x_in) xa[s][k][j].load(x, un[k][j], C_in, i0 + c4);
                else xa[s][k][j].zero();
        }
    };
    // the bias sums the output gradient as stored (fp32 rows unrounded)
    auto add_bias = [&](int64_t k0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t v = k0 + 2 * rp + j;
            if (v >= hi || !g_in) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t at = v * C_out + o0 + c4 + e;
                bsum[e] += G_BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t *>(g)[at])
                                  : reinterpret_cast<const float *>(g)[at];
            }
        }
    };
    // registers -> LDS: word e of a thread = channel c4 + e of rows 2 rp, 2 rp + 1
    auto put = [&](char *base, const auto &r0, const auto &r1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            char *at = base + (c4 + e) * kTRow + 4 * rp;
            if constexpr (CM == 3) {
                uint32_t hh, mm, ll;
                split3(r0.f[e], r1.f[e], hh, mm, ll);
                *reinterpret_cast<uint32_t *>(at) = hh;
                *reinterpret_cast<uint32_t *>(at + PLANE) = mm;
                *reinterpret_cast<uint32_t *>(at + 2 * PLANE) = ll;
            } else {
                *reinterpret_cast<uint32_t *>(at) = r0.pair(r1, e);
            }
        }
    };
    auto step = [&](int64_t k0, int s) {
        if (do_bias) add_bias(k0);
        put(gs, ga[s][0], ga[s][1]);
#pragma unroll
        for (int k = 0; k < kTaps; ++k) put(xs + k * Z * PLANE, xa[s][k][0], xa[s][k][1]);
        __syncthreads();
        load_step(k0 + 2 * kTStep, s);
        load_index(k0 + 3 * kTStep);
#pragma unroll
        for (int q = 0; q < kTStep / 16; ++q) {
            const int at = (lane & 31) * kTRow + 32 * q + 16 * h;
            u32x4_t a[Z];
#pragma unroll
            for (int z = 0; z < Z; ++z) a[z] = *reinterpret_cast<const u32x4_a4_t *>(gs + z * PLANE + ow * kTRow + at);
#pragma unroll
            for (int k = 0; k < kTaps; ++k) {
                u32x4_t b[Z];
#pragma unroll
                for (int z = 0; z < Z; ++z)
                    b[z] = *reinterpret_cast<const u32x4_a4_t *>(xs + (k * Z + z) * PLANE + iw * kTRow + at);
                constexpr int NP = CM == 3 ? 6 : 1;
                constexpr int za[6] = {0, 2, 1, 0, 1, 0}, zb[6] = {2, 0, 1, 1, 0, 0};  // smallest first
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    acc[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8_t, a[CM == 3 ? za[p] : 0]),
                        __builtin_bit_cast(bf16x8_t, b[CM == 3 ? zb[p] : 0]), acc[k], 0, 0, 0);
            }
        }
        __syncthreads();
    };
    if (lo < hi) {
        load_index(lo);
        load_step(lo, 0);
        load_index(lo + kTStep);
        load_step(lo + kTStep, 1);
        load_index(lo + 2 * kTStep);
    }
    for (int64_t k0 = lo; k0 < hi; k0 += 2 * kTStep) {
        step(k0, 0);
        if (k0 + kTStep < hi) step(k0 + kTStep, 1);
    }

    // element r of acc: output channel 8 (r / 4) + 4 h + r % 4, input channel l % 32
    const int ic = i0 + iw + (lane & 31);
    auto oc_of = [&](int r) { return o0 + ow + 8 * (r >> 2) + 4 * h + (r & 3); };
    if constexpr (CM == 3) {
        // a sum that is not finite may come from a value too large for the
        // split, or not finite itself: this wavefront's sums once more, on
        // fp32 MFMA (32x32x2: lane l supplies row l / 32 of a pair) with the
        // operands straight from memory, kRedo pairs and their indices in
        // flight.  An absent neighbour is left out (0 times 0), not taken as
        // a zero row, whose product with an infinity would be NaN.  One
        // infinity, us: V = 10 200 64 -> 64 29 -> 38, 128 -> 128 44 -> 101,
        // V = 75 500 64 -> 157, 199 -> 559 (every row infinite: 170, 636)
        bool bad = false;
#pragma unroll
        for (int k = 0; k < kTaps; ++k)
#pragma unroll
            for (int r = 0; r < 16; ++r) bad |= !(fabsf(acc[k][r]) <= 3.402823466e38f);
        if (__ballot(bad) != 0ull) {
            constexpr int kRedo = 4;
            const int oc = o0 + ow + (lane & 31);
            int32_t u[kRedo][kTaps];
            auto indices = [&](int64_t v0) {
#pragma unroll
                for (int j = 0; j < kRedo; ++j)
#pragma unroll
                    for (int k = 0; k < kTaps; ++k) {
                        const int64_t v = v0 + 2 * j + h;
                        u[j][k] = v < hi && t0 + k < T ? nbr[v * T + t0 + k] : -1;
                    }
            };
#pragma unroll
            for (int k = 0; k < kTaps; ++k)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[k][r] = 0.f;
            indices(lo);
            for (int64_t v0 = lo; v0 < hi; v0 += 2 * kRedo) {
                float a[kRedo], b[kRedo][kTaps];
                bool on[kRedo][kTaps];
#pragma unroll
                for (int j = 0; j < kRedo; ++j) {
                    const int64_t v = v0 + 2 * j + h;
                    a[j] = v < hi && oc < C_out ? reinterpret_cast<const float *>(g)[v * C_out + oc] : 0.f;
#pragma unroll
                    for (int k = 0; k < kTaps; ++k) {
                        on[j][k] = u[j][k] >= 0;
                        b[j][k] = on[j][k] && ic < C_in
                                      ? reinterpret_cast<const float *>(x)[(int64_t)u[j][k] * C_in + ic]
                                      : 0.f;
                    }
                }
                indices(v0 + 2 * kRedo);
#pragma unroll
                for (int j = 0; j < kRedo; ++j)
#pragma unroll
                    for (int k = 0; k < kTaps; ++k)
                        acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(on[j][k] ? a[j] : 0.f, b[j][k], acc[k], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int k = 0; k < kTaps; ++k)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[k][r] *= kSplitBack;
        }
    }
    float *dst = partial + (int64_t)chunk * C_out * T * C_in;
#pragma unroll
    for (int k = 0; k < kTaps; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int oc = oc_of(r);
            if (oc < C_out && ic < C_in && t0 + k < T) dst[((int64_t)oc * T + t0 + k) * C_in + ic] = acc[k][r];
        }
    if (do_bias) {
        // threads tid and tid + 16 k (k = 0..15) share channel chunk c4
#pragma unroll
        for (int e = 0; e < 4; ++e) bred[rp][c4 + e] = bsum[e];
        __syncthreads();
        if (tid < kTile) {
            float sacc = 0.f;
            for (int q = 0; q < kBlock / 16; ++q) sacc += bred[q][tid];
            if (o0 + tid < C_out) pbias[(int64_t)chunk * C_out + o0 + tid] = sacc;
        }
    }
}

// out[j] = sum over the nch chunk partials part[c][j], in a fixed order:
// a workgroup owns 64 consecutive outputs; its four wavefronts sum the
// chunks c = g, g+4, g+8, ... (g = wavefront) with four loads in flight, and
// the four group sums are added in group order.
constexpr int kRedCols = 64;
__global__ __launch_bounds__(kBlock) void k_wgrad_reduce(const float *__restrict__ part,
                                                         const int32_t *__restrict__ counters, ChunkRule rule,
                                                         int64_t n, float *__restrict__ out) {
    __shared__ float red[kBlock / kRedCols][kRedCols];
    const int nch = counters ? rule.used(counters[CNT_V]) : rule.most;
    const int g = threadIdx.x / kRedCols;
    const int64_t j = (int64_t)blockIdx.x * kRedCols + (threadIdx.x % kRedCols);
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (j < n) {
        constexpr int G = kBlock / kRedCols;
        // (past the last chunk the group's first one is loaded, and not added)
        for (int c = g; c < nch; c += 4 * G) {
            const int c1 = c + G, c2 = c + 2 * G, c3 = c + 3 * G;
            const float x0 = part[(int64_t)c * n + j], x1 = part[(int64_t)(c1 < nch ? c1 : c) * n + j];
            const float x2 = part[(int64_t)(c2 < nch ? c2 : c) * n + j];
            const float x3 = part[(int64_t)(c3 < nch ? c3 : c) * n + j];
            s0 += x0;
            s1 += c1 < nch ? x1 : 0.f;
            s2 += c2 < nch ? x2 : 0.f;
            s3 += c3 < nch ? x3 : 0.f;
        }
    }
    red[g][threadIdx.x % kRedCols] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (g == 0 && j < n) {
        float t = 0.f;
        for (int q = 0; q < kBlock / kRedCols; ++q) t += red[q][threadIdx.x];
        out[j] = t;
    }
}

// W'[i][s][o] = W[o][flip(s)][i]; flip(0) = 0, flip(1+j) = d+2+j, flip(d+2+j) = 1+j.
template <typename E>
__global__ __launch_bounds__(kBlock) void k_flip_weights(const E *__restrict__ w, int C_out, int T, int C_in,
                                                         E *__restrict__ wt) {
    const int64_t n = (int64_t)C_out * T * C_in;
    const int half = (T - 1) / 2;  // d + 1
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x; q < n; q += stride) {
        // q indexes W' [C_in][T][C_out]
        const int o = (int)(q % C_out);
        const int s = (int)((q / C_out) % T);
        const int i = (int)(q / ((int64_t)C_out * T));
        const int fs = s == 0 ? 0 : (s <= half ? s + half : s - half);
        wt[q] = w[((int64_t)o * T + fs) * C_in + i];
    }
}

}  // namespace

// Whether the rows take loads of four channels, and whether k_conv_wgrad_taps
// takes the operands.
static bool wgrad_vec(const void *g, lattice_dtype g_dt, int C_out, const void *x, lattice_dtype x_dt, int C_in) {
    return C_out % 4 == 0 && C_in % 4 == 0 && (reinterpret_cast<uintptr_t>(g) & (g_dt == LATTICE_BF16 ? 7 : 15)) == 0 &&
           (reinterpret_cast<uintptr_t>(x) & (x_dt == LATTICE_BF16 ? 7 : 15)) == 0;
}
static bool wgrad_taps(const void *g, lattice_dtype g_dt, int C_out, const void *x, lattice_dtype x_dt, int C_in,
                       lattice_dtype dt) {
    return wgrad_vec(g, g_dt, C_out, x, x_dt, C_in) &&
           (dt == LATTICE_BF16 || (g_dt == LATTICE_F32 && x_dt == LATTICE_F32));
}

// Number of vertex chunks of the weight gradient, a multiple of 8 (the
// chunk's workgroups of every tap then share one XCD's L2) and no more than
// steps of 32 rows in the largest lattice.  One tap per workgroup: about
// kWgPerCu workgroups per CU over all taps and tiles.  kTaps per workgroup:
// about two per CU, as far as the partials stay within the allocation-free
// call's workspace (where the first count's do; else that count, so that
// the same shapes fit it).
int wgrad_chunks(const lattice *L, const void *g, lattice_dtype g_dt, int C_out, const void *x, lattice_dtype x_dt,
                 int C_in, lattice_dtype dt) {
    const int64_t tiles = (int64_t)((C_out + kTile - 1) / kTile) * ((C_in + kTile - 1) / kTile);
    const int64_t per = (kWgPerCu * (int64_t)L->cu_count + tiles * L->T - 1) / (tiles * L->T);
    int64_t nch = (per + 7) / 8 * 8;
    const int64_t n = (int64_t)C_out * L->T * C_in;
    const int64_t room = LATTICE_NOALLOC_WORKSPACE_BYTES - (n * 4 + 255) / 256 * 256;
    const int64_t fit = room / ((n + C_out) * 4) / 8 * 8;
    // rounded down: 528 workgroups over 512 places took a second round (fp32
    // 32 -> 32 on V = 278 788 246 us against 167 for 64 -> 64)
    int64_t want = 2 * (int64_t)L->cu_count / (tiles * ((L->T + kTaps - 1) / kTaps)) / 8 * 8;
    if (want > fit) want = fit;
    if (want < 8) want = 8;
    if (nch <= fit && wgrad_taps(g, g_dt, C_out, x, x_dt, C_in, dt)) nch = want;
    const int64_t steps = (L->max_vertices + kStep - 1) / kStep;
    if (nch > steps) nch = steps;
    if (nch < 1) nch = 1;
    if (nch > 1024) nch = 1024;
    return (int)nch;
}

hipError_t launch_conv_wgrad(lattice *L, const void *g, lattice_dtype g_dt, int C_out, const void *x,
                             lattice_dtype x_dt, int C_in, lattice_dtype dt, int nch, float *partial,
                             float *pbias, float *grad_w, float *grad_bias) {
    const bool gb = g_dt == LATTICE_BF16, xb = x_dt == LATTICE_BF16, rnd = dt == LATTICE_BF16;
    const bool vec = wgrad_vec(g, g_dt, C_out, x, x_dt, C_in);
    const dim3 grid((unsigned)nch, (unsigned)L->T,
                    (unsigned)(((C_out + kTile - 1) / kTile) * ((C_in + kTile - 1) / kTile)));
    const ChunkRule rule = chunk_rule(nch, (int)grid.z, rnd);
    const int32_t *used = nullptr;  // the counters, where the kernel leaves chunks out
    if (wgrad_taps(g, g_dt, C_out, x, x_dt, C_in, dt)) {
        used = L->counters;
        const dim3 grid3(grid.x, (unsigned)((L->T + kTaps - 1) / kTaps), grid.z);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid3, dim3(kBlock), 0, L->stream, g, C_out, x, C_in, L->T, L->nbr, L->counters,
                               rule, partial, grad_bias ? pbias : nullptr);
        };
        if (!rnd) go(k_conv_wgrad_taps<3, false, false>);
        else if (gb && xb) go(k_conv_wgrad_taps<1, true, true>);
        else if (gb) go(k_conv_wgrad_taps<1, true, false>);
        else if (xb) go(k_conv_wgrad_taps<1, false, true>);
        else go(k_conv_wgrad_taps<1, false, false>);
    } else {
#define WG(GB, XB, RN, VC)                                                                                      \
    hipLaunchKernelGGL((k_conv_wgrad<GB, XB, RN, VC>), grid, dim3(kBlock), 0, L->stream, g, C_out, x, C_in, L->T, \
                       L->nbr, L->counters, nch, partial, grad_bias ? pbias : nullptr)
#define WG_V(GB, XB) \
    if (vec)         \
        WG(GB, XB, false, true); \
    else             \
        WG(GB, XB, false, false)
        // bf16 products here have odd widths or unaligned rows, fp32 ones
        // those or bf16 rows
        if (gb) {
            if (xb && rnd) WG(true, true, true, false);
            else if (xb) { WG_V(true, true); }
            else if (rnd) WG(true, false, true, false);
            else { WG_V(true, false); }
        } else {
            if (xb && rnd) WG(false, true, true, false);
            else if (xb) { WG_V(false, true); }
            else if (rnd) WG(false, false, true, false);
            else WG(false, false, false, false);
        }
#undef WG_V
#undef WG
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (grad_w) {
        const int64_t n = (int64_t)C_out * L->T * C_in;
        hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((n + kRedCols - 1) / kRedCols)), dim3(kBlock), 0,
                           L->stream, partial, used, rule, n, grad_w);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (grad_bias) {
        hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((C_out + kRedCols - 1) / kRedCols)), dim3(kBlock), 0,
                           L->stream, pbias, used, rule, (int64_t)C_out, grad_bias);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_flip_weights(lattice *L, const void *w, bool bf16, int C_out, int C_in, void *wt) {
    const int64_t n = (int64_t)C_out * L->T * C_in;
    const unsigned grid = grid_for(n, kBlock, L->cu_count, 2);
    if (bf16)
        hipLaunchKernelGGL(k_flip_weights<uint16_t>, dim3(grid), dim3(kBlock), 0, L->stream,
                           reinterpret_cast<const uint16_t *>(w), C_out, L->T, C_in, reinterpret_cast<uint16_t *>(wt));
    else
        hipLaunchKernelGGL(k_flip_weights<float>, dim3(grid), dim3(kBlock), 0, L->stream,
                           reinterpret_cast<const float *>(w), C_out, L->T, C_in, reinterpret_cast<float *>(wt));
    return hipGetLastError();
}
