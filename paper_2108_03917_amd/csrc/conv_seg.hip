// 1-hop-ring lattice convolution for channel counts that the resident-weight
// kernels of conv.hip are not built for (e.g. 8 -> 16, 32, 48, 96, 100
// channels): Y[V x C_out] = Z[V x K] W^T over the flattened K = T C_in, row v
// of Z being the concatenation of the T neighbour rows of v.
//
// Both sides are walked in segments of SE consecutive channels that never
// cross a tap: a tap has ceil(C_in / SE) of them, and segment s of a row is
// the s-th of all its taps'.  K has no padding beyond that (C_in is a multiple
// of SE, or, for bf16 rows, of SE / 2: then the last segment of a tap loads
// the tap's last SE channels and keeps the upper half), and every load is one
// 16-byte access, the lanes of a row's chunk reading consecutive segments.
//
// A workgroup of four wavefronts owns a BM x BN output tile, BN the whole of
// C_out up to 128, so that a neighbour row is gathered once per tap.  Chunks
// of 128 LDS bytes per row (64 bf16 or 32 fp32 of K) go through a register
// ring of two chunks into two LDS buffers, one barrier a chunk.  Rows are
// padded to 144 bytes: 16 rows read 16 bytes each on 64 different banks.
// The product runs on MFMA 16x16 (16x16x32 bf16, 16x16x4 fp32) with the
// weights as the A operand, so that a lane ends up with four consecutive
// output channels of one row and stores them at once.
//
// fp32 products run on the bf16 matrix cores, 15 times as fast, as six
// products of three-term splits (see split3), which keep every bit of the
// values; their error against 64 bits is a little below fp32 MFMA's (64 -> 64
// 3e-7 against 4e-7, 128 -> 128 4e-7 against 5e-7: fewer roundings of the
// running sum).  A tile with a result that is not finite is computed once
// more on fp32 MFMA: with one infinity among the rows 96 -> 96 on V = 75 500 takes
// 119 -> 179 us, 128 -> 128 186 -> 274.
//
// What bounds it: bf16, the gathers and the weight rows through L2 (each tile
// re-reads W); the split, its own vector instructions (6.5 a value and stage)
// and LDS; fp32 MFMA, the matrix cores (90 of 154 TFLOP/s).  Against the
// element-wise kernel that took these shapes before (us, before -> now), 9
// taps: V = 278 788 bf16 32 -> 32 115 -> 30, 96 -> 96 546 -> 109, 100 -> 100
// 583 -> 159, fp32 8 -> 16 90 -> 24; V = 263 000 fp32 96 -> 96 1031 -> 297,
// 100 -> 100 1106 -> 374; V = 32 000 fp32 96 -> 96 118 -> 48.
#include <type_traits>

#include "internal.h"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef u32x4_t u32x4_a8_t __attribute__((aligned(8)));

// One segment from memory.  bf16 rows (and weights) of C_in mod 8 = 4 channels
// start on 8 bytes, so their 16-byte loads promise no more than that.
template <typename T, bool A8>
__device__ __forceinline__ T load_seg(const char *p) {
    if constexpr (A8) return *reinterpret_cast<const u32x4_a8_t *>(p);
    else return *reinterpret_cast<const T *>(p);
}

constexpr int kMaxTaps = LATTICE_TAPS(LATTICE_MAX_D);
constexpr int kThreads = 256;

// CM 0: fp32 rows and weights, fp32 MFMA; CM 3: the same on bf16 MFMA, see
// split3; CM 1: fp32 rows rounded to bf16
// while staging, bf16 weights; CM 2: bf16 rows and weights.  The four
// wavefronts are WM x (4 / WM), each TI x TJ tiles of 16 x 16.
template <int CM, int WM, int TI, int TJ>
struct Shape {
    static constexpr int WN = 4 / WM;
    static constexpr int BM = WM * TI * 16, BN = WN * TJ * 16;
    static constexpr int SE = CM == 2 ? 8 : 4;               // channels per segment
    static constexpr bool SPLIT = CM == 3;
    static constexpr int ESZ = CM == 0 || SPLIT ? 4 : 2;     // weight element (and staged element, unless split)
    static constexpr int SB = SE * ESZ;                      // LDS (and weight) bytes per segment
    static constexpr int XESZ = CM == 2 ? 2 : 4;             // stored input element: 16 bytes of input per segment
    static constexpr int SEGS = 128 / SB;                    // segments per row and chunk
    static constexpr int RPP = kThreads / SEGS;              // rows per pass
    static constexpr int AP = (BM + RPP - 1) / RPP, BP = (BN + RPP - 1) / RPP;
    static constexpr int AR = AP * RPP, BR = BP * RPP;       // LDS rows (whole passes)
    // One LDS row: 128 bytes and 16 of padding (16 rows read 16 bytes each on
    // 64 different banks), or three planes of 64 bytes without: four rows'
    // 8-byte writes then fill the 64 banks, and 16-byte chunk c of row r sits at
    // c ^ (r / 4 % 4), which spreads the reads of 16 rows the same way (padded
    // rows had 2-way conflicts on the writes, half of the LDS time)
    static constexpr int kRowBytes = SPLIT ? 3 * 64 : 128 + 16;
    // LDS buffers: the split's planes take one (two to four workgroups per CU
    // hide its second barrier), the others two
    static constexpr int BUFS = SPLIT ? 1 : 2;
    static constexpr int kLds = BUFS * (AR + BR) * kRowBytes;
    static constexpr int kNbr = AR * kMaxTaps;
};

struct Args {
    const void *in;
    int C_in;
    const void *wv;
    int C_out, T;
    const float *bias;
    void *out;
    int out_bf16, out_vec;
    const int32_t *nbr, *counters;
    const float *zero_row;
};

// The tiles of one workgroup, with Shape's LDS (redo_s: the split's only).
template <int CM, int WM, int TI, int TJ>
__device__ __forceinline__ void conv_tiles(const void *__restrict__ in, int C_in, const void *__restrict__ wv,
                                           int C_out, int T, const float *__restrict__ bias, void *__restrict__ out,
                                           int out_bf16, int out_vec, const int32_t *__restrict__ nbr, int64_t V,
                                           const float *__restrict__ zero_row, char *lds, int32_t *nbr_s,
                                           int *redo_s) {
    typedef Shape<CM, WM, TI, TJ> S;
    constexpr int WN = S::WN, BM = S::BM, BN = S::BN, SE = S::SE, ESZ = S::ESZ, SB = S::SB, XESZ = S::XESZ;
    constexpr int SEGS = S::SEGS, RPP = S::RPP, AP = S::AP, BP = S::BP, AR = S::AR, BR = S::BR;
    constexpr int kRowBytes = S::kRowBytes, BUFS = S::BUFS;
    constexpr bool SPLIT = S::SPLIT;
    constexpr int P = 2;                              // chunks in the register ring
    typedef u32x4_t xseg_t;
    typedef typename std::conditional<SB == 16, u32x4_t, u32x2_t>::type wseg_t;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int j16 = lane & 15, q4 = lane >> 4;
    const int seg = tid % SEGS, row0 = tid / SEGS;
    const int64_t n_mt = (V + BM - 1) / BM;
    const int n_nt = (C_out + BN - 1) / BN;
    const int spr = (C_in + SE - 1) / SE;             // segments per tap
    const bool half = C_in % SE != 0;                 // the last one of a tap is its upper half
    const int64_t K = (int64_t)T * C_in;
    const int NS = T * spr;                           // segments of a whole row
    const int NQ = (NS + SEGS - 1) / SEGS;

    for (int64_t tile = blockIdx.x; tile < n_mt * n_nt; tile += gridDim.x) {
        const int64_t row_base = (tile / n_nt) * BM;
        const int col_base = (int)(tile % n_nt) * BN;
        for (int i = tid; i < AR * T; i += kThreads) {
            const int64_t e = row_base * T + i;
            nbr_s[i] = (i < BM * T && e < V * T) ? nbr[e] : -1;
        }
        __syncthreads();

        f32x4_t acc[TI][TJ];
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        xseg_t areg[P][AP];
        wseg_t breg[P][BP];
        uint32_t mask[P];  // bit i: row pass i present; bit 15 + i: weight pass i inside; bit 31: half
        int lt = 0, lc = seg;  // this thread's next segment: tap, segment of the tap
        while (lc >= spr) {
            lc -= spr;
            ++lt;
        }
        // Branch-free loads of the next chunk into ring slot s: an absent
        // neighbour, a segment past K and a column past C_out read row 0 and
        // are zeroed when they go to LDS.  Past the last chunk the slot's
        // loads are those of row 0 and nobody uses them.
        auto load_chunk = [&](int s) {
            const bool in_k = lt < T;
            uint32_t mk = 0;
            const int t = in_k ? lt : 0;
            int c = in_k ? lc * SE : 0;  // first channel loaded
            if (CM == 2 && half && c + SE > C_in) {
                c = C_in - SE;
                mk = 1u << 31;
            }
#pragma unroll
            for (int i = 0; i < AP; ++i) {
                const int u = nbr_s[(row0 + i * RPP) * T + t];
                if (in_k && u >= 0) mk |= 1u << i;
                const int64_t row = u >= 0 ? u : 0;
                // (SPLIT reads zeros there instead: every select saved is an
                // issue slot, which is what it is short of)
                const char *at = reinterpret_cast<const char *>(in) + (row * C_in + c) * XESZ;
                if (SPLIT) at = in_k && u >= 0 ? at : reinterpret_cast<const char *>(zero_row);
                areg[s][i] = load_seg<xseg_t, CM == 2>(at);
            }
#pragma unroll
            for (int i = 0; i < BP; ++i) {
                const int n = col_base + row0 + i * RPP;
                const bool ok = in_k && n < C_out && row0 + i * RPP < BN;
                if (ok) mk |= 1u << (15 + i);
                breg[s][i] = load_seg<wseg_t, CM == 2>(reinterpret_cast<const char *>(wv) +
                                                      ((ok ? n : 0) * K + t * C_in + c) * ESZ);
            }
            mask[s] = mk;
            lc += SEGS;
            while (lc >= spr) {
                lc -= spr;
                ++lt;
            }
        };
        // one staged segment: at its place in the row, or split over the planes
        auto put = [&](char *row, wseg_t y) {
            if constexpr (SPLIT) {
                uint32_t h[2], m[2], l[2];
                split3(__uint_as_float(y[0]), __uint_as_float(y[1]), h[0], m[0], l[0]);
                split3(__uint_as_float(y[2]), __uint_as_float(y[3]), h[1], m[1], l[1]);
                // (rows a multiple of 32 apart: r / 4 % 4 is row0's for every pass)
                char *at = row + 16 * ((seg >> 1) ^ ((row0 >> 2) & 3)) + 8 * (seg & 1);
                *reinterpret_cast<u32x2_t *>(at) = u32x2_t{h[0], h[1]};
                *reinterpret_cast<u32x2_t *>(at + 64) = u32x2_t{m[0], m[1]};
                *reinterpret_cast<u32x2_t *>(at + 128) = u32x2_t{l[0], l[1]};
            } else {
                *reinterpret_cast<wseg_t *>(row + seg * SB) = y;
            }
        };
        auto store_chunk = [&](int s, int buf) {
            const bool hi = CM == 2 && (mask[s] >> 31);
            char *A = lds + buf * (AR + BR) * kRowBytes;
            char *B = A + AR * kRowBytes;
#pragma unroll
            for (int i = 0; i < AP; ++i) {
                const bool on = (mask[s] >> i) & 1u;
                wseg_t y;
                if constexpr (CM == 1) {
                    const xseg_t x = areg[s][i];
                    y[0] = pack_bf16(__uint_as_float(x[0]), __uint_as_float(x[1]));
                    y[1] = pack_bf16(__uint_as_float(x[2]), __uint_as_float(x[3]));
                } else {
                    y = areg[s][i];
                    if constexpr (CM == 2) y = hi ? u32x4_t{y[2], y[3], 0u, 0u} : y;
                }
#pragma unroll
                for (int k = 0; k < SB / 4; ++k) y[k] = on || SPLIT ? y[k] : 0u;
                put(A + (row0 + i * RPP) * kRowBytes, y);
            }
#pragma unroll
            for (int i = 0; i < BP; ++i) {
                const bool on = (mask[s] >> (15 + i)) & 1u;
                wseg_t y = breg[s][i];
                if constexpr (CM == 2) y = hi ? u32x4_t{y[2], y[3], 0u, 0u} : y;
#pragma unroll
                for (int k = 0; k < SB / 4; ++k) y[k] = on ? y[k] : 0u;
                put(B + (row0 + i * RPP) * kRowBytes, y);
            }
        };
        // lane quarter q holds bytes 16 q .. of each 64: the same K in A and B
        auto compute = [&](int buf) {
            const int qc = SPLIT ? q4 ^ ((j16 >> 2) & 3) : q4;  // (tiles start at multiples of 16 rows)
            const char *A = lds + buf * (AR + BR) * kRowBytes + (wm * TI * 16 + j16) * kRowBytes + 16 * qc;
            const char *B = lds + buf * (AR + BR) * kRowBytes + (AR + wn * TJ * 16 + j16) * kRowBytes + 16 * qc;
            if constexpr (SPLIT) {
                u32x4_t b[3][TJ];
#pragma unroll
                for (int z = 0; z < 3; ++z)
#pragma unroll
                    for (int j = 0; j < TJ; ++j)
                        b[z][j] = *reinterpret_cast<const u32x4_t *>(B + j * 16 * kRowBytes + 64 * z);
                // two row tiles at a time; smallest products first
                constexpr int za[6] = {0, 2, 1, 0, 1, 0}, zb[6] = {2, 0, 1, 1, 0, 0};
                constexpr int TU = TI < 2 ? TI : 2;
#pragma unroll
                for (int i0 = 0; i0 < TI; i0 += TU) {
                    u32x4_t a[3][TU];
#pragma unroll
                    for (int z = 0; z < 3; ++z)
#pragma unroll
                        for (int i = 0; i < TU; ++i)
                            a[z][i] = *reinterpret_cast<const u32x4_t *>(A + (i0 + i) * 16 * kRowBytes + 64 * z);
#pragma unroll
                    for (int z = 0; z < 6; ++z)
#pragma unroll
                        for (int i = 0; i < TU; ++i)
#pragma unroll
                            for (int j = 0; j < TJ; ++j)
                                acc[i0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(bf16x8_t, b[zb[z]][j]),
                                    __builtin_bit_cast(bf16x8_t, a[za[z]][i]), acc[i0 + i][j], 0, 0, 0);
                }
                return;
            }
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                u32x4_t a[TI], b[TJ];
#pragma unroll
                for (int i = 0; i < TI; ++i)
                    a[i] = *reinterpret_cast<const u32x4_t *>(A + i * 16 * kRowBytes + 64 * g);
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    b[j] = *reinterpret_cast<const u32x4_t *>(B + j * 16 * kRowBytes + 64 * g);
                if constexpr (CM == 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int i = 0; i < TI; ++i)
#pragma unroll
                            for (int j = 0; j < TJ; ++j)
                                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    __uint_as_float(b[j][c]), __uint_as_float(a[i][c]), acc[i][j], 0, 0, 0);
                } else {
#pragma unroll
                    for (int i = 0; i < TI; ++i)
#pragma unroll
                        for (int j = 0; j < TJ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, b[j]),
                                                                                __builtin_bit_cast(bf16x8_t, a[i]),
                                                                                acc[i][j], 0, 0, 0);
                }
            }
        };

        // ring slot s holds chunk s mod 2; with two LDS buffers, buffer s holds
        // it while it is multiplied
        load_chunk(0);
        load_chunk(1);
        if constexpr (BUFS == 1) {
            for (int q = 0; q < NQ; q += 2) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    if (q + s >= NQ) break;
                    store_chunk(s, 0);
                    __syncthreads();
                    load_chunk(s);
                    compute(0);
                    __syncthreads();
                }
            }
        } else {
            store_chunk(0, 0);
            __syncthreads();
            const int NQP = NQ / 2 * 2;
            for (int q = 0; q < NQP; q += 2) {
                load_chunk(0);
                compute(0);
                store_chunk(1, 1);
                __syncthreads();
                load_chunk(1);
                compute(1);
                store_chunk(0, 0);
                __syncthreads();
            }
            if (NQ & 1) {
                compute(0);
                __syncthreads();  // the LDS is rewritten by the next tile
            }
        }

        if constexpr (SPLIT) {
            // a result that is not finite may come from an input that is not,
            // or is too large for the split: the tile once more on fp32 MFMA,
            // the operands straight from memory, 16 channels of a tap at a
            // time (lane quarter q holds channels 4 q .. of them)
            if (tid == 0) *redo_s = 0;
            __syncthreads();
            bool bad = false;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) bad |= !(fabsf(acc[i][j][r]) <= 3.402823466e38f);
            if (bad) *redo_s = 1;
            __syncthreads();
            if (*redo_s) {
                const float *X = reinterpret_cast<const float *>(in), *W = reinterpret_cast<const float *>(wv);
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int t = 0; t < T; ++t) {
#pragma unroll 1
                    for (int c = 4 * q4; c < C_in + 4 * q4; c += 16) {
                        f32x4_t x4[TI], w4[TJ];
#pragma unroll
                        for (int i = 0; i < TI; ++i) {
                            const int u = nbr_s[((wm * TI + i) * 16 + j16) * T + t];
                            x4[i] = u >= 0 && c < C_in ? *reinterpret_cast<const f32x4_t *>(X + (int64_t)u * C_in + c)
                                                       : f32x4_t{0.f, 0.f, 0.f, 0.f};
                        }
#pragma unroll
                        for (int j = 0; j < TJ; ++j) {
                            const int n = col_base + (wn * TJ + j) * 16 + j16;
                            w4[j] = n < C_out && c < C_in ? *reinterpret_cast<const f32x4_t *>(W + n * K + t * C_in + c)
                                                          : f32x4_t{0.f, 0.f, 0.f, 0.f};
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int i = 0; i < TI; ++i)
#pragma unroll
                                for (int j = 0; j < TJ; ++j)
                                    acc[i][j] =
                                        __builtin_amdgcn_mfma_f32_16x16x4f32(w4[j][e], x4[i][e], acc[i][j], 0, 0, 0);
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[i][j][r] *= kSplitBack;
            }
            __syncthreads();  // nbr_s is rewritten by the next tile
        }

        // register r of lane (j16, q4): row j16, column 4 q4 + r of each tile
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const int64_t row = row_base + (wm * TI + i) * 16 + j16;
            if (row >= V) continue;
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int col = col_base + (wn * TJ + j) * 16 + 4 * q4;
                f32x4_t y = acc[i][j];
                if (bias) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[r] += col + r < C_out ? bias[col + r] : 0.f;
                }
                const int64_t at = row * C_out + col;
                if (out_vec) {  // C_out a multiple of 4, rows aligned for it
                    if (col >= C_out) continue;
                    if (out_bf16) {
                        u32x2_t pk;
                        pk[0] = bf16_bits(y[0]) | (bf16_bits(y[1]) << 16);
                        pk[1] = bf16_bits(y[2]) | (bf16_bits(y[3]) << 16);
                        *reinterpret_cast<u32x2_t *>(reinterpret_cast<uint16_t *>(out) + at) = pk;
                    } else {
                        *reinterpret_cast<f32x4_t *>(reinterpret_cast<float *>(out) + at) = y;
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (col + r >= C_out) continue;
                        if (out_bf16) reinterpret_cast<uint16_t *>(out)[at + r] = (uint16_t)bf16_bits(y[r]);
                        else reinterpret_cast<float *>(out)[at + r] = y[r];
                    }
                }
            }
        }
    }
}

template <int CM, int WM, int TI, int TJ>
__global__ __launch_bounds__(kThreads) void k_conv_seg(Args a) {
    typedef Shape<CM, WM, TI, TJ> S;
    __shared__ __attribute__((aligned(16))) char lds[S::kLds];
    __shared__ int32_t nbr_s[S::kNbr];
    conv_tiles<CM, WM, TI, TJ>(a.in, a.C_in, a.wv, a.C_out, a.T, a.bias, a.out, a.out_bf16, a.out_vec, a.nbr,
                               a.counters[CNT_V], a.zero_row, lds, nbr_s, nullptr);
}

// fp32 where the split may pay: up to small_v vertices, which the lattice's
// bound does not tell (a coarse level keeps its cloud's), fp32 MFMA in tiles of
// 32 rows (64 of narrow outputs), above the split's WM, TI, TJ.  V = 2 871 with
// a bound of 400 000, us, split alone | with this: 64 -> 64 21.0 | 13.4, 96 -> 96
// 52 | 22.6, 128 -> 128 79 | 22.6, 256 -> 256 151 | 61 (the kernels before both 16.7,
// 45, 28.7, 52).  (Register bounds: as many workgroups per CU as the split
// alone would have.)
template <int WM, int TI, int TJ, int SM, int SI, int SJ>
__global__ __launch_bounds__(kThreads, TI * TJ > 6 ? 2 : TI * TJ == 6 ? 3 : 4) void k_conv_seg_split(Args a,
                                                                                                    int small_v) {
    typedef Shape<3, WM, TI, TJ> S;
    typedef Shape<0, SM, SI, SJ> F;
    __shared__ __attribute__((aligned(16))) char lds[S::kLds > F::kLds ? S::kLds : F::kLds];
    __shared__ int32_t nbr_s[S::kNbr > F::kNbr ? S::kNbr : F::kNbr];
    __shared__ int redo_s;
    const int64_t V = a.counters[CNT_V];
    if (V <= small_v)
        conv_tiles<0, SM, SI, SJ>(a.in, a.C_in, a.wv, a.C_out, a.T, a.bias, a.out, a.out_bf16, a.out_vec, a.nbr, V,
                                  a.zero_row, lds, nbr_s, nullptr);
    else
        conv_tiles<3, WM, TI, TJ>(a.in, a.C_in, a.wv, a.C_out, a.T, a.bias, a.out, a.out_bf16, a.out_vec, a.nbr, V,
                                  a.zero_row, lds, nbr_s, &redo_s);
}

Args args(lattice *L, const void *in, int C_in, const void *w, int C_out, const float *bias, void *out, bool out_bf16,
          bool out_vec) {
    return Args{in,  C_in, w, C_out, L->T, bias, out, out_bf16 ? 1 : 0, out_vec ? 1 : 0, L->nbr, L->counters,
                reinterpret_cast<const float *>(L->zero_row)};
}

// Four workgroups per CU walk the tiles, or as many as there can be tiles.
unsigned grid_of(const lattice *L, int BM, int BN, int C_out) {
    const int64_t tiles = ((L->max_vertices + BM - 1) / BM) * ((C_out + BN - 1) / BN);
    int64_t grid = (int64_t)L->cu_count * 4;
    if (grid > tiles) grid = tiles;
    return (unsigned)(grid < 1 ? 1 : grid);
}

template <int CM, int WM, int TI, int TJ>
hipError_t go(lattice *L, const void *in, int C_in, const void *w, int C_out, const float *bias, void *out,
              bool out_bf16, bool out_vec) {
    typedef Shape<CM, WM, TI, TJ> S;
    hipLaunchKernelGGL((k_conv_seg<CM, WM, TI, TJ>), dim3(grid_of(L, S::BM, S::BN, C_out)), dim3(kThreads), 0,
                       L->stream, args(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec));
    return hipGetLastError();
}

template <int WM, int TI, int TJ, int SM, int SI, int SJ>
hipError_t go_split(lattice *L, const void *in, int C_in, const void *w, int C_out, const float *bias, void *out,
                    bool out_bf16, bool out_vec, int64_t small_v) {
    typedef Shape<0, SM, SI, SJ> F;
    hipLaunchKernelGGL((k_conv_seg_split<WM, TI, TJ, SM, SI, SJ>), dim3(grid_of(L, F::BM, F::BN, C_out)),
                       dim3(kThreads), 0, L->stream, args(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec),
                       (int)small_v);
    return hipGetLastError();
}

// The tile's width: of 16, 32, 48 (four wavefronts along the rows) and 64,
// 96, 128 (two by two) the one that costs least, a tile costing its columns
// and the gather of its rows, about as much as 64 columns.
int tile_width(int C_out) {
    static const int w[6] = {128, 96, 64, 48, 32, 16};
    int best = 128, cost = 1 << 30;
    for (int n : w) {
        const int c = (C_out + n - 1) / n * (n + 64);
        if (c < cost) {
            cost = c;
            best = n;
        }
    }
    return best;
}

template <int CM, int M4, int M2>
hipError_t by_width(lattice *L, const void *in, int C_in, const void *w, int C_out, const float *bias, void *out,
                    bool out_bf16, bool out_vec) {
    switch (tile_width(C_out)) {
        case 16: return go<CM, 4, M4, 1>(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec);
        case 32: return go<CM, 4, M4, 2>(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec);
        case 48: return go<CM, 4, M4, 3>(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec);
        case 64: return go<CM, 2, M2, 2>(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec);
        case 96: return go<CM, 2, M2, 3>(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec);
        default: return go<CM, 2, M2, 4>(L, in, C_in, w, C_out, bias, out, out_bf16, out_vec);
    }
}

}  // namespace

bool conv_seg_covers(lattice_dtype in_dt, int C_in, lattice_dtype dt) {
    if (dt == LATTICE_F32) return in_dt == LATTICE_F32 && C_in % 4 == 0;
    return C_in % 4 == 0 && (in_dt == LATTICE_F32 || C_in >= 8);
}

hipError_t launch_conv_seg(lattice *L, const void *in, lattice_dtype in_dt, int C_in, const void *w, int C_out,
                           lattice_dtype dt, const float *bias, void *out, lattice_dtype out_dt) {
    const bool ob = out_dt == LATTICE_BF16;
    const bool vec = C_out % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & (ob ? 7 : 15)) == 0;
    // Rows per tile (V is on the device: the lattice's bound stands for it; a
    // lattice far below its bound pays for it, bf16 96 -> 96 on V = 2 900 in tiles
    // of 32, 64 and 128 rows 10.8, 13.0 and 17.3).
    // Clouds whose bound gives fewer tiles of 64 rows than CUs take half
    // tiles (one part-segmentation object, V = 5 211, us: bf16 64 -> 96 8.7
    // against 7.8, fp32 96 -> 96 32.8 against 22.5); 96-wide tiles of large
    // lattices take 128 rows, which halves the weight reads (bf16 96 -> 96 on
    // V = 278 788: 131 against 109, on V = 143 537: 74 against 68, both with
    // bounds above 500 000; on V = 70 989 of 160 000 35 against 38).
    const bool small = L->max_vertices <= 64 * (int64_t)L->cu_count;
    if (dt == LATTICE_F32) {
        if (small) return by_width<0, 1, 1>(L, in, C_in, w, C_out, bias, out, ob, vec);
        const int width = tile_width(C_out);
        const bool large = L->max_vertices >= kConvLarge;
        // The split takes tiles at least 64 wide, on large lattices 32, and 128
        // rows there (which halves the weights' splitting) for all widths but
        // 64: narrower ones are bound by their gathers.  us, fp32 MFMA -> split:
        // 96 -> 96 on V = 31 500 / 98 600 / 263 000 58 -> 48, 177 -> 128, 505 -> 297,
        // 100 -> 100 82 -> 61, 262 -> 194, 644 -> 374, 32 -> 32 and 48 -> 48 on
        // V = 263 000 69 -> 56, 137 -> 120; 32 -> 32 on V = 71 000 21.9 -> 21.6, on
        // V = 32 000 12.0 -> 16.5, 8 -> 16 on V = 278 788 23.9 -> 38.7.  Below 64
        // vertices per CU it leaves CUs idle (V = 10 200 64 -> 64 18.9 -> 22.5,
        // 96 -> 96 36.8 -> 40.1), of narrow outputs below 256.
        const int64_t v64 = 64 * (int64_t)L->cu_count, v256 = 4 * v64;
        switch (width < 64 && !large ? 0 : width) {
            case 32: return go_split<4, 2, 2, 4, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec, v256);
            case 48: return go_split<4, 2, 3, 4, 1, 3>(L, in, C_in, w, C_out, bias, out, ob, vec, v256);
            case 64: return go_split<2, 2, 2, 2, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec, v64);
            case 96:
                return large ? go_split<2, 4, 3, 2, 1, 3>(L, in, C_in, w, C_out, bias, out, ob, vec, v64)
                             : go_split<2, 2, 3, 2, 1, 3>(L, in, C_in, w, C_out, bias, out, ob, vec, v64);
            case 128:
                return large ? go_split<2, 4, 4, 2, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec, v64)
                             : go_split<2, 2, 4, 2, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec, v64);
            default: return by_width<0, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec);
        }
    }
    if (in_dt == LATTICE_F32) {
        if (small) return by_width<1, 1, 1>(L, in, C_in, w, C_out, bias, out, ob, vec);
        return by_width<1, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec);
    }
    if (small) return by_width<2, 1, 1>(L, in, C_in, w, C_out, bias, out, ob, vec);
    if (tile_width(C_out) == 96 && L->max_vertices >= kConvLarge)
        return go<2, 2, 4, 3>(L, in, C_in, w, C_out, bias, out, ob, vec);
    return by_width<2, 1, 2>(L, in, C_in, w, C_out, bias, out, ob, vec);
}
