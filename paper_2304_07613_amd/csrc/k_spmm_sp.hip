// k_spmm_sp.hip -- Y = W_s X for weights whose aligned groups of 4 columns
// keep at most 2 (n = 1, or n = 2 with m % 4 == 0), whatever rows share a
// pattern: group layouts with any g and the paper's chunked layout alike, on
// gfx950's sparse matrix instructions v_smfmac_f32_16x16x64_f16.
//
// Two kernels.  k_sp_prepare / k_sp_prepare_chunked write the weight once per
// call as a stream of instruction operands ("weight stream") in scratch
// memory, and (binary32) the scale of every token of X beside it; k_spmm_sp
// multiplies.
//
// Binary32.  Every entry, scaled by a power of two (one per token of X and per
// row of W, in the chunked layout per workgroup of the preparation, up to 256
// rows: the largest finite magnitude goes to [2^14, 2^15)), is carried as
// two binary16 numbers, h = f16(v) and l = f16(2^11 (v - h)), and the product
// is summed in binary32 from h h (one accumulator) and h l + l h (another,
// scaled back by 2^-11 at the end).  Each rounding to nearest leaves at most
// 2^-11 of its number: h + 2^-11 l is within 2^-22 |v| of v, and l l, left
// out, below 2^-22 |w x|, both of either sign.  The binary32 families round
// once per kept column on the running sum; here the sum of h h is rounded once
// per 8 stored columns, so the error against 64 bits is smaller: 1.3e-7 to
// 2.6e-7 (2-norm, K = 768 to 3072) where the binary32 matrix instructions give
// 2.5e-7 to 7e-7 on the same inputs.  Three sparse binary16 products count half
// of K's columns each at 16 times the rate of v_mfma_f32_16x16x4f32.  (Three
// exact bfloat16 parts need no scales, but six products: 65 us and 2.9e-7
// against 50 us and 1.5e-7 at 3072 x 768 x 4096.)
//
// Entries below 2^-14 of the scaled range (2^-28 of the largest) are no longer
// within 2^-22 of themselves, but within 2^-36: an output whose kept columns
// miss the large entries would lose all of its bits.  So the preparation also
// finds the smallest magnitude that is not 0 of every token and row.  Where it
// is that far down (the range is "wide"), an output with kk kept columns
// differs by less than kk 2^-20 in scaled units on top of the roundings above
// (every product at most 2^15 2^-36 for either operand): at least kk in
// magnitude, that is within 2^-20 of itself; below, it is summed again.  With
// entries N(0, 1) a token of 768 columns in 10^5 is wide, and an output in 10^6
// of it below kk.  (Rows of the chunked layout share a scale because a packed
// row of a chunk holds blocks of many of its rows: the rows' own maxima would
// take 37 000 LDS atomics a workgroup of the preparation.)
//
// These outputs, and those that are not finite, are summed again from the
// packed weight in binary32 multiply-adds (sp_exact, sp_again), so that
// infinities and NaN in X reach the outputs whose kept columns select them --
// kept zeros among them -- and no others.
//
// Binary16.  One part, products exact in binary32, as the other binary16
// kernels (and the same recomputation for results that are not finite).
//
// Weight stream, for every tile of 16 rows and step of 64 columns: PARTS
// operands of 64 lanes x 16 bytes, then 64 position words of 4 bytes.  Lane l
// holds row l % 16 and columns 16 (l / 16) .. + 15: stored value 2 q + j is
// the j-th kept one of columns 4 q .. 4 q + 3, its offset in bits 4 q + 2 j;
// places without a kept column hold 0.
//
// X.  The other operand wants, per lane, 8 consecutive columns of one token
// side by side.  A lane loads 8 rows x 2 tokens of X, splits and packs them
// along the columns and writes 16-byte units to LDS, unit (column / 8, token)
// -- so the operand is two plain 16-byte LDS reads, X may have any alignment
// and any token count, and no transposing read is left.  X and Y move as
// vectors that are only element-aligned (the hardware takes unaligned global
// accesses): rows of an odd number of tokens cost the same instructions
// (binary16 3072 x 768 x 2047: 28 us with element-wise loads and stores).
// Eight waves (4 x 2) share a tile of 64 RT rows x 128 tokens, one workgroup
// per CU.  X goes through two LDS buffers: pass p + 1 is split and written
// between the products of pass p, while pass p + 2 is loaded.
#include "chunked.hpp"

namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h16 __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u8v __attribute__((ext_vector_type(8)));

constexpr int kSpTok = 128;            // tokens per workgroup
constexpr int kSpK = 64;               // columns per step
constexpr int kSpWaves = 8;            // 4 row x 2 token blocks of 16 RT rows x 64 tokens
constexpr int kSpThreads = 64 * kSpWaves;

template <typename T> constexpr int sp_parts() { return std::is_same<T, float>::value ? 2 : 1; }
__host__ __device__ constexpr int sp_tile_bytes(int parts) { return parts * 1024 + 256; }

// the two parts of two binary32 numbers times `scale` (a power of two), packed
// (first in the low half): the scaled number and 2^11 times its remainder are
// exact, each rounded once to binary16.  (Vector conversions, so that the
// remainders stay v_fma_mix_f32 + v_cvt_pk_f16_f32: v_fma_mixlo_f16 issues at
// half the rate.)
constexpr float kSpLow = 2048.f, kSpLowInv = 1.f / 2048.f;
struct SpPair {
    uint32_t h, l;
};
__device__ __forceinline__ SpPair sp_split(float a, float b, float scale) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    a *= scale;
    b *= scale;
    const h2 h = __builtin_convertvector(f2{a, b}, h2);
    const h2 l = __builtin_convertvector(f2{__builtin_fmaf((float)h[0], -kSpLow, a * kSpLow),
                                            __builtin_fmaf((float)h[1], -kSpLow, b * kSpLow)}, h2);
    return SpPair{__builtin_bit_cast(uint32_t, h), __builtin_bit_cast(uint32_t, l)};
}
// Largest and smallest magnitude (as bits) of a set of binary32 numbers, zeros,
// infinities and NaN left out (the latter come out of sp_split as such at any
// scale)
struct SpRange {
    uint32_t mx = 0, mn1 = ~0u;    // mn1: the smallest less 1
    __device__ __forceinline__ void take(uint32_t u) {
        u &= 0x7fffffffu;
        u = u < 0x7f800000u ? u : 0u;
        mx = max(mx, u);
        mn1 = min(mn1, u - 1u);
    }
    // exponent fields: the largest's plus 1 in the high half, 255 less the
    // smallest's in the low half (0: no such number)
    __device__ __forceinline__ uint32_t word() const {
        return mx == 0 ? 0u : ((mx >> 23) + 1u) << 16 | (255u - ((mn1 + 1u) >> 23));
    }
};
__device__ __forceinline__ uint32_t sp_join(uint32_t a, uint32_t b) {
    return max(a & ~0xffffu, b & ~0xffffu) | max(a & 0xffffu, b & 0xffffu);
}
// A set's scale: four times the exponent that brings its largest magnitude to
// [2^14, 2^15) (at most 2^126, so that the scale itself is a binary32 number),
// + 1 where its range is wide, or + 2 where it has no magnitudes.
constexpr int kSpWide = 1, kSpZero = 2;
__device__ __forceinline__ int sp_scale_code(uint32_t range) {
    if (range == 0) return kSpZero;
    const int e = min(14 + 127 - (int)((range >> 16) - 1u), 126);
    const int low = 255 - (int)(range & 0xffffu);         // the smallest's exponent field
    return 4 * e + ((low == 0 ? -149 : low - 127) + e < -14 ? kSpWide : 0);
}
__device__ __forceinline__ int sp_scale_exp(int code) { return code >> 2; }
// Scaled magnitude from which on an output of a token and row stands: kk kept
// columns, 0 where neither range is wide or all products are 0
__device__ __forceinline__ float sp_floor(int xcode, int wcode, float kk) {
    return ((xcode | wcode) & (kSpWide | kSpZero)) == kSpWide ? kk : 0.f;
}

// One lane's stored values (8, binary32 or binary16) and positions to the stream
template <typename T>
__device__ __forceinline__ void sp_store(char *tile, int lane, const T (&v)[8], uint32_t pos, float scale) {
    if constexpr (sp_parts<T>() == 2) {
        u4 h, l;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const SpPair p = sp_split(v[2 * k], v[2 * k + 1], scale);
            h[k] = p.h;
            l[k] = p.l;
        }
        reinterpret_cast<u4 *>(tile)[lane] = h;
        reinterpret_cast<u4 *>(tile + 1024)[lane] = l;
    } else {
        reinterpret_cast<h8 *>(tile)[lane] = h8{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
    }
    reinterpret_cast<uint32_t *>(tile + sp_parts<T>() * 1024)[lane] = pos;
}

// Range (SpRange::word) of `count` consecutive binary32 numbers, by a
// workgroup of TH threads; red: TH / 64 words of LDS
template <int TH>
__device__ __forceinline__ uint32_t sp_block_range(const float *p, int64_t count, uint32_t *red) {
    SpRange r;
    const int tid = threadIdx.x;
    // 16 bytes a load where the numbers allow, 4 loads in flight (past the
    // end: the last one again)
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0 && count % 4 == 0) {
        const u4 *v = reinterpret_cast<const u4 *>(p);
        const int64_t nv = count / 4;
        for (int64_t i = tid; i < nv; i += 4 * TH) {
            u4 u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = v[min(i + k * TH, nv - 1)];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) r.take(u[k][e]);
        }
    } else {
        for (int64_t i = tid; i < count; i += 8 * TH) {
            uint32_t u[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = __builtin_bit_cast(uint32_t, p[min(i + k * TH, count - 1)]);
#pragma unroll
            for (int k = 0; k < 8; ++k) r.take(u[k]);
        }
    }
    uint32_t w = r.word();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) w = sp_join(w, (uint32_t)__shfl_xor((int)w, o));
    if ((tid & 63) == 0) red[tid >> 6] = w;
    __syncthreads();
    w = 0;
#pragma unroll
    for (int k = 0; k < TH / 64; ++k) w = sp_join(w, red[k]);
    return w;
}

// Ranges of 64 tokens of X over kSpXRows rows, by a workgroup of TH threads:
// part `rb` of the tokens' ranges
constexpr int kSpXRows = 192;
template <int TH>
__device__ __forceinline__ void sp_token_range(const float *X, int64_t ldx, int K, int N, int t0, int rb,
                                               uint32_t *xrange, uint32_t *red) {
    const int tid = threadIdx.x, c = tid & 63, r0 = tid >> 6;
    constexpr int RG = TH / 64, IT = kSpXRows / RG;
    const float *xc = X + min(t0 + c, N - 1);
    uint32_t u[IT];
#pragma unroll
    for (int j = 0; j < IT; ++j)
        u[j] = __builtin_bit_cast(uint32_t, xc[(int64_t)min(rb * kSpXRows + r0 + j * RG, K - 1) * ldx]);
    SpRange r;
#pragma unroll
    for (int j = 0; j < IT; ++j) r.take(u[j]);
    red[tid] = r.word();
    __syncthreads();
    if (tid < 64 && t0 + tid < N) {
        uint32_t w = red[tid];
#pragma unroll
        for (int k = 1; k < RG; ++k) w = sp_join(w, red[k * 64 + tid]);
        xrange[(int64_t)rb * N + t0 + tid] = w;
    }
}
// the token's scale code from the parts
__device__ __forceinline__ int sp_token_code(const uint32_t *xrange, int parts, int N, int tok) {
    uint32_t w = 0;
    for (int p = 0; p < parts; p += 8) {
        uint32_t u[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) u[j] = xrange[(int64_t)min(p + j, parts - 1) * N + tok];
#pragma unroll
        for (int j = 0; j < 8; ++j) w = sp_join(w, u[j]);
    }
    return sp_scale_code(w);
}

// The packed weight as its owner holds it, for the outputs that are summed
// again from it
struct SpPacked {
    const void *values;
    const uint8_t *index;
    int n, m, g, C;   // C chunks (chunked layout: block columns) a row
    int S;            // rows of a chunk of the chunked layout, 0: group layout
};

// Scratch memory: the weight stream, (chunked layout) where every row's kept
// weights lie, the partial sums of a product whose columns are split over
// workgroups, and (binary32) the scale codes of rows and tokens and the
// partial ranges of the tokens
struct SpScratch {
    char *stream;
    uint16_t *origin;   // per 16-row tile, step and lane: its 16 / m blocks'
                        // position in the chunk (8 bits) and kept offsets (4 each)
    int *wcode;
    uint32_t *xrange;
    int xparts;
    int *xcode;
    float *part;     // splits x M x N, or NULL
    int splits;
};
inline int64_t sp_xparts(int64_t K) { return (K + kSpXRows - 1) / kSpXRows; }
inline int64_t sp_tiles(int64_t M) { return (M + 15) / 16; }
// (binary16: whole passes of two steps, the last one's columns past K empty)
inline int64_t sp_steps(int64_t K, int parts) {
    return parts == 2 ? (K + kSpK - 1) / kSpK : (K + 2 * kSpK - 1) / (2 * kSpK) * 2;
}
inline int64_t sp_scale_offset(int64_t M, int64_t K, int parts) {
    return sp_tiles(M) * sp_steps(K, parts) * sp_tile_bytes(parts);     // a multiple of 256
}
// Passes a workgroup makes, and workgroups the columns are split over.  A
// layer whose 64-row tiles leave half of the compute units idle and whose
// columns make many passes is split, 6 passes a workgroup or more; a second
// kernel adds the parts in order.  768 x 3072: binary32 at 16 tokens 53 -> 19
// us, binary16 30 -> 15; binary16 at 1000 tokens 36 -> 29.  At 768 columns
// (12 passes, 6 in binary16) the second kernel costs what the split saves.
inline int sp_passes(int64_t K, int parts) { return (int)(sp_steps(K, parts) / (3 - parts)); }
inline int sp_splits(int64_t M, int64_t K, int64_t N, int parts) {
    const int64_t wgs = (M + 63) / 64 * ((N + kSpTok - 1) / kSpTok), cus = device_cus();
    const int np = sp_passes(K, parts);
    if (2 * wgs > cus || np < 16) return 1;
    const int64_t s = std::min<int64_t>(std::min<int64_t>(cus / wgs, np / 6), 8);
    if (s < 2) return 1;
    const int per = (int)((np + s - 1) / s);
    return (np + per - 1) / per;     // none empty
}
// (chunk_m: m of the chunked layout, 0: group layout)
inline int64_t sp_origin_bytes(int64_t M, int64_t K, int parts, int chunk_m) {
    return chunk_m > 0 ? sp_tiles(M) * sp_steps(K, parts) * 64 * (16 / chunk_m) * 2 : 0;   // a multiple of 128
}
inline SpScratch sp_scratch(void *ws, int64_t M, int64_t K, int64_t N, int parts, int chunk_m) {
    char *p = static_cast<char *>(ws);
    SpScratch r = {};
    r.stream = p;
    p += sp_scale_offset(M, K, parts);
    r.origin = reinterpret_cast<uint16_t *>(p);
    p += sp_origin_bytes(M, K, parts, chunk_m);
    r.xparts = (int)sp_xparts(K);
    r.splits = sp_splits(M, K, N, parts);
    if (r.splits > 1) {
        r.part = reinterpret_cast<float *>(p);
        p += r.splits * M * N * 4;
    }
    r.wcode = reinterpret_cast<int *>(p);
    r.xcode = r.wcode + 16 * sp_tiles(M);
    r.xrange = reinterpret_cast<uint32_t *>(r.xcode + N);
    return r;
}

// Kept values of one 16-column range, gathered column by column
template <typename T> struct SpLane {
    T v[8];
    uint32_t pos = 0, filled = 0;
    __device__ __forceinline__ SpLane() {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (T)0;
    }
    // `col` in 0 .. 15, ascending over the calls
    __device__ __forceinline__ void put(int col, T w, bool ok) {
        const int q = col >> 2;
        const int e = 2 * q + ((filled >> q) & 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = ok && e == i ? w : v[i];
        if (ok) {
            pos |= (uint32_t)(col & 3) << (2 * e);
            filled |= 1u << q;
        }
    }
};

// MC: m when it is 4, 8 or 16 (a lane's 16 columns are whole chunks), else 0
template <typename T, int MC>
__device__ __forceinline__ void sp_gather(const T *__restrict__ values, const uint8_t *__restrict__ indices,
                                          int row, int k0, int M, int K, int n, int m, int g, int C,
                                          SpLane<T> &a) {
    if (row >= M || k0 >= K) return;
    const int64_t ldv = (int64_t)C * n;
    const T *vr = values + row * ldv;
    const uint8_t *ir = indices + (row / g) * ldv;
    if constexpr (MC > 0) {
        constexpr int CH = 16 / MC;      // whole chunks, at most 8 slots
        T w[2 * CH];
        int o[2 * CH];
        const int c0 = k0 / MC;
        typedef T TV __attribute__((ext_vector_type(2 * CH)));
        typedef uint8_t IV __attribute__((ext_vector_type(2 * CH)));
        const T *v0 = vr + 2 * c0;
        const uint8_t *i0 = ir + 2 * c0;
        if (n == 2 && c0 + CH <= C &&
            (reinterpret_cast<uintptr_t>(v0) & (sizeof(T) * 2 * CH > 16 ? 15 : sizeof(TV) - 1)) == 0 &&
            (reinterpret_cast<uintptr_t>(i0) & (2 * CH - 1)) == 0) {
            // two of every chunk, all of them there: whole vectors
            IV iv = *reinterpret_cast<const IV *>(i0);
            if constexpr (sizeof(TV) > 16) {
                typedef T HV __attribute__((ext_vector_type(CH)));
                const HV a0 = reinterpret_cast<const HV *>(v0)[0], a1 = reinterpret_cast<const HV *>(v0)[1];
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    w[k] = a0[k];
                    w[CH + k] = a1[k];
                }
            } else {
                const TV tv = *reinterpret_cast<const TV *>(v0);
#pragma unroll
                for (int k = 0; k < 2 * CH; ++k) w[k] = tv[k];
            }
#pragma unroll
            for (int k = 0; k < 2 * CH; ++k) o[k] = iv[k];
        } else {
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const bool ok = t < n && c0 + c < C;
                    const int64_t ks = ok ? (int64_t)(c0 + c) * n + t : 0;
                    w[2 * c + t] = vr[ks];
                    o[2 * c + t] = ir[ks];
                }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                a.put(min(c * MC + min(o[2 * c + t], MC - 1), 15), w[2 * c + t], t < n && c0 + c < C);
    } else {
        for (int c = k0 / m; c < C && c * m < k0 + 16; ++c)
            for (int t = 0; t < n; ++t) {
                const int64_t ks = (int64_t)c * n + t;
                const int col = c * m + min((int)ir[ks], m - 1) - k0;
                a.put(min(max(col, 0), 15), vr[ks], col >= 0 && col < 16);
            }
    }
}

// Binary16: one wave per (16-row tile, step).
template <int MC>
__global__ __launch_bounds__(kBlock) void k_sp_prepare_f16(const _Float16 *__restrict__ values,
                                                           const uint8_t *__restrict__ indices,
                                                           char *__restrict__ stream, int M, int K,
                                                           int n, int m, int g, int C, int nsteps,
                                                           int total) {
    const int lane = threadIdx.x & 63;
    const int id = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (id >= total) return;
    const int rt = id / nsteps, s = id - rt * nsteps;
    SpLane<_Float16> a;
    sp_gather<_Float16, MC>(values, indices, 16 * rt + (lane & 15), kSpK * s + 16 * (lane >> 4), M, K, n, m,
                            g, C, a);
    sp_store<_Float16>(stream + (int64_t)id * sp_tile_bytes(1), lane, a.v, a.pos, 1.f);
}

// Binary32: a workgroup per 16-row tile and 8 steps (the rows' scales from the
// ranges of their kept weights, two rows a wave, found again by each of the
// tile's workgroups; then a step per wave), and one per 64 tokens and 192 rows
// of X (part of the tokens' ranges).
constexpr int kSpPrep = 512;
template <int MC>
__global__ __launch_bounds__(kSpPrep) void k_sp_prepare(const float *__restrict__ values,
                                                        const uint8_t *__restrict__ indices,
                                                        const float *__restrict__ X, int64_t ldx,
                                                        SpScratch ws, int M, int K, int N, int n, int m,
                                                        int g, int C, int nsteps, int sgroups, int wblocks) {
    __shared__ uint32_t red[kSpPrep];
    const int lane = threadIdx.x & 63;
    if ((int)blockIdx.x >= wblocks) {
        const int i = blockIdx.x - wblocks;
        sp_token_range<kSpPrep>(X, ldx, K, N, 64 * (i / ws.xparts), i % ws.xparts, ws.xrange, red);
        return;
    }
    const int rt = blockIdx.x / sgroups, s = ((int)blockIdx.x - rt * sgroups) * (kSpPrep / 64) + (threadIdx.x >> 6);
    const int64_t ldv = (int64_t)C * n;
    SpLane<float> a;   // gathered while the range is found
    if (s < nsteps)
        sp_gather<float, MC>(values, indices, 16 * rt + (lane & 15), kSpK * s + 16 * (lane >> 4), M, K, n, m,
                             g, C, a);
    const int r0 = 2 * (threadIdx.x >> 6);
    SpRange range[2];
    const bool vec = (reinterpret_cast<uintptr_t>(values) & 15) == 0 && ldv % 4 == 0;
    const float *row[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) row[h] = values + min(16 * rt + r0 + h, M - 1) * ldv;
    // (past the end: the last one again)
    if (vec) {
        for (int64_t i = lane; i < ldv / 4; i += 128) {
            u4 u[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    u[h][k] = reinterpret_cast<const u4 *>(row[h])[min(i + 64 * k, ldv / 4 - 1)];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int k = 0; k < 8; ++k) range[h].take(u[h][k >> 2][k & 3]);
        }
    } else {
        for (int64_t i = lane; i < ldv; i += 256) {
            uint32_t u[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int k = 0; k < 4; ++k) u[h][k] = __builtin_bit_cast(uint32_t, row[h][min(i + 64 * k, ldv - 1)]);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int k = 0; k < 4; ++k) range[h].take(u[h][k]);
        }
    }
    uint32_t word[2] = {range[0].word(), range[1].word()};
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int h = 0; h < 2; ++h) word[h] = sp_join(word[h], (uint32_t)__shfl_xor((int)word[h], o));
    if (lane < 2) red[r0 + lane] = (uint32_t)sp_scale_code(lane == 0 ? word[0] : word[1]);
    __syncthreads();
    const int code = (int)red[lane & 15];        // (the same from each of the tile's workgroups)
    if (threadIdx.x < 16) ws.wcode[16 * rt + threadIdx.x] = code;
    if (s < nsteps)
        sp_store<float>(ws.stream + ((int64_t)rt * nsteps + s) * sp_tile_bytes(2), lane, a.v, a.pos,
                        __builtin_ldexpf(1.f, sp_scale_exp(code)));
}

constexpr int kSpcRows = 256;          // chunk rows per workgroup, at most (S <= 256)
constexpr int kSpcSteps = 2;           // steps per workgroup
constexpr int kSpcThreads = 512;

// the offsets of at most 8 patterns, n each, worked out on the host (the
// unranking divides 64-bit numbers: 2 us at the head of the kernel)
constexpr int kSpFew = 8;
struct SpPatterns {
    uint8_t off[kSpFew * 2];
};

// The chunked layout (m in {4, 8, 16}, n <= 2): a workgroup takes `cpw` chunks
// (whole 16-row tiles, at most 256 rows) of 2 steps' block columns, inverts
// their index in LDS and gathers every row's blocks.  Binary32: its rows share
// one scale, from the range of their kept weights (found again by each
// workgroup of the same chunks: they lie side by side in memory).  One
// workgroup per 64 tokens and 192 rows of X finds part of the tokens' ranges.
template <typename T>
__global__ __launch_bounds__(kSpcThreads) void k_sp_prepare_chunked(
    const T *__restrict__ values, const uint8_t *__restrict__ index, const T *__restrict__ X, int64_t ldx,
    SpScratch ws, SpPatterns few, int M, int M16, int K, int N, int n, int m, int g, int P, int S, int B,
    int cpw, int nsteps, int groups, int sblocks) {
    __shared__ uint8_t inv[kSpcSteps * 16 * kSpcRows];    // position of (block column, chunk row)
    __shared__ uint8_t pat[256 * 2];
    __shared__ uint32_t red[kSpcThreads];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= groups * sblocks) {
        const int i = (int)blockIdx.x - groups * sblocks;
        if constexpr (sp_parts<T>() == 2)
            sp_token_range<kSpcThreads>(X, ldx, K, N, 64 * (i / ws.xparts), i % ws.xparts, ws.xrange, red);
        return;
    }
    const int grp = blockIdx.x / sblocks, s0 = ((int)blockIdx.x - grp * sblocks) * kSpcSteps;
    const int r0 = grp * cpw * S;
    const int rows = min(cpw * S, M - r0);    // whole chunks
    const int bps = kSpK / m;                 // block columns of a step
    const int b0 = s0 * bps, ns = min(kSpcSteps, nsteps - s0);
    const int nb = min(ns * bps, B - b0);
    const int64_t ldv = (int64_t)B * n;
    if (P <= kSpFew) {
        if (tid < kSpFew * 2) pat[tid] = few.off[tid];
    } else {
        for (int p = tid; p < P; p += kSpcThreads) p_unrank(m, n, p, pat + p * n);
    }
    for (int i = tid; i < ns * bps * kSpcRows / 4; i += kSpcThreads) reinterpret_cast<uint32_t *>(inv)[i] = 0;
    float scale = 1.f;
    if constexpr (sp_parts<T>() == 2) {
        const int code =
            sp_scale_code(sp_block_range<kSpcThreads>(values + (int64_t)r0 * ldv, (int64_t)rows * ldv, red));
        scale = __builtin_ldexpf(1.f, sp_scale_exp(code));
        if (s0 == 0)
            for (int t = tid; t < (rows + 15) / 16 * 16; t += kSpcThreads) ws.wcode[r0 + t] = code;
    }
    __syncthreads();
    // stored row j's index bytes of the block columns, 4 at a time where its
    // rows are whole words
    const uint32_t ms = magic_u16(S);
    if (B % 4 == 0 && nb % 4 == 0 && b0 % 4 == 0 && (reinterpret_cast<uintptr_t>(index) & 3) == 0) {
        const int nw = nb >> 2;
        const uint32_t mw = magic_u16(nw);
        for (int i = tid; i < rows * nw; i += kSpcThreads) {
            const int j = (int)div_u16(i, mw, nw), w = 4 * (i - j * nw);
            const int ch = (int)div_u16(j, ms, S);
            const uint32_t v = *reinterpret_cast<const uint32_t *>(index + (int64_t)(r0 + j) * B + b0 + w);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                inv[(w + k) * kSpcRows + ch * S + min((int)((v >> (8 * k)) & 0xffu), S - 1)] = (uint8_t)(j - ch * S);
        }
    } else {
        const uint32_t mb = magic_u16(nb);
        for (int i = tid; i < rows * nb; i += kSpcThreads) {
            const int j = (int)div_u16(i, mb, nb), w = i - j * nb;
            const int ch = (int)div_u16(j, ms, S);
            const int r = min((int)index[(int64_t)(r0 + j) * B + b0 + w], S - 1);
            inv[w * kSpcRows + ch * S + r] = (uint8_t)(j - ch * S);
        }
    }
    __syncthreads();
    const int bpl = 16 / m;                   // blocks per lane
    // 4 column ranges of every row and step, rows fastest
    const uint32_t mr = magic_u16(rows), mg = magic_u16(g);
    for (int i = tid; i < rows * 4 * ns; i += kSpcThreads) {
        const int sq = (int)div_u16(i, mr, rows), rr = i - sq * rows;   // chunk row
        const int sl = sq >> 2, q = sq & 3;                             // step, 16-column range
        const int base = (int)div_u16(rr, ms, S) * S;
        // the row's 1 to 4 blocks: every load in flight together
        T w0[4], w1[4];
        int o0[4], o1[4];
        uint64_t from = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int w = min((4 * sl + q) * bpl + min(k, bpl - 1), nb - 1);
            const int j = inv[w * kSpcRows + rr];
            const T *v = values + (int64_t)(r0 + base + j) * ldv + (int64_t)(b0 + w) * n;
            const uint8_t *off = pat + div_u16(j, mg, g) * n;
            w0[k] = v[0];
            w1[k] = n == 2 ? v[1] : v[0];
            o0[k] = off[0];
            o1[k] = off[n - 1];
            from |= (uint64_t)(uint32_t)(j | o0[k] << 8 | o1[k] << 12) << (16 * k);
        }
        SpLane<T> a;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool in = k < bpl && (4 * sl + q) * bpl + k < nb;
            a.put(min(k * m + o0[k], 15), w0[k], in);
            a.put(min(k * m + o1[k], 15), w1[k], in && n == 2);
        }
        const int row = r0 + rr;
        const int64_t tile = (int64_t)(row >> 4) * nsteps + s0 + sl;
        sp_store<T>(ws.stream + tile * sp_tile_bytes(sp_parts<T>()), (row & 15) + 16 * q, a.v, a.pos, scale);
        uint16_t *org = ws.origin + (tile * 64 + (row & 15) + 16 * q) * bpl;
        if (bpl == 4) *reinterpret_cast<uint64_t *>(org) = from;
        else if (bpl == 2) *reinterpret_cast<uint32_t *>(org) = (uint32_t)from;
        else *org = (uint16_t)from;
    }
    // rows past M in the last tile
    if (r0 + rows == M)
        for (int i = tid; i < (M16 - M) * 4 * ns; i += kSpcThreads) {
            const int row = M + i / (4 * ns), sq = i % (4 * ns);
            const SpLane<T> a;
            sp_store<T>(ws.stream + ((int64_t)(row >> 4) * nsteps + s0 + (sq >> 2)) * sp_tile_bytes(sp_parts<T>()),
                        (row & 15) + 16 * (sq & 3), a.v, a.pos, 1.f);
        }
}

// ---------------------------------------------------------------- the product

// this wave's LDS operations are done, then the workgroup barrier; loads from
// global memory stay in flight
__device__ __forceinline__ void sp_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

// A pointer the same in every lane, in scalar registers: loads at it plus a
// lane's 32-bit offset then need no 64-bit vector arithmetic (the compiler
// otherwise folds the row's offset into the lane's: three vector instructions
// a load)
typedef __attribute__((address_space(1))) const char sp_global;
__device__ __forceinline__ sp_global *sp_uniform(const char *p) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return reinterpret_cast<sp_global *>(((uint64_t)hi << 32) | lo);
#else
    return (sp_global *)p;
#endif
}

// Kept slot s of a row of the packed weight: its value and column
template <typename T>
__device__ __forceinline__ T sp_slot(const SpPacked &pk, const uint16_t *origin, int row, int s, int nsteps,
                                     int &col) {
    const int ldv = pk.C * pk.n, two = pk.n == 2 ? 1 : 0;     // n is 1 or 2
    const T *values = static_cast<const T *>(pk.values);
    if (pk.S == 0) {
        col = (s >> two) * pk.m + pk.index[(int64_t)(row / pk.g) * ldv + s];
        return values[(int64_t)row * ldv + s];
    }
    // m is 4, 8 or 16: 16 / m blocks a lane of the stream
    const int b = s >> two, lb = pk.m == 4 ? 2 : pk.m == 8 ? 1 : 0, sq = b >> lb;    // sq: 16-column range
    const int64_t lane = ((int64_t)(row >> 4) * nsteps + (sq >> 2)) * 64 + (row & 15) + 16 * (sq & 3);
    const uint32_t e = origin[(lane << lb) + (b & ((1 << lb) - 1))];
    col = b * pk.m + (int)((e >> (8 + 4 * (s & two))) & 15u);
    return values[(int64_t)(row - row % pk.S + (int)(e & 255u)) * ldv + s];
}

// One output by a wave: lane l sums the kept slots l, l + 64, .. of the row, the
// lanes' sums are added as a tree (every lane gets the result).  U slots a lane
// in flight; a NaN ends it.
template <typename T, int U>
__device__ __forceinline__ float sp_exact(const SpPacked &pk, const uint16_t *origin, const T *X, int64_t ldx,
                                          int row, int tok, int K, int nsteps) {
    const int lane = threadIdx.x & 63, ldv = pk.C * pk.n;
    float acc = 0.f;
    for (int i = 0; i < ldv; i += 64 * U) {
        T w[U];
        int col[U];
#pragma unroll
        for (int j = 0; j < U; ++j)
            w[j] = sp_slot<T>(pk, origin, row, min(i + 64 * j + lane, ldv - 1), nsteps, col[j]);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const float f = fmaf((float)w[j], (float)X[min(col[j], K - 1) * ldx + tok], acc);
            acc = i + 64 * j + lane < ldv ? f : acc;
        }
        if (__any(isnan(acc))) return __builtin_nanf("");
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    return acc;
}

// One output a lane (the same row in most lanes: its slots are broadcasts and
// its entries of X whole runs), ascending columns
template <typename T>
__device__ __forceinline__ float sp_exact_lane(const SpPacked &pk, const uint16_t *origin, const T *X, int64_t ldx,
                                               int row, int tok, int K, int nsteps) {
    constexpr int U = 4;
    const int ldv = pk.C * pk.n;
    float acc = 0.f;
    for (int i = 0; i < ldv; i += U) {
        T w[U];
        int col[U];
#pragma unroll
        for (int j = 0; j < U; ++j) w[j] = sp_slot<T>(pk, origin, row, min(i + j, ldv - 1), nsteps, col[j]);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const float f = fmaf((float)w[j], (float)X[min(col[j], K - 1) * ldx + tok], acc);
            acc = i + j < ldv ? f : acc;
        }
        if (isnan(acc)) break;
    }
    return acc;
}

// The flagged outputs of a workgroup's 64 RT rows x 128 tokens (bit t % 32 of
// flag[row][t / 32]) summed again, by all of its waves.  Few of them: one a
// wave at a time.  Many: 128 columns of X at a time in LDS, lane = two tokens,
// 8 rows a wave; a lane fetches one of the row's kept slots and hands it to the
// others, ascending columns.  3072 x 768 x 4096, 2:4:1, 59 us with none: one
// token (1500 outputs) 131 us, every output 930 us.  A wave takes about 6.6 us
// an output, the whole tile 440 us: equal near 530.
constexpr int kSpAgainFew = 512;
template <typename T>
__device__ __forceinline__ void sp_again(const SpPacked &pk, const uint16_t *origin, const T *X, int64_t ldx,
                                         T *Y, int64_t ldy, const T *R, int64_t ldr, int M, int K, int N,
                                         int nsteps, int row0, int t0, int rows, int count,
                                         const uint32_t (*flag)[kSpTok / 32], T *win) {
    constexpr int KW = 128;
    static_assert(KW * kSpTok * sizeof(T) <= 2 * 2 * 8 * kSpTok * 16, "the window fits the staging buffers");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto put = [&](int row, int tok, float y) __attribute__((always_inline)) {
        T v = (T)y;
        if (R != nullptr) v = (T)((float)v + (float)R[(int64_t)row * ldr + tok]);
        Y[(int64_t)row * ldy + tok] = v;
    };
    if (count <= kSpAgainFew) {
        for (int r = wave; r < rows; r += kSpWaves)
            for (int q = 0; q < kSpTok / 32; ++q)
                for (uint32_t bits = __builtin_amdgcn_readfirstlane(flag[r][q]); bits != 0; bits &= bits - 1) {
                    const int tok = t0 + 32 * q + __builtin_ctz(bits);
                    const float y = sp_exact<T, 8>(pk, origin, X, ldx, row0 + r, tok, K, nsteps);
                    if (lane == 0) put(row0 + r, tok, y);
                }
        return;
    }
    const int ldv = pk.C * pk.n;
    for (int rb = 0; rb < rows; rb += 8 * kSpWaves) {
        float acc[8][2];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j][0] = acc[j][1] = 0.f;
        for (int k0 = 0; k0 < K; k0 += KW) {
            __syncthreads();
            const int c = threadIdx.x % kSpTok;
#pragma unroll 16
            for (int r = threadIdx.x / kSpTok; r < KW; r += kSpThreads / kSpTok)
                win[r * kSpTok + c] = X[(int64_t)min(k0 + r, K - 1) * ldx + min(t0 + c, N - 1)];
            __syncthreads();
            // at most 64 slots have their column in the window: n of m <= 1 of 2
            const int s = k0 / pk.m * pk.n + lane, last = min(ldv, (k0 + KW + pk.m - 1) / pk.m * pk.n);
            T w8[8];
            int col8[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)   // (rows past M: the last one again, not stored)
                w8[j] = sp_slot<T>(pk, origin, min(row0 + rb + 8 * wave + j, M - 1), min(s, ldv - 1), nsteps, col8[j]);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float w = (float)w8[j];
                const uint64_t in = __ballot(s < last && col8[j] >= k0 && col8[j] < k0 + KW);
                const int off = min(max(col8[j] - k0, 0), KW - 1) * kSpTok;
                const int q1 = in != 0 ? 64 - __builtin_clzll(in) : 0;
                auto slots = [&](int q, auto count) __attribute__((always_inline)) {
                    constexpr int Q = decltype(count)::value;
                    T x[Q][2];
#pragma unroll
                    for (int k = 0; k < Q; ++k) {
                        const T *p = win + __builtin_amdgcn_readlane(off, q + k) + 2 * lane;
                        x[k][0] = p[0];
                        x[k][1] = p[1];
                    }
#pragma unroll
                    for (int k = 0; k < Q; ++k) {
                        const float wq = __builtin_bit_cast(
                            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), q + k));
                        acc[j][0] = fmaf(wq, (float)x[k][0], acc[j][0]);
                        acc[j][1] = fmaf(wq, (float)x[k][1], acc[j][1]);
                    }
                };
                int q = in != 0 ? __builtin_ctzll(in) : 0;
                for (; q + 8 <= q1; q += 8) slots(q, std::integral_constant<int, 8>{});
                for (; q < q1; ++q) slots(q, std::integral_constant<int, 1>{});
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int r = rb + 8 * wave + j;
            const uint32_t bits = flag[r][lane >> 4] >> (2 * lane & 31);
            if (bits & 1u) put(row0 + r, t0 + 2 * lane, acc[j][0]);
            if (bits & 2u) put(row0 + r, t0 + 2 * lane + 1, acc[j][1]);
        }
    }
}

// RT 16-row tiles per wave; VEC: two tokens a load (N >= 2); SPLIT: the
// columns are split over gridDim.y workgroups, whose sums go to ws.part
template <typename T, int RT, bool VEC, bool SPLIT>
__global__ __launch_bounds__(kSpThreads) void k_spmm_sp(SpScratch ws, SpPacked pk,
                                                        const T *__restrict__ X, int64_t ldx,
                                                        T *__restrict__ Y, int64_t ldy, int M, int K,
                                                        const T *__restrict__ R, int64_t ldr, int N,
                                                        int nsteps, int tiles16, int row_blocks,
                                                        bool yvec) {
    constexpr int PARTS = sp_parts<T>(), TB = sp_tile_bytes(PARTS);
    constexpr int SUB = 2 / PARTS;                 // 64-column steps per pass of the pipeline
    constexpr int ES = (int)sizeof(T);
    constexpr int UNITS = 8 * kSpTok;              // 16-byte units per plane (8 column groups)
    constexpr int OPITCH = 64 * ES + 16;           // output rows in LDS
    constexpr int OTILE = 16 * OPITCH;             // one wave's 16 x 64 outputs
    static_assert(kSpWaves * OTILE <= 2 * 2 * UNITS * 16, "outputs fit the staging buffers");
    // two buffers of two planes: the parts of one step (binary32), two steps (binary16)
    __shared__ __attribute__((aligned(16))) char xs[2 * 2 * UNITS * 16];
    __shared__ int tcode[PARTS == 2 ? kSpTok : 1]; // the tokens' scale codes
    // outputs to be summed again: a bit each, and their number
    __shared__ uint32_t flag[SPLIT ? 1 : 64 * RT][kSpTok / 32];
    __shared__ int flagged;

    const char *const stream = ws.stream;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int rb = tile % row_blocks, tt0 = tile / row_blocks;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 3, wt = wave >> 2;
    const int t0 = tt0 * kSpTok;
    const int rt0 = rb * (4 * RT) + wr * RT;       // this wave's first 16-row tile
    // this workgroup's passes (host: whole passes, none empty)
    const int per = SPLIT ? (nsteps / SUB + (int)gridDim.y - 1) / (int)gridDim.y : 0;
    const int p0 = SPLIT ? (int)blockIdx.y * per : 0;
    const int npass = SPLIT ? min(nsteps / SUB, p0 + per) : nsteps / SUB;

    // ---- the weight stream, one pass ahead (two sets)
    struct AOps {
        h8 a[RT][2];                               // parts, or the two steps' operands
        int ix[RT][SUB];
    };
    AOps aops[2];
    const char *arow[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) arow[i] = stream + (int64_t)min(rt0 + i, tiles16 - 1) * nsteps * TB;
    const uint32_t alane = (uint32_t)lane * 16;
    auto load_a = [&](int p, AOps &o) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const char *tp = arow[i] + (int64_t)p * (SUB * TB);
#pragma unroll
            for (int k = 0; k < 2; ++k)
                o.a[i][k] = *reinterpret_cast<const h8 *>(tp + (SUB == 2 ? k * TB : k * 1024) + alane);
#pragma unroll
            for (int k = 0; k < SUB; ++k)
                o.ix[i][k] = *reinterpret_cast<const int *>(tp + k * TB + PARTS * 1024 + lane * 4);
        }
    };

    // ---- X, one to two passes ahead: wave w takes column group w of each
    // step, every lane 8 rows x 2 tokens
    constexpr int XR = 8 * SUB;
    typedef T X2 __attribute__((ext_vector_type(2)));
    typedef X2 X2u __attribute__((aligned(sizeof(T))));   // element-aligned
    X2 x[XR];
    int xt[2];                                      // this lane's tokens within the tile
    uint32_t xoff[2];                               // bytes
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        xt[j] = VEC ? 2 * lane + j : lane + 64 * j;
        xoff[j] = (uint32_t)min(t0 + xt[j], VEC ? N - 2 + j : N - 1) * ES;
    }
    // a pair that starts with the last token is loaded one token earlier, and
    // written with its two places exchanged
    if (VEC && t0 + xt[0] == N - 1) {
        xt[1] = xt[0];
        xt[0] ^= 1;
    }
    float xscale[2] = {1.f, 1.f};
    const uint32_t ldb = (uint32_t)(ldx * ES);      // host: ldx ES < 2^31
    auto load_x = [&](int p) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < SUB; ++q) {
            // row by row from a scalar pointer; past K the last row again
            // (zero weights)
            const int k = (p * SUB + q) * kSpK + 8 * wave;
            sp_global *xb = sp_uniform(reinterpret_cast<const char *>(X) + (uint64_t)(uint32_t)min(k, K - 1) * ldb);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                X2 &d = x[8 * q + r];
                if constexpr (VEC) {
                    d = *(__attribute__((address_space(1))) const X2u *)(xb + xoff[0]);
                } else {
#pragma unroll
                    for (int j = 0; j < 2; ++j) d[j] = *(__attribute__((address_space(1))) const T *)(xb + xoff[j]);
                }
                xb += k + r + 1 < K ? ldb : 0u;
            }
        }
    };
    u4 *const units = reinterpret_cast<u4 *>(xs);
    // token j of this lane's 2 into buffer `buf`
    auto write_x = [&](int buf, int j) __attribute__((always_inline)) {
        u4 *dst = units + buf * (2 * UNITS) + wave * kSpTok + xt[j];
        if constexpr (PARTS == 2) {
            u4 h, l;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const SpPair p = sp_split(x[2 * k][j], x[2 * k + 1][j], xscale[j]);
                h[k] = p.h;
                l[k] = p.l;
            }
            dst[0] = h;
            dst[UNITS] = l;
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                dst[q * UNITS] = __builtin_bit_cast(
                    u4, h8{x[8 * q][j], x[8 * q + 1][j], x[8 * q + 2][j], x[8 * q + 3][j], x[8 * q + 4][j],
                           x[8 * q + 5][j], x[8 * q + 6][j], x[8 * q + 7][j]});
        }
    };

    // ---- operands of a 16-token tile: columns 8 (lane / 16) .. + 7 and 32 more
    h16 b[2][2];                                    // [tile parity][plane]
    const u4 *const bsrc = units + (lane >> 4) * kSpTok + 64 * wt + (lane & 15);
    auto read_b = [&](int buf, int t, int p) __attribute__((always_inline)) {
        const u4 *src = bsrc + (buf * 2 + p) * UNITS + 16 * t;
        const u4 lo = src[0], hi = src[4 * kSpTok];
        b[t & 1][p] = __builtin_bit_cast(h16, u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
    };

    // acc: h h (binary16: the product); low: h l + l h, times 2^11
    v4f acc[RT][4], low[PARTS == 2 ? RT : 1][4];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc[i][t] = v4f{0.f, 0.f, 0.f, 0.f};
            if constexpr (PARTS == 2) low[i][t] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    // C[.][t] += plane `pa` of the weights times plane `pb` of X's tile t
    auto mul = [&](const AOps &o, auto &c, int t, int pa, int pb, int px) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
            c[i][t] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(o.a[i][pa], b[t & 1][pb], c[i][t], o.ix[i][px], 0, 0);
    };

    // pass p from buffer `buf` with operand set `buf`: X of pass p + 1 (in
    // registers) goes to the other buffer between the products and its
    // registers take pass p + 2, the weights of pass p + 1 are loaded
    auto pass = [&](int p, auto bc) __attribute__((always_inline)) {
        constexpr int buf = decltype(bc)::value;
        const AOps &o = aops[buf];
        sp_barrier();   // buffer `buf` is complete, the other one no longer read
        read_b(buf, 0, 0);
        read_b(buf, 0, 1);
        load_a(min(p + 1, npass - 1), aops[buf ^ 1]);
        if constexpr (PARTS == 2) {
            // two tiles at a time, so that the three products of one
            // accumulator lie 2 RT instructions apart
            read_b(buf, 1, 0);
            read_b(buf, 1, 1);
#pragma unroll
            for (int t = 0; t < 4; t += 2) {
                mul(o, low, t, 0, 1, 0);                 // h l
                mul(o, low, t + 1, 0, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t == 0) write_x(buf ^ 1, 0);
                mul(o, low, t, 1, 0, 0);                 // l h
                mul(o, low, t + 1, 1, 0, 0);
                mul(o, acc, t, 0, 0, 0);                 // h h
                mul(o, acc, t + 1, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t == 0) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        read_b(buf, 2, 1 - q);
                        read_b(buf, 3, 1 - q);
                    }
                    write_x(buf ^ 1, 1);
                    load_x(min(p + 2, npass - 1));
                }
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (t < 3) {
                    read_b(buf, t + 1, 0);
                    read_b(buf, t + 1, 1);
                }
                mul(o, acc, t, 0, 0, 0);
                mul(o, acc, t, 1, 1, SUB - 1);
                if (t < 2) write_x(buf ^ 1, t);
                if (t == 1) load_x(min(p + 2, npass - 1));
            }
            // the order of issue: the next tile's LDS reads, then its products
            // with the packing of X in between
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 2 * RT + RT * SUB, 0);
            static_for<4>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                if constexpr (t < 3) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
                static_for<2 * RT>([&](auto) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if constexpr (t < 2) __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                });
                if constexpr (t < 2) __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);
                if constexpr (t == 1) __builtin_amdgcn_sched_group_barrier(0x020, XR * (VEC ? 1 : 2), 0);
            });
        }
    };
    load_x(p0);
    load_a(p0, aops[0]);
    if constexpr (!SPLIT) {   // (a barrier of the loop comes before their use)
        for (int i = tid; i < 64 * RT * (kSpTok / 32); i += kSpThreads) (&flag[0][0])[i] = 0;
        if (tid == 0) flagged = 0;
    }
    if constexpr (PARTS == 2) {
        if (tid < kSpTok) {
            const int code = sp_token_code(ws.xrange, ws.xparts, N, min(t0 + tid, N - 1));
            tcode[tid] = code;
            if (SPLIT && rb == 0 && blockIdx.y == 0 && t0 + tid < N) ws.xcode[t0 + tid] = code;
        }
        sp_barrier();
#pragma unroll
        for (int j = 0; j < 2; ++j) xscale[j] = __builtin_ldexpf(1.f, sp_scale_exp(tcode[xt[j]]));
    }
    write_x(0, 0);
    write_x(0, 1);
    load_x(min(p0 + 1, npass - 1));
    for (int p = p0; p < npass; p += 2) {
        pass(p, std::integral_constant<int, 0>{});
        if (p + 1 < npass) pass(p + 1, std::integral_constant<int, 1>{});
    }

    // ---- outputs: register r of (i, t) is row 16 (rt0 + i) + 4 (lane / 16) +
    // r, token t0 + 64 wt + 16 t + lane % 16; through this wave's share of LDS
    // so that every store writes whole runs of a row
    if constexpr (SPLIT) {
        // a part of the sum, still scaled: k_sp_reduce adds them up
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * (rt0 + i) + 4 * (lane >> 4) + r, tok = t0 + 64 * wt + 16 * t + (lane & 15);
                    float y = acc[i][t][r];
                    if constexpr (PARTS == 2) y = fmaf(low[i][t][r], kSpLowInv, y);
                    if (row < M && tok < N) ws.part[((int64_t)blockIdx.y * M + row) * N + tok] = y;
                }
        return;
    }
    sp_barrier();
    char *const ob = xs + wave * OTILE;
    constexpr int EPL = 16 / ES;                    // elements per lane
    constexpr int LPR = 64 / EPL;                   // lanes per row
    constexpr int RPI = 64 / LPR;                   // rows per store instruction
    typedef T OV __attribute__((ext_vector_type(EPL)));
    typedef OV OVu __attribute__((aligned(sizeof(T))));   // element-aligned
    int xc[4] = {0, 0, 0, 0};
    if constexpr (PARTS == 2) {
#pragma unroll
        for (int t = 0; t < 4; ++t) xc[t] = tcode[64 * wt + 16 * t + (lane & 15)];
    }
    const float kk = (float)(pk.C * pk.n);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        uint64_t doubt = 0;   // lanes with an output that is not finite, or a wide range
        int wc[4] = {0, 0, 0, 0};
        if constexpr (PARTS == 2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) wc[r] = ws.wcode[16 * min(rt0 + i, tiles16 - 1) + 4 * (lane >> 4) + r];
            doubt = __ballot(((xc[0] | xc[1] | xc[2] | xc[3] | wc[0] | wc[1] | wc[2] | wc[3]) & kSpWide) != 0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float y = acc[i][t][r];
                if constexpr (PARTS == 2)
                    y = __builtin_ldexpf(fmaf(low[i][t][r], kSpLowInv, y),
                                         -(sp_scale_exp(wc[r]) + sp_scale_exp(xc[t])));
                doubt |= __ballot(!(fabsf(y) < __builtin_inff()));
                *reinterpret_cast<T *>(ob + (4 * (lane >> 4) + r) * OPITCH + (16 * t + (lane & 15)) * ES) = (T)y;
            }
        p_wave_sync();
        if (__builtin_expect(doubt != 0, 0)) {
            uint32_t again = 0;   // bit 4 t + r: this lane's output (t, r) does not stand
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float y = acc[i][t][r];
                    bool stands = true;
                    if constexpr (PARTS == 2) {
                        y = fmaf(low[i][t][r], kSpLowInv, y);
                        stands = fabsf(y) >= sp_floor(xc[t], wc[r], kk);
                        y = __builtin_ldexpf(y, -(sp_scale_exp(wc[r]) + sp_scale_exp(xc[t])));
                    }
                    const int row = 16 * (rt0 + i) + 4 * (lane >> 4) + r, tok = t0 + 64 * wt + 16 * t + (lane & 15);
                    stands = stands && fabsf(y) < __builtin_inff();
                    if (!stands && row < M && tok < N) again |= 1u << (4 * t + r);
                }
            if (again != 0) atomicAdd(&flagged, __popc(again));
            for (uint32_t bits = again; bits != 0; bits &= bits - 1) {
                const int at = __builtin_ctz(bits), c = 64 * wt + 16 * (at >> 2) + (lane & 15);
                atomicOr(&flag[16 * (wr * RT + i) + 4 * (lane >> 4) + (at & 3)][c >> 5], 1u << (c & 31));
            }
        }
#pragma unroll
        for (int r0 = 0; r0 < 16; r0 += RPI) {
            const int r = r0 + lane / LPR, c = (lane % LPR) * EPL;
            const int row = 16 * (rt0 + i) + r, tok = t0 + 64 * wt + c;
            OV v = *reinterpret_cast<const OV *>(ob + r * OPITCH + c * ES);
            if (row >= M || rt0 + i >= tiles16) continue;
            T *y = Y + (int64_t)row * ldy + tok;
            if (R != nullptr) {   // the sum in binary32 of the rounded product and R, rounded again
                const T *res = R + (int64_t)row * ldr + tok;
                OV rv = {};
                if (tok + EPL <= N) {
                    rv = *reinterpret_cast<const OVu *>(res);
                } else {
#pragma unroll
                    for (int e = 0; e < EPL; ++e)
                        if (tok + e < N) rv[e] = res[e];
                }
#pragma unroll
                for (int e = 0; e < EPL; ++e) v[e] = (T)((float)v[e] + (float)rv[e]);
            }
            if (tok + EPL <= N) {
                // whole aligned rows past the caches; unaligned runs share
                // lines with their neighbours, which the caches merge
                if (yvec) __builtin_nontemporal_store(v, reinterpret_cast<OV *>(y));
                else *reinterpret_cast<OVu *>(y) = v;
            } else {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (tok + e < N) y[e] = v[e];
            }
        }
        p_wave_sync();
    }
    sp_barrier();
    if (__builtin_expect(flagged != 0, 0)) {
        __threadfence();    // the stores above come before the ones here
        __syncthreads();
        sp_again<T>(pk, ws.origin, X, ldx, Y, ldy, R, ldr, M, K, N, nsteps, rb * (64 * RT), t0, 64 * RT,
                    flagged, flag, reinterpret_cast<T *>(xs));
    }
}

// The parts of a split product added in order, scaled back (or recomputed
// where not finite or below its floor), the residual added: one thread per output
template <typename T>
__global__ __launch_bounds__(kBlock) void k_sp_reduce(SpScratch ws, SpPacked pk, const T *__restrict__ X, int64_t ldx,
                                                      T *__restrict__ Y, int64_t ldy, int M, int K,
                                                      const T *__restrict__ R, int64_t ldr, int N,
                                                      int nsteps) {
    const int64_t mn = (int64_t)M * N, at = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = min(at, mn - 1);   // (lanes past the end stay for the wave's recomputations)
    const int row = (int)(i / N), tok = (int)(i - (int64_t)row * N);
    float u[8];   // splits <= 8: every load in flight
#pragma unroll
    for (int z = 0; z < 8; ++z) u[z] = ws.part[min(z, ws.splits - 1) * mn + i];
    float y = u[0];
#pragma unroll
    for (int z = 1; z < 8; ++z) y = z < ws.splits ? y + u[z] : y;
    bool stands = true;
    if constexpr (sp_parts<T>() == 2) {
        const int wc = ws.wcode[row], xc = ws.xcode[tok];
        stands = fabsf(y) >= sp_floor(xc, wc, (float)(pk.C * pk.n));
        y = __builtin_ldexpf(y, -(sp_scale_exp(wc) + sp_scale_exp(xc)));
    }
    const bool again = at < mn && !(stands && fabsf(y) < __builtin_inff());
    uint64_t todo = __ballot(again);
    if (__popcll(todo) > 8) {
        if (again) y = sp_exact_lane<T>(pk, ws.origin, X, ldx, row, tok, K, nsteps);
        todo = 0;
    }
    for (; todo != 0; todo &= todo - 1) {   // a wave an output
        const int of = __builtin_ctzll(todo);
        const float z = sp_exact<T, 4>(pk, ws.origin, X, ldx, __builtin_amdgcn_readlane(row, of),
                                       __builtin_amdgcn_readlane(tok, of), K, nsteps);
        y = (int)(threadIdx.x & 63) == of ? z : y;
    }
    if (at >= mn) return;
    T v = (T)y;
    if (R != nullptr) v = (T)((float)v + (float)R[(int64_t)row * ldr + tok]);
    Y[(int64_t)row * ldy + tok] = v;
}

// --------------------------------------------------------------- launchers

// Row tiles per wave (1 .. 3, binary16 .. 4): rounds of workgroups (one per
// CU) times the rows of one plus a fixed share for its X.
int sp_row_tiles(int64_t M, int64_t N, int most) {
    const int64_t cus = device_cus(), tt = (N + kSpTok - 1) / kSpTok;
    int best = 1;
    int64_t cost = -1;
    for (int rt = most; rt >= 1; --rt) {
        const int64_t wgs = (M + 64 * rt - 1) / (64 * rt) * tt;
        const int64_t c = (wgs + cus - 1) / cus * (64 * rt + 64);
        if (cost < 0 || c < cost) {
            cost = c;
            best = rt;
        }
    }
    return best;
}

struct SpOut {
    void *Y;
    int64_t ldy;
    const void *R;   // residual to add, or NULL
    int64_t ldr;
};

template <typename T, int RT>
void sp_launch(const SpScratch &ws, const SpPacked &pk, const void *X, int64_t ldx, int M, int K, int N, const SpOut &o,
               hipStream_t stream) {
    const int nsteps = (int)sp_steps(K, sp_parts<T>()), tiles16 = (int)sp_tiles(M);
    const int row_blocks = (tiles16 + 4 * RT - 1) / (4 * RT);
    const int tok_tiles = (N + kSpTok - 1) / kSpTok;
    const bool vec = N >= 2;
    constexpr int EPL = 16 / (int)sizeof(T);
    const bool yvec = aligned(o.Y, 16) && o.ldy % EPL == 0;
    const dim3 grid((unsigned)(row_blocks * tok_tiles), (unsigned)ws.splits), block(kSpThreads);
#define NMG_SP(VEC, SPLIT)                                                                         \
    hipLaunchKernelGGL((k_spmm_sp<T, RT, VEC, SPLIT>), grid, block, 0, stream, ws, pk, (const T *)X, ldx, \
                       (T *)o.Y, o.ldy, M, K, (const T *)o.R, o.ldr, N, nsteps, tiles16, row_blocks, yvec)
    if constexpr (RT == 1) {   // split products have one row tile a wave
        if (ws.splits > 1) {
            if (vec) NMG_SP(true, true);
            else NMG_SP(false, true);
        }
    }
    if (ws.splits <= 1) {
        if (vec) NMG_SP(true, false);
        else NMG_SP(false, false);
    }
#undef NMG_SP
    if (ws.splits > 1)
        hipLaunchKernelGGL((k_sp_reduce<T>), dim3((unsigned)(((int64_t)M * N + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, stream, ws, pk, (const T *)X, ldx, (T *)o.Y, o.ldy, M, K,
                           (const T *)o.R, o.ldr, N, nsteps);
}

template <typename T>
nmg_status sp_product(const SpScratch &ws, const SpPacked &pk, const void *X, int64_t ldx, int M, int K, int N,
                      const SpOut &o, hipStream_t stream) {
    switch (ws.splits > 1 ? 1 : sp_row_tiles(M, N, sp_parts<T>() == 2 ? 3 : 4)) {
        case 4:
            if constexpr (sp_parts<T>() == 1) sp_launch<T, 4>(ws, pk, X, ldx, M, K, N, o, stream);
            break;
        case 3: sp_launch<T, 3>(ws, pk, X, ldx, M, K, N, o, stream); break;
        case 2: sp_launch<T, 2>(ws, pk, X, ldx, M, K, N, o, stream); break;
        default: sp_launch<T, 1>(ws, pk, X, ldx, M, K, N, o, stream); break;
    }
    return launched();
}

// chunks per workgroup of k_sp_prepare_chunked: whole 16-row tiles, 64 rows or
// more, at most 256; 0 if there is no such number
int spc_chunks(int S) {
    int cpw = 1;
    while (cpw * S % 16 != 0) ++cpw;
    const int unit = cpw;
    while (cpw * S < 64) cpw += unit;
    return cpw * S <= kSpcRows ? cpw : 0;
}

}  // namespace

int64_t nmg_internal::sp_stream_bytes(nmg_dtype dtype, int64_t M, int64_t K, int64_t N, int chunk_m) {
    const bool f32 = dtype == NMG_F32;
    const int splits = sp_splits(M, K, N, f32 ? 2 : 1);
    return sp_scale_offset(M, K, f32 ? 2 : 1) + sp_origin_bytes(M, K, f32 ? 2 : 1, chunk_m) +
           (splits > 1 ? splits * M * N * 4 : 0) + (f32 ? 4 * (16 * sp_tiles(M) + N + sp_xparts(K) * N) : 0);
}

// 32-bit offsets along a row of X; every launch below 2^32 threads (HIP refuses
// more): both preparations and the product at one row tile a wave
bool nmg_internal::sp_args_supported(nmg_dtype dtype, int64_t M, int64_t K, int64_t ldx, int64_t N) {
    const int64_t es = (int64_t)elem_size(dtype), threads = (int64_t)1 << 32;
    const int64_t prep = sp_tiles(M) * ((K + 511) / 512) + (N + 63) / 64 * sp_xparts(K);
    return ldx * es < (int64_t)1 << 31 && sp_tiles(M) * sp_steps(K, 1) * 64 < threads &&
           prep * kSpPrep < threads && (M + 63) / 64 * ((N + kSpTok - 1) / kSpTok) * kSpThreads < threads;
}

// at most 2 kept of every aligned 4 columns: one of m >= 2 (a chunk ends
// between any two kept columns), or two of whole fours
bool nmg_internal::sp_layout_supported(const nmg_layout *L) {
    return (L->n == 1 && L->m >= 2) || (L->n == 2 && L->m % 4 == 0);
}

// AUTO's rule, over its choice without a workspace (us a call, that choice /
// this one, through the binding).  Its own cost is two launches, the weight
// stream (about 1.25 us per 10^6 entries of W, a third more for n = 1) and half
// of K's columns whatever is kept; theirs is launch plus kept columns, so it
// loses where few are kept, and on small products:
//  - Binary32 needs 64 kept columns a row: below that a chain of multiply-adds
//    rounds as rarely as this product does (1:20 of 768 columns: error 1.14e-7
//    against 1.22e-7; 1:10: 1.58e-7 against 1.45e-7).
//  - The expanded product and the staged vector kernel lose everywhere (2:4:1 at
//    3072 x 768: 79 / 23 at one token, 188 / 56 at 4096; 768 x 3072 262 / 55
//    and 286 / 72; 1:10:1 135 / 23 and 162 / 53; 1:32:1 at 4096 x 4096 by 1.5
//    to 9 times).
//  - The vector kernel: binary32 everywhere (1:128:1 at 1024 x 8192 3.4 times at
//    512 tokens, 170 / 178 at 4096), binary16 down to one column in 32; beyond,
//    a row's chain costs it 1 us a kept column (2 for groups of one row, whose
//    indices no other row shares), which has to make up for the stream: 1:64:1
//    30 / 13 at 768 x 768, 1:64:8 17 / 22 and 1:128:8 10 / 22 at 8192 x 1024,
//    31 / 31 at 4096 x 4096, 1:255:8 15 / 27 at 768 x 3072.
//  - mfma_scalar, binary32: its X goes through registers when the tokens do
//    not fill its tiles (1:4:8 at 1021 tokens 44 / 34; 1:8:8 30 / 28 at 1000,
//    21 / 31 at 17, 8192 x 1024); at half density it loses but for one tile of
//    64 tokens (2:4:8 31 / 25 at 512, 104 / 56 at 4096; 2:4:32 at 64 tokens of
//    8192 x 1024 25 / 28); at a quarter from about 10^9 kept products (1:4:8
//    19 / 27 at 512 tokens, 36 / 34 at 2048, 60 / 56 at 4096) where there are
//    tokens enough for the stream of many rows (8192 x 1024 1:4:8 59 / 64 at
//    1024, 190 / 182 at 4096, 1:4:32 89 / 98 at 2048); below a quarter it wins
//    (1:8:8 39 / 52 at 4096, 8192 x 1024 121 / 172).  Binary16 goes there only
//    for token counts off 8: 2:8:8 31 / 15 at one token, 55 / 26 at 1021, not
//    for a few columns (64 x 256, 1:8: 9 / 12).
//  - mfma_direct keeps its layouts (few kept columns, few rows or tokens),
//    where its partial sums also round less, but for half density from 2048
//    columns: 768 x 3072 2:4:4 40 / 19 at 16 tokens, 113 / 40 at 1021, 2:4:16
//    28 / 19 and 74 / 41, errors 1.9e-7 to 2.6e-7 / 1.3e-7 to 2.0e-7; with many
//    rows only for groups of 4 (4096 x 4096 2:4:4 91 / 70, 2:4:32 55 / 70).
//  - smfmac, whose columns are one chain: from 3 10^9 expanded products in 1000
//    tokens or more (2:4:1 30 / 20 at 2048, 11 / 16 at 512; 8192 x 1024 1:4:1
//    52 / 46 at 1000, 24 / 36 at 512), or 2048 columns (768 x 3072 50 / 15 at 16
//    tokens), with many rows at few tokens only (4096 x 4096 2:4:1 38 / 29 at 8,
//    43 / 47 at 512, 1:4:1 38 / 49 at 8).
//  - mfma_f16 at half density: 2:4 from 4 10^9 (2:4:8 13 / 16 at 512 tokens,
//    35 / 20 at 2048) or 2048 columns (768 x 3072 2:4:8 29 / 16 at 16 tokens,
//    2:4:32 25 / 26 at 1024); 1:2, whose stream takes longer, likewise but for
//    large groups (1:2:32 16 / 21 at 1000 tokens; 8192 x 1024 38 / 40) and many
//    rows at few tokens (4096 x 4096 1:2:8 37 / 38 at 8, 55 / 58 at 512).
//  The choice is the same for every epilogue, so that an epilogue gives the bits
//  of the product followed by it; GELU, which the binary16 kernels fold in and
//  this one takes as a pass of its own, still gains (3072 x 768 2:4:8 38 / 29
//  at 2048 tokens, 45 / 42 at 4096; 768 x 3072 34 / 19 at 64; at worst 1:2:32
//  768 x 3072 38 / 40 at 2048).
bool nmg_internal::sp_preferred(const nmg_layout *L, nmg_kernel family, int64_t N) {
    const int64_t M = L->M, K = L->K, n = L->n, m = L->m, g = L->g, slots = (int64_t)L->C * n;
    const double kept = (double)M * slots * (double)N, dense = (double)M * K * (double)N;
    const bool f32 = L->dtype == NMG_F32, half = 2 * n >= m, quarter = 4 * n >= m;
    if (f32 && slots < 64) return false;
    switch (family) {
        case NMG_KERNEL_MFMA_EXPAND:
        case NMG_KERNEL_VALU_STAGED: return true;
        case NMG_KERNEL_VALU:
            return f32 || m <= 32 * n ||
                   ((g == 1 || m <= 128 * n) && (double)slots * (g == 1 ? 2 : 1) >= 6 + 1.25e-6 * (double)M * K);
        case NMG_KERNEL_MFMA_DIRECT: return f32 && half && K >= 2048 && (M <= 2048 || g <= 4);
        case NMG_KERNEL_MFMA_SCALAR:
            if (!f32) return half || K >= 512;
            if (half) return N != 64 || g <= 8;
            if (N % 64 != 0) return quarter ? N >= 64 || g <= 8 : N >= 512;
            return quarter && kept >= 1e9 && (g <= 4 || M <= (g <= 8 ? 4 : 2) * N);
        case NMG_KERNEL_SMFMAC_F16:
            return (dense >= 3e9 && N >= 1000) ||
                   (K >= 2048 && (M <= 2048 || (N <= 256 && (n == 2 || m >= 8))));
        case NMG_KERNEL_MFMA_F16:
            if (!half) return false;
            if (n == 2) return dense >= 4e9 || (K >= 2048 && (g <= 8 || N <= 512));
            return (dense >= 4e9 && N >= 1000 && (g <= 8 || K >= 2048 || dense >= 1.2e10)) ||
                   (K >= 2048 && (M <= 2048 || g <= 4) && (g <= 8 || N <= 512));
        default: return false;
    }
}

bool nmg_internal::sp_p_preferred(const nmg_p_layout *L, int64_t N) {
    (void)N;
    return L->dtype == NMG_F16 || (int64_t)L->B * L->n >= 64;
}

nmg_status nmg_internal::spmm_sp(const SpmmArgs &a, void *ws_) {
    const nmg_layout *L = a.L;
    const SpOut out{a.Y, a.ldy, a.epi == NMG_EPILOGUE_ADD ? a.R : nullptr, a.ldr};
    const int parts = L->dtype == NMG_F32 ? 2 : 1;
    const int nsteps = (int)sp_steps(L->K, parts), tiles = (int)sp_tiles(L->M);
    const SpScratch ws = sp_scratch(ws_, L->M, L->K, a.N, parts, 0);
    const SpPacked pk{a.values, a.indices, L->n, L->m, L->g, L->C, 0};
    if (L->dtype == NMG_F32) {
        const int sgroups = (nsteps + kSpPrep / 64 - 1) / (kSpPrep / 64), wblocks = tiles * sgroups;
        const dim3 grid((unsigned)(wblocks + (a.N + 63) / 64 * ws.xparts));
#define NMG_SP_PREP(MC)                                                                             \
    hipLaunchKernelGGL((k_sp_prepare<MC>), grid, dim3(kSpPrep), 0, a.stream,                        \
        (const float *)a.values, a.indices, (const float *)a.X, a.ldx, ws, L->M, L->K, a.N, L->n, L->m,          \
        L->g, L->C, nsteps, sgroups, wblocks)
        switch (L->m) {
            case 4: NMG_SP_PREP(4); break;
            case 8: NMG_SP_PREP(8); break;
            case 16: NMG_SP_PREP(16); break;
            default: NMG_SP_PREP(0); break;
        }
#undef NMG_SP_PREP
        const nmg_status st = launched();
        if (st != NMG_OK) return st;
        return sp_product<float>(ws, pk, a.X, a.ldx, L->M, L->K, a.N, out, a.stream);
    }
    const int total = tiles * nsteps;
    const dim3 grid((unsigned)((total + kBlock / 64 - 1) / (kBlock / 64)));
#define NMG_SP_PREP(MC)                                                                             \
    hipLaunchKernelGGL((k_sp_prepare_f16<MC>), grid, dim3(kBlock), 0, a.stream,                     \
        (const _Float16 *)a.values, a.indices, ws.stream, L->M, L->K, L->n, L->m, L->g, L->C,              \
        nsteps, total)
    switch (L->m) {
        case 4: NMG_SP_PREP(4); break;
        case 8: NMG_SP_PREP(8); break;
        case 16: NMG_SP_PREP(16); break;
        default: NMG_SP_PREP(0); break;
    }
#undef NMG_SP_PREP
    const nmg_status st = launched();
    if (st != NMG_OK) return st;
    return sp_product<_Float16>(ws, pk, a.X, a.ldx, L->M, L->K, a.N, out, a.stream);
}

bool nmg_internal::sp_p_layout_supported(const nmg_p_layout *L) {
    return L->n <= 2 && (L->m == 4 || L->m == 8 || L->m == 16) && L->P <= 256 && L->S <= kSpcRows &&
           spc_chunks(L->S) > 0;
}

nmg_status nmg_internal::p_spmm_sp(const nmg_p_layout *L, const void *values, const uint8_t *index,
                                   const void *X, int64_t ldx, int N, void *Y, int64_t ldy, void *ws_,
                                   hipStream_t stream) {
    const bool f32 = L->dtype == NMG_F32;
    const int nsteps = (int)sp_steps(L->K, f32 ? 2 : 1), cpw = spc_chunks(L->S);
    const int groups = (L->M / L->S + cpw - 1) / cpw, sblocks = (nsteps + kSpcSteps - 1) / kSpcSteps;
    const SpScratch ws = sp_scratch(ws_, L->M, L->K, N, f32 ? 2 : 1, L->m);
    const SpPacked pk{values, index, L->n, L->m, L->g, L->B, L->S};
    const SpOut out{Y, ldy, nullptr, 0};
    SpPatterns few = {};
    for (int p = 0; L->P <= kSpFew && p < L->P; ++p) p_unrank(L->m, L->n, p, few.off + p * L->n);
    const int64_t blocks = (int64_t)groups * sblocks + (f32 ? (int64_t)(N + 63) / 64 * ws.xparts : 0);
    if (blocks > INT32_MAX) return NMG_ERR_PARAM;
#define NMG_SPC(T)                                                                                  \
    hipLaunchKernelGGL((k_sp_prepare_chunked<T>), dim3((unsigned)blocks), dim3(kSpcThreads),        \
        0, stream, (const T *)values, index, (const T *)X, ldx, ws, few, L->M, (L->M + 15) /        \
        16 * 16, L->K, N, L->n, L->m, L->g, L->P, L->S, L->B, cpw, nsteps, groups, sblocks)
    if (f32) NMG_SPC(float);
    else NMG_SPC(_Float16);
#undef NMG_SPC
    const nmg_status st = launched();
    if (st != NMG_OK) return st;
    if (f32) return sp_product<float>(ws, pk, X, ldx, L->M, L->K, N, out, stream);
    return sp_product<_Float16>(ws, pk, X, ldx, L->M, L->K, N, out, stream);
}
