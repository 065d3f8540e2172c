// k_chunked_pack.hip -- the converters of the paper's chunked layout (Section
// 5.2) for chunks with few patterns (P <= 8, m <= 8: 1:4, 2:4, 1:8, 3:4, ...):
// the greedy of the CPU converter and the swap search of the GPU converter,
// one wave per chunk (several small chunks share a wave), every lane holding
// whole rows -- their m weights and the magnitude every pattern keeps -- in
// registers.
//
//   greedy    The sequential greedy takes the largest eligible (row, pattern)
//             pair S times.  Between two moments at which a pattern fills up,
//             the set of open patterns does not change, so every free row
//             stands with its best open pattern and the greedy just walks the
//             rows by that one key: the rows above the first one that finds
//             its pattern full can be placed at once.  That is one phase; it
//             fills at least one pattern, so P phases do the work of S steps,
//             with the same pairs chosen.  A wave with one chunk finds the
//             phase's limit by bisecting the key range (ballots of "key >= t"
//             counted per pattern on the scalar unit); chunks that share a
//             wave count each row's rank within its pattern instead.
//   swaps     The gain of exchanging rows r (pattern a) and q (pattern e) is
//             D(r; a -> e) + D(q; e -> a), D(x; u -> v) = the magnitude row x
//             keeps under v less that under u.  For row r only the best q of
//             every pattern e matters, and which q that is does not depend on
//             r: one maximum per ordered pattern pair and round instead of a
//             scan of all rows by every row (S P + P^2 against S^2).  This
//             needs exact arithmetic: the magnitudes of a wave are taken as
//             whole multiples of the smallest one's unit in the last place,
//             in binary64 with the partner's row in the low 8 bits (larger
//             gain, then lower row), which is exact when the magnitudes lie
//             within a factor 2^19 of each other (zeros apart); binary64 sums
//             of the magnitudes themselves are then exact too, so that the
//             choices are those of the plain scan.  Waves outside that range
//             (or with infinities or NaN) run the plain scan.
//
// Bound by the latency of each wave's chain of instructions (3 waves a SIMD;
// the weights are 9 MB): 3072 x 768, binary32, 2:4, g = 32 has 3072 chunks of
// 192 rows; greedy 341 -> 42 us (2000 vector and 3100 scalar instructions a
// chunk), swap search 922 -> 69 us (75 with every table recomputed each round).
#include "chunked.hpp"

namespace {

constexpr int kCpWaves = 4;      // waves per workgroup
constexpr int kCpMaxP = 8;

struct PatMasks {
    uint8_t bits[kCpMaxP];       // columns of every pattern
};

typedef unsigned long long u64;

// How a chunk lies on a wave: S <= 64 packs 64 / S chunks, lane = chunk * S +
// row; larger ones take the wave alone, row = lane + 64 * i.
struct CpPlace {
    int chunks_per_wave, slots;
};
inline CpPlace cp_place(int S) { return S <= 64 ? CpPlace{64 / S, 1} : CpPlace{1, (S + 63) / 64}; }

__device__ __forceinline__ int cp_popc(u64 m) { return __popcll(m); }
// lanes below this one in mask m
__device__ __forceinline__ int cp_below(u64 m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// One row's weights (raw) and the magnitudes its patterns keep.
template <typename T, int MM, int PM, bool VEC> struct CpRow {
    using Bt = typename Bits<T>::type;
    Bt w[MM];
    __device__ __forceinline__ void load(const T *src, int m) {
        if constexpr (VEC) {     // m == MM, rows of whole 8- or 16-byte vectors
            typedef Bt BV __attribute__((ext_vector_type(MM)));
            const BV v = *reinterpret_cast<const BV *>(src);
#pragma unroll
            for (int k = 0; k < MM; ++k) w[k] = v[k];
        } else {
#pragma unroll
            for (int k = 0; k < MM; ++k) w[k] = k < m ? reinterpret_cast<const Bt *>(src)[k] : (Bt)0;
        }
    }
    // magnitude pattern p keeps: binary32, its offsets ascending, from +0
    __device__ __forceinline__ void scores(const PatMasks &pm, int P, float (&sc)[PM]) const {
#pragma unroll
        for (int p = 0; p < PM; ++p) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < MM; ++k) {
                const float a = fabsf((float)__builtin_bit_cast(T, w[k]));
                s = (pm.bits[p] >> k) & 1 ? s + a : s;
            }
            sc[p] = p < P ? s : 0.f;
        }
    }
    // the kept weights of the pattern with columns `bits`, to dst[0 .. n)
    __device__ __forceinline__ void store(uint32_t bits, int n, Bt *dst) const {
        int s = 0;
#pragma unroll
        for (int k = 0; k < MM; ++k)
            if ((bits >> k) & 1u) {
                if (s < n) dst[s] = w[k];
                ++s;
            }
    }
};

__device__ __forceinline__ uint32_t cp_mask_of(const PatMasks &pm, int p) {
    uint32_t b = pm.bits[0];
#pragma unroll
    for (int i = 1; i < kCpMaxP; ++i) b = p == i ? (uint32_t)pm.bits[i] : b;
    return b;
}

// Wave geometry of this lane
template <int SL> struct CpLane {
    int lane, c, r0;             // chunk within the wave; row of slot 0
    int64_t id;                  // chunk number over the grid
    bool on;                     // this lane holds rows of a chunk
    u64 own;                     // lanes of this lane's chunk
    __device__ __forceinline__ CpLane(int wave, int S, int64_t wave_id, int cpw, int64_t chunks) {
        (void)wave;
        lane = threadIdx.x & 63;
        if constexpr (SL == 1) {
            c = lane / S;
            r0 = lane - c * S;
        } else {
            c = 0;
            r0 = lane;
        }
        id = wave_id * cpw + c;
        on = c < cpw && id < chunks;
        if (SL == 1 && S < 64) own = on ? ((1ull << S) - 1) << (c * S) : 0ull;
        else own = ~0ull;
    }
};

// Every row's place (patterns in order, rows of a group ascending) and the
// packed chunk: pat[i] is the pattern of row r0 + 64 i.
template <typename T, int MM, int PM, int SL, bool VEC>
__device__ __forceinline__ void cp_write(const CpLane<SL> &ln, const CpRow<T, MM, PM, VEC> (&rows)[SL],
                                         const int (&pat)[SL], const bool (&live)[SL],
                                         const PatMasks &pm, T *values, uint8_t *index, int n, int g,
                                         int P, int S, int B, int64_t row0, int b) {
    using Bt = typename Bits<T>::type;
    int pos[SL];
#pragma unroll
    for (int i = 0; i < SL; ++i) pos[i] = pat[i] * g;
#pragma unroll
    for (int p = 0; p < PM; ++p) {
        if (p >= P) break;
        int before = 0;
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const u64 mk = __ballot(live[i] && pat[i] == p) & ln.own;
            if (pat[i] == p) pos[i] += before + cp_below(mk);
            before += cp_popc(mk);
        }
    }
    const int64_t ldv = (int64_t)B * n;
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        if (!live[i]) continue;
        const int64_t row = row0 + min(pos[i], S - 1);
        index[row * B + b] = (uint8_t)(ln.r0 + 64 * i);
        rows[i].store(cp_mask_of(pm, pat[i]), n, reinterpret_cast<Bt *>(values) + row * ldv + (int64_t)b * n);
    }
}

// maximum / minimum of a 32-bit key over the wave (in every lane): lane
// exchanges inside rows of 16 by DPP, then gfx950's row and half-wave swaps --
// an LDS shuffle a step would put 12 LDS round trips into every phase
template <bool MAX> __device__ __forceinline__ uint32_t cp_pick(uint32_t a, uint32_t b) {
    return MAX ? max(a, b) : min(a, b);
}
template <bool MAX> __device__ __forceinline__ uint32_t cp_wave_pick(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    v = cp_pick<MAX>(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, false));   // ^ 1
    v = cp_pick<MAX>(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, false));   // ^ 2
    v = cp_pick<MAX>(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xf, 0xf, false));  // 8 mirrored
    v = cp_pick<MAX>(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xf, 0xf, false));  // 16 mirrored
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = cp_pick<MAX>(r[0], r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return cp_pick<MAX>(h[0], h[1]);
#else
    return v;
#endif
}
__device__ __forceinline__ uint32_t cp_wave_max(uint32_t v) { return cp_wave_pick<true>(v); }
__device__ __forceinline__ uint32_t cp_wave_min(uint32_t v) { return cp_wave_pick<false>(v); }

// SL rows a lane; PACKED: several chunks on the wave (SL = 1)
template <typename T, int MM, int PM, int SL, bool PACKED, bool VEC>
__global__ __launch_bounds__(64 * kCpWaves) void k_p_greedy(const T *__restrict__ W, int64_t ldw,
                                                            T *__restrict__ values,
                                                            uint8_t *__restrict__ index, PatMasks pm,
                                                            int n, int m, int g, int P, int S, int B,
                                                            int cpw, int64_t chunks) {
    static_assert(!PACKED || SL == 1, "packed chunks hold one row a lane");
    __shared__ u64 keys_all[PACKED ? kCpWaves : 1][PACKED ? 64 : 1];
    __shared__ u64 limit_all[PACKED ? kCpWaves : 1][PACKED ? 64 : 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t wave_id = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * kCpWaves + wave;
    if (wave_id * cpw >= chunks) return;  // whole waves; no workgroup barrier follows
    const CpLane<SL> ln(wave, S, wave_id, cpw, chunks);
    const int64_t cid = min(ln.id, chunks - 1);
    const int64_t row0 = cid / B * S;
    const int b = (int)(cid % B);

    CpRow<T, MM, PM, VEC> rows[SL];
    uint32_t key[SL][PM];
    bool live[SL];
    int pat[SL];
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int r = ln.r0 + 64 * i;
        live[i] = ln.on && r < S;
        rows[i].load(W + (row0 + min(r, S - 1)) * ldw + (int64_t)b * m, m);
    }
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        float sc[PM];
        rows[i].scores(pm, P, sc);
#pragma unroll
        for (int p = 0; p < PM; ++p)   // NaN above every number
            key[i][p] = isnan(sc[p]) ? 0x7fc00000u : __builtin_bit_cast(uint32_t, sc[p]);
        pat[i] = -1;
    }

    if constexpr (PACKED) {
        // ---- several chunks: ranks within the pattern, counted through LDS
        u64 *keys = keys_all[wave], *limit = limit_all[wave];
        const int base = ln.c * S;
        int room[PM];
#pragma unroll
        for (int p = 0; p < PM; ++p) room[p] = p < P ? g : 0;
        bool free_ = live[0];
        for (int phase = 0; phase < P; ++phase) {
            if (!__any(free_)) break;
            uint32_t kb = 0;
            int bp = -1, rm = 0;
#pragma unroll
            for (int p = 0; p < PM; ++p)
                if (room[p] > 0 && (bp < 0 || key[0][p] > kb)) {
                    kb = key[0][p];
                    bp = p;
                    rm = room[p];
                }
            const bool act = free_ && bp >= 0;
            // larger magnitude, then lower pattern, then lower row (never 0)
            const u64 mine = act ? ((u64)kb << 32) | (1u << 16) | (uint32_t)((255 - bp) << 8) |
                                       (uint32_t)(255 - ln.r0)
                                 : 0ull;
            keys[ln.lane] = mine;
            limit[ln.lane] = 0ull;
            p_wave_sync();
            int rank = 0;
            if (act)
                for (int j = 0; j < S; ++j) {
                    const u64 o = keys[base + j];
                    rank += (o > mine && (((uint32_t)o ^ (uint32_t)mine) & 0xff00u) == 0u) ? 1 : 0;
                }
            // the largest key that finds its pattern full ends the phase
            if (act && rank >= rm) atomicMax(&limit[base], mine);
            p_wave_sync();
            const bool take = act && mine > limit[base];
#pragma unroll
            for (int p = 0; p < PM; ++p)
                room[p] -= cp_popc(__ballot(take && bp == p) & ln.own);
            if (take) {
                pat[0] = bp;
                free_ = false;
            }
            p_wave_sync();   // keys and limits are read before they are rewritten
        }
    } else {
        // ---- one chunk: the phase's limit by bisection, counts on the scalar unit
        int room[PM];
#pragma unroll
        for (int p = 0; p < PM; ++p) room[p] = p < P ? g : 0;
        for (int phase = 0; phase < P; ++phase) {
            uint32_t kb[SL];
            int bp[SL];
            u64 mk[PM][SL];
            int cnt[PM];
            uint32_t over = 0;   // patterns more rows ask for than have room
            uint32_t hi_k = 0, lo_k = 0xffffffffu;
            bool any = false;
#pragma unroll
            for (int i = 0; i < SL; ++i) {
                kb[i] = 0;
                bp[i] = -1;
#pragma unroll
                for (int p = 0; p < PM; ++p)
                    if (room[p] > 0 && (bp[i] < 0 || key[i][p] > kb[i])) {
                        kb[i] = key[i][p];
                        bp[i] = p;
                    }
                if (!live[i] || pat[i] >= 0) bp[i] = -1;
                if (bp[i] >= 0) {
                    hi_k = max(hi_k, kb[i]);
                    lo_k = min(lo_k, kb[i]);
                    any = true;
                }
            }
            if (!__any(any)) break;
#pragma unroll
            for (int p = 0; p < PM; ++p) {
                cnt[p] = 0;
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    mk[p][i] = __ballot(bp[i] == p);
                    cnt[p] += cp_popc(mk[p][i]);
                }
                if (cnt[p] > room[p]) over |= 1u << p;
            }
            // smallest t at which no pattern's rows with key >= t exceed its room
            uint32_t hi = 0;
            bool tie = false;
            if (over != 0) {
                uint32_t lo = __builtin_amdgcn_readfirstlane(cp_wave_min(lo_k));  // exceeds
                hi = __builtin_amdgcn_readfirstlane(cp_wave_max(hi_k)) + 1;       // no rows
                tie = true;
                while (hi - lo > 1) {
                    const uint32_t t = lo + (hi - lo) / 2;
                    u64 ge[SL];
#pragma unroll
                    for (int i = 0; i < SL; ++i) ge[i] = __ballot(kb[i] >= t);
                    bool exceed = false, full = false;
#pragma unroll
                    for (int p = 0; p < PM; ++p) {
                        if (!((over >> p) & 1u)) continue;
                        int k = 0;
#pragma unroll
                        for (int i = 0; i < SL; ++i) k += cp_popc(mk[p][i] & ge[i]);
                        exceed = exceed || k > room[p];
                        full = full || k == room[p];
                    }
                    if (exceed) {
                        lo = t;
                    } else {
                        hi = t;
                        if (full) {   // the next key below finds a full pattern
                            tie = false;
                            break;
                        }
                    }
                }
            }
            // the rows from hi up; when equal keys (hi - 1) straddle the
            // limit, also the tied rows by pattern and row until one fills
            u64 ge[SL], eq[SL];
#pragma unroll
            for (int i = 0; i < SL; ++i) {
                ge[i] = __ballot(kb[i] >= hi);
                eq[i] = __ballot(tie && kb[i] == hi - 1);
            }
            bool stop = !tie;
#pragma unroll
            for (int p = 0; p < PM; ++p) {
                int k = 0, e = 0;
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    k += cp_popc(mk[p][i] & ge[i]);
                    e += cp_popc(mk[p][i] & eq[i]);
                }
                const int left = stop ? 0 : room[p] - k;   // places for the tied rows
                int before = 0;
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    const u64 tm = mk[p][i] & eq[i];
                    const bool tied = kb[i] == hi - 1 && before + cp_below(tm) < left;
                    if (bp[i] == p && (kb[i] >= hi || tied)) pat[i] = p;
                    before += cp_popc(tm);
                }
                room[p] -= k + min(e, left);
                stop = stop || e > left;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < SL; ++i) pat[i] = max(pat[i], 0);
    cp_write<T, MM, PM, SL, VEC>(ln, rows, pat, live, pm, values, index, n, g, P, S, B, row0, b);
}

// ------------------------------------------------------------ swap search

template <int CTRL> __device__ __forceinline__ double cp_dpp(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
    const u64 u = __builtin_bit_cast(u64, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp((int)u, (int)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp((int)(u >> 32), (int)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
#else
    return v;
#endif
}
// max(v, v of lane ^ 16) / lane ^ 32: gfx950's row and half-wave swaps of a
// register with itself leave one half of the pair in each result
template <int LANES> __device__ __forceinline__ double cp_swap_max(double v) {
#if defined(__HIP_DEVICE_COMPILE__)
    const u64 u = __builtin_bit_cast(u64, v);
    const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
    u64 a, b;
    if constexpr (LANES == 16) {
        const auto rl = __builtin_amdgcn_permlane16_swap(l, l, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(h, h, false, false);
        a = ((u64)rh[0] << 32) | rl[0];
        b = ((u64)rh[1] << 32) | rl[1];
    } else {
        const auto rl = __builtin_amdgcn_permlane32_swap(l, l, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
        a = ((u64)rh[0] << 32) | rl[0];
        b = ((u64)rh[1] << 32) | rl[1];
    }
    return fmax(__builtin_bit_cast(double, a), __builtin_bit_cast(double, b));
#else
    return v;
#endif
}
// Maximum over aligned segments of `g` lanes (a power of two; no NaN); every
// lane of a segment gets it.
__device__ __forceinline__ double cp_seg_max(double v, int g) {
    if (g > 1) v = fmax(v, cp_dpp<0xB1>(v));    // lanes ^ 1
    if (g > 2) v = fmax(v, cp_dpp<0x4E>(v));    // lanes ^ 2
    if (g > 4) v = fmax(v, cp_dpp<0x141>(v));   // the other 4 of 8 (mirrored)
    if (g > 8) v = fmax(v, cp_dpp<0x140>(v));   // the other 8 of 16 (mirrored)
    if (g > 16) v = cp_swap_max<16>(v);
    if (g > 32) v = cp_swap_max<32>(v);
    return v;
}

// the same for a 32-bit whole number
template <int CTRL> __device__ __forceinline__ int cp_dpp_max(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false));
#else
    return v;
#endif
}
__device__ __forceinline__ int cp_seg_max(int v, int g) {
    if (g > 1) v = cp_dpp_max<0xB1>(v);
    if (g > 2) v = cp_dpp_max<0x4E>(v);
    if (g > 4) v = cp_dpp_max<0x141>(v);
    if (g > 8) v = cp_dpp_max<0x140>(v);
    if (g > 16) v = max(v, __shfl_xor(v, 16));
    if (g > 32) v = max(v, __shfl_xor(v, 32));
    return v;
}

// Largest ratio (in binary exponents) of a wave's nonzero magnitudes for the
// gain and the partner's row to fit one binary64 (24 + 19 + 2 + 8 bits), and
// for sums of four magnitudes to be exact in binary64 (24 + 28 + 1)
constexpr int kCpRangeBits = 19, kCpWideBits = 28;

template <typename T, int MM, int PM, int SL, bool VEC>
__global__ __launch_bounds__(64 * kCpWaves) void k_p_swaps(const T *__restrict__ W, int64_t ldw,
                                                           T *__restrict__ values,
                                                           uint8_t *__restrict__ index, PatMasks pm,
                                                           int n, int m, int g, int P, int S, int B,
                                                           int cpw, int64_t chunks) {
    constexpr int ROWS = 64 * SL;
    __shared__ float score_all[kCpWaves][ROWS * PM];
    __shared__ double table_all[kCpWaves][64 * PM];     // best change of pattern e to a, per chunk
    __shared__ int row_all[kCpWaves][64 * PM];          // ... and its row, kept apart (wide range)
    __shared__ int pa_all[kCpWaves][ROWS];              // pattern of each row
    __shared__ int best_all[kCpWaves][ROWS];            // best improving partner, or -1
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t wave_id = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * kCpWaves + wave;
    if (wave_id * cpw >= chunks) return;  // whole waves; no workgroup barrier follows
    const CpLane<SL> ln(wave, S, wave_id, cpw, chunks);
    const int64_t cid = min(ln.id, chunks - 1);
    const int64_t row0 = cid / B * S;
    const int b = (int)(cid % B);
    const int base = ln.on ? ln.c * S : 0;              // LDS row of chunk row 0
    float *score = score_all[wave];
    double *table = table_all[wave];
    int *pa = pa_all[wave], *best = best_all[wave], *rtab = row_all[wave];

    CpRow<T, MM, PM, VEC> rows[SL];
    bool live[SL];
    uint32_t emax = 0, emin = 255, bad = 0;             // exponent fields of the nonzero magnitudes
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int r = ln.r0 + 64 * i;
        live[i] = ln.on && r < S;
        rows[i].load(W + (row0 + min(r, S - 1)) * ldw + (int64_t)b * m, m);
    }
    int at[SL];      // the chunk row now in this lane's place (place j = r0 + 64 i, pattern j / g)
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int j = min(ln.r0 + 64 * i, S - 1);
        at[i] = min((int)index[(row0 + j) * B + b], S - 1);
    }
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        float sc[PM];
        rows[i].scores(pm, P, sc);
        const int r = ln.r0 + 64 * i;
        if (live[i]) {
            pa[base + r] = 0;   // a malformed index leaves rows on pattern 0
#pragma unroll
            for (int p = 0; p < PM; ++p) {
                score[(base + r) * PM + p] = sc[p];
                const uint32_t u = __builtin_bit_cast(uint32_t, sc[p]);
                if (u != 0) {
                    const uint32_t e = max(u >> 23, 1u);
                    emax = max(emax, e);
                    emin = min(emin, e);
                    bad |= e >= 255u ? 1u : 0u;
                }
            }
        }
    }
    p_wave_sync();
    emax = __builtin_amdgcn_readfirstlane(cp_wave_max(emax));
    emin = __builtin_amdgcn_readfirstlane(cp_wave_min(emin));
    const bool exact = !__any(bad != 0) && (emax == 0 || emax - emin <= (uint32_t)kCpWideBits);
    if (exact) {
        // magnitudes as whole numbers of 2^(emin - 150)
        const int up = emax == 0 ? 0 : 150 - (int)emin;
        const int lg = 31 - __builtin_clz(g);
        int own_p[SL];
        double D[SL][PM];        // change of this place's row to pattern p
        auto take_row = [&](int i) __attribute__((always_inline)) {
            const float *s = score + (base + at[i]) * PM;
            double v[PM], o = 0.0;
#pragma unroll
            for (int p = 0; p < PM; ++p) v[p] = __builtin_ldexp((double)s[p], up);
#pragma unroll
            for (int p = 0; p < PM; ++p) o = p == own_p[i] ? v[p] : o;
#pragma unroll
            for (int p = 0; p < PM; ++p) D[i][p] = v[p] - o;
        };
        // places lie g to a segment of lanes
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            own_p[i] = min(ln.r0 + 64 * i, S - 1) >> lg;
            take_row(i);
        }
        // WIDE: gain and row compared one after the other, not in one number
        auto rounds = [&](auto wc) __attribute__((always_inline)) {
            constexpr bool WIDE = decltype(wc)::value;
            constexpr double kUnit = WIDE ? 1.0 : 256.0;
            bool moved[SL];   // a row of these 64 places changed: its patterns' best changes do too
#pragma unroll
            for (int i = 0; i < SL; ++i) moved[i] = true;
            for (int round = 0; round < 8 * S; ++round) {
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    if (!moved[i]) continue;   // uniform across the wave
#pragma unroll
                    for (int p = 0; p < PM; ++p) {
                        if (p >= P) break;
                        // (places past S hold no row: kept out by -inf)
                        const double x = WIDE ? D[i][p] : __builtin_fma(D[i][p], 256.0, (double)(255 - at[i]));
                        const double v = live[i] ? x : -__builtin_inf();
                        const double mx = cp_seg_max(v, g);
                        const bool first = live[i] && ((ln.r0 + 64 * i) & (g - 1)) == 0;
                        const int e = (ln.c * P + own_p[i]) * PM + p;
                        if constexpr (WIDE) {
                            const int q = cp_seg_max(live[i] && v == mx ? 255 - at[i] : -1, g);
                            if (first) rtab[e] = q;
                        }
                        if (first) table[e] = mx;
                    }
                }
                p_wave_sync();
                int bq[SL];
                bool found = false;
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    double bg = 0.0;
                    int br = -1;
#pragma unroll
                    for (int e = 0; e < PM; ++e) {
                        if (e >= P) break;
                        const int te = ((ln.on ? ln.c : 0) * P + e) * PM + own_p[i];
                        const double v = __builtin_fma(D[i][e], kUnit, table[te]);
                        if constexpr (WIDE) {
                            const int r = rtab[te];
                            const bool up_ = e != own_p[i] && (v > bg || (v == bg && r > br));
                            bg = up_ ? v : bg;
                            br = up_ ? r : br;
                        } else {
                            bg = e != own_p[i] ? fmax(bg, v) : bg;
                        }
                    }
                    const bool up_ = live[i] && bg >= kUnit;   // a gain of at least one unit
                    if constexpr (!WIDE) br = (int)(bg - 256.0 * __builtin_floor(bg * (1.0 / 256.0)));
                    bq[i] = up_ ? 255 - br : -1;
                    if (live[i]) best[base + at[i]] = bq[i];
                    found = found || up_;
                }
                if (!__any(found)) break;  // uniform across the wave
                p_wave_sync();
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    const bool swap = bq[i] >= 0 && best[base + bq[i]] == at[i];   // mutual: disjoint pairs
                    if (swap) {
                        at[i] = bq[i];
                        take_row(i);
                    }
                    moved[i] = __any(swap);
                }
                p_wave_sync();   // tables and partners are read before they are rewritten
            }
        };
        if (emax - min(emin, emax) <= (uint32_t)kCpRangeBits) rounds(std::false_type{});
        else rounds(std::true_type{});
#pragma unroll
        for (int i = 0; i < SL; ++i)
            if (live[i]) pa[base + at[i]] = own_p[i];
    } else {
#pragma unroll
        for (int i = 0; i < SL; ++i)
            if (live[i]) pa[base + at[i]] = (ln.r0 + 64 * i) / g;
        p_wave_sync();
        for (int round = 0; round < 8 * S; ++round) {
            bool found = false;
            for (int i = 0; i < SL; ++i) {
                const int r = ln.r0 + 64 * i;
                if (!ln.on || r >= S) continue;
                const float *sr = score + (base + r) * PM;
                const int a = pa[base + r];
                int bq = -1;
                double bg = 0.0;
                for (int q = 0; q < S; ++q) {
                    const int e = pa[base + q];
                    if (e == a) continue;
                    const float *sq = score + (base + q) * PM;
                    const double gain = ((double)sr[e] + (double)sq[a]) - ((double)sr[a] + (double)sq[e]);
                    if (gain > bg) {  // strictly larger: ties keep the lower q
                        bg = gain;
                        bq = q;
                    }
                }
                best[base + r] = bq;
                found = found || bq >= 0;
            }
            if (!__any(found)) break;  // uniform across the wave
            p_wave_sync();
            for (int i = 0; i < SL; ++i) {
                const int r = ln.r0 + 64 * i;
                if (!ln.on || r >= S) continue;
                const int q = best[base + r];
                if (q > r && best[base + q] == r) {  // mutual best partners: disjoint pairs
                    const int a = pa[base + r];
                    pa[base + r] = pa[base + q];
                    pa[base + q] = a;
                }
            }
            p_wave_sync();
        }
    }
    p_wave_sync();
    int pat[SL];
#pragma unroll
    for (int i = 0; i < SL; ++i) pat[i] = live[i] ? pa[base + ln.r0 + 64 * i] : 0;
    cp_write<T, MM, PM, SL, VEC>(ln, rows, pat, live, pm, values, index, n, g, P, S, B, row0, b);
}

// --------------------------------------------------------------- launchers

PatMasks cp_masks(const nmg_p_layout *L) {
    PatMasks pm = {};
    uint8_t off[kCpMaxP];
    for (int p = 0; p < L->P; ++p) {
        p_unrank(L->m, L->n, p, off);
        for (int k = 0; k < L->n; ++k) pm.bits[p] |= (uint8_t)(1u << off[k]);
    }
    return pm;
}

struct CpArgs {
    const nmg_p_layout *L;
    const void *W;
    int64_t ldw;
    void *values;
    uint8_t *index;
    hipStream_t stream;
    bool swaps;
};

template <typename T, int MM, int PM, bool VEC, int SL>
void cp_launch_sl(const CpArgs &a) {
    const nmg_p_layout *L = a.L;
    const CpPlace pl = cp_place(L->S);
    const int64_t chunks = (int64_t)(L->M / L->S) * L->B;
    const int64_t per = (int64_t)pl.chunks_per_wave * kCpWaves;
    const dim3 grid((unsigned)((chunks + per - 1) / per)), block(64 * kCpWaves);
    const PatMasks pm = cp_masks(L);
#define NMG_CP(K)                                                                                  \
    hipLaunchKernelGGL(K, grid, block, 0, a.stream, (const T *)a.W, a.ldw, (T *)a.values, a.index, \
                       pm, L->n, L->m, L->g, L->P, L->S, L->B, pl.chunks_per_wave, chunks)
    if (a.swaps) NMG_CP((k_p_swaps<T, MM, PM, SL, VEC>));
    else if constexpr (SL == 1) {
        // ranks cost S steps a phase for all of a wave's chunks together, the
        // bisection about 10 of three times the work for one: two or more
        // chunks on a wave take the ranks
        if (pl.chunks_per_wave > 1) NMG_CP((k_p_greedy<T, MM, PM, 1, true, VEC>));
        else NMG_CP((k_p_greedy<T, MM, PM, 1, false, VEC>));
    } else NMG_CP((k_p_greedy<T, MM, PM, SL, false, VEC>));
#undef NMG_CP
}

template <typename T, int MM, int PM, bool VEC>
void cp_launch(const CpArgs &a) {
    switch (cp_place(a.L->S).slots) {
        case 1: cp_launch_sl<T, MM, PM, VEC, 1>(a); break;
        case 2: cp_launch_sl<T, MM, PM, VEC, 2>(a); break;
        case 3: cp_launch_sl<T, MM, PM, VEC, 3>(a); break;
        default: cp_launch_sl<T, MM, PM, VEC, 4>(a); break;
    }
}

template <typename T>
void cp_launch_t(const CpArgs &a) {
    // rows of a block as one vector: m = 4 whole vectors of an aligned W
    const bool vec = a.L->m == 4 && aligned(a.W, 4 * sizeof(T)) && a.ldw % 4 == 0;
    if (vec && a.L->P <= 4) cp_launch<T, 4, 4, true>(a);
    else if (vec) cp_launch<T, 4, 6, true>(a);
    else cp_launch<T, 8, 8, false>(a);
}

}  // namespace

// The row-register converters take layouts with at most 8 patterns of at most
// 8 columns; the swap search also needs whole lane segments per group (g a
// power of two of at most 64).
bool nmg_internal::p_pack_rows_supported(const nmg_p_layout *L, bool swaps) {
    const int64_t chunks = (int64_t)(L->M / L->S) * L->B;
    return L->P <= kCpMaxP && L->m <= 8 && L->S <= 256 && chunks < ((int64_t)1 << 31) &&
           (!swaps || ((L->g & (L->g - 1)) == 0 && L->g <= 64));
}

nmg_status nmg_internal::p_pack_rows(const nmg_p_layout *L, const void *W, int64_t ldw, void *values,
                                     uint8_t *index, bool swaps, hipStream_t stream) {
    const CpArgs a{L, W, ldw, values, index, stream, swaps};
    if (L->dtype == NMG_F32) cp_launch_t<float>(a);
    else cp_launch_t<_Float16>(a);
    return launched();
}
