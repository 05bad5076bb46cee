// aspis_device.h -- device code shared by the kernel sources: keys, group
// reductions, the selections on LDS tiles, row loads.  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "aspis_internal.h"

namespace aspis {

namespace {

// ---------------------------------------------------------------------------
// helpers

// Order-preserving map of a binary32 bit pattern to an unsigned key:
// unsigned order of keys == IEEE-754 totalOrder of the floats.
__device__ __forceinline__ uint32_t to_key(uint32_t b) {
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ uint32_t from_key(uint32_t k) {
    return (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
}

// Reductions over groups of G consecutive lanes (G a power of two <= 64).
// Offsets below 16 use DPP row permutations: after the two quad steps every
// lane of a quad holds the quad's value, and the half-row / row mirrors pair
// each lane with one lane of the other half.
enum class Op { And, Or, Add, Max, Min };

template <Op OP>
__device__ __forceinline__ uint32_t combine(uint32_t a, uint32_t b) {
    if constexpr (OP == Op::And) return a & b;
    if constexpr (OP == Op::Or) return a | b;
    if constexpr (OP == Op::Max) return a > b ? a : b;
    if constexpr (OP == Op::Min) return a < b ? a : b;
    return a + b;
}

// Two 16-bit unsigned lanes of a word at once (v_pk_min_u16, v_pk_max_u16,
// v_pk_add_u16: integer lanes, no carry between them).
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_add_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

template <int G, Op OP>
__device__ __forceinline__ uint32_t group_reduce(uint32_t v) {
    static_assert(G >= 1 && G <= 64 && (G & (G - 1)) == 0, "group size");
    if constexpr (G >= 2) v = combine<OP>(v, dpp<0xB1>(v));    // quad_perm [1,0,3,2]
    if constexpr (G >= 4) v = combine<OP>(v, dpp<0x4E>(v));    // quad_perm [2,3,0,1]
    if constexpr (G >= 8) v = combine<OP>(v, dpp<0x141>(v));   // row_half_mirror
    if constexpr (G >= 16) v = combine<OP>(v, dpp<0x140>(v));  // row_mirror
    if constexpr (G >= 32) v = combine<OP>(v, (uint32_t)__shfl_xor((int)v, 16, 64));
    if constexpr (G >= 64) v = combine<OP>(v, (uint32_t)__shfl_xor((int)v, 32, 64));
    return v;
}

// Inclusive prefix sum over groups of G consecutive lanes; g = lane index
// within the group.  A group inside one 16-lane row shifts with DPP row_shr;
// row_shr does not cross rows, so wider groups shift through ds_bpermute.
template <int G>
__device__ __forceinline__ uint32_t group_scan(uint32_t v, int g) {
#pragma unroll
    for (int k = 1; k < G; k <<= 1) {
        uint32_t y;
        if constexpr (G <= 16) {
            if (k == 1) y = dpp<0x111>(v);
            else if (k == 2) y = dpp<0x112>(v);
            else if (k == 4) y = dpp<0x114>(v);
            else y = dpp<0x118>(v);
        } else {
            y = (uint32_t)__shfl_up((int)v, k, 64);
        }
        v += (g >= k) ? y : 0u;
    }
    return v;
}

// Threads per workgroup of the tile kernels for tile width T: 1024 down to
// 16-wide tiles, then one wave (64 lanes) per column.
template <int T>
constexpr int tile_block() { return T >= 16 ? 1024 : 64 * T; }

// LDS layout of a [rows x T] key tile read by G lanes per column.  Row j
// lives at j*T; within the row, column c is stored at c ^ swz(j % G).  The
// G lanes of a column read rows j == g (mod G); the swizzle puts the 32
// lanes of every half-wave in 32 distinct banks.
template <int T, int G>
__host__ __device__ constexpr int tile_swz_of(int g) {
    static_assert(T == 4 || T == 8 || T == 16 || T == 32 || T == 64 || T == 128, "tile width");
    static_assert(G >= 1 && G <= 64 && (G & (G - 1)) == 0, "lanes per column");
    if constexpr (T >= 32) {
        static_assert(G <= 32, "swizzle needs at most 32 lanes per wide column");
        return g * (32 / G);
    } else {
        return (g / (32 / T)) & (T - 1);
    }
}

// The promise above, checked at compile time for every (T, G) the kernels
// instantiate: the first word each lane of a half-wave reads lies in a bank
// (of 32) of its own.  A lane's later rows lie G*T words further, a multiple
// of 32, so they keep the same banks.
template <int T, int G>
constexpr bool tile_swz_conflict_free() {
    for (int h = 0; h < T * G; h += 32) {
        uint32_t used = 0;
        for (int i = h; i < h + 32 && i < T * G; ++i) {
            const int c = i / G, g = i % G;
            const int bank = (g * T + (c ^ tile_swz_of<T, G>(g))) % 32;
            if (used & (1u << bank)) return false;
            used |= 1u << bank;
        }
    }
    return true;
}

template <int T, int G>
__device__ __forceinline__ int tile_swz(int g) {
    static_assert(tile_swz_conflict_free<T, G>(), "tile swizzle leaves a bank conflict");
    return tile_swz_of<T, G>(g);
}

// Store the keys of row j, columns 4cq..4cq+3.
template <int T, int G>
__device__ __forceinline__ void put_keys(uint32_t *tile, int j, int cq, const uint32_t k[4]) {
    const int sw = tile_swz<T, G>(j % G);
    if constexpr (T >= 32 && (32 / G) % 4 == 0) {
        // the swizzle keeps each aligned group of four columns together
        *reinterpret_cast<uint4 *>(&tile[j * T + ((4 * cq) ^ sw)]) = make_uint4(k[0], k[1], k[2], k[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[j * T + ((4 * cq + e) ^ sw)] = k[e];
    }
}

constexpr int kSelBatch = 8;   // LDS reads in flight per lane

// Per-column histogram of the selection (kHistBuckets buckets plus one
// overflow bucket); the column stride of kHistStride words keeps each
// column's bucket block 16-byte aligned and puts equal buckets of
// neighbouring columns in different banks.
constexpr int kHistWindow = 7;   // key bits resolved by one histogram round
static_assert(kHistBuckets == 1 << kHistWindow && kHistStride > kHistBuckets, "histogram");

__host__ __device__ constexpr int64_t hist_words(int T) { return (int64_t)T * kHistStride; }

// One pass over a lane's candidates, in batches of kSelBatch LDS reads.
template <int STRIDE, typename F>
__device__ __forceinline__ void for_each_candidate(const uint32_t *base, int cnt, F &&fn) {
    int x = 0;
    for (; x + kSelBatch <= cnt; x += kSelBatch) {
        uint32_t v[kSelBatch];
#pragma unroll
        for (int u = 0; u < kSelBatch; ++u) v[u] = base[(x + u) * STRIDE];
#pragma unroll
        for (int u = 0; u < kSelBatch; ++u) fn(v[u]);
    }
    for (; x < cnt; ++x) fn(base[x * STRIDE]);
}

// In-place compaction of a lane's candidates: keeps the values for which
// keep(v) holds, in order.  Every value is stored at the write cursor, which
// advances only for kept values; a batch is read before any of its slots is
// overwritten and the cursor never passes the read point.  Returns the
// number kept.
template <int STRIDE, typename F>
__device__ __forceinline__ int compact(uint32_t *base, int cnt, F &&keep) {
    int w = 0, x = 0;
    for (; x + kSelBatch <= cnt; x += kSelBatch) {
        uint32_t v[kSelBatch];
#pragma unroll
        for (int u = 0; u < kSelBatch; ++u) v[u] = base[(x + u) * STRIDE];
#pragma unroll
        for (int u = 0; u < kSelBatch; ++u) {
            base[w * STRIDE] = v[u];
            w += keep(v[u]) ? 1 : 0;
        }
    }
    for (; x < cnt; ++x) {
        const uint32_t v = base[x * STRIDE];
        base[w * STRIDE] = v;
        w += keep(v) ? 1 : 0;
    }
    return w;
}

// Lower median (rank floor((n-1)/2)) of each of the T columns of the LDS key
// tile holding n rows, found by the G lanes stid = c*G + g of each column c;
// written to out[k0 + c] for k0 + c < d.  hist: the workgroup's histogram
// block (hist_words(T) words, zero on entry; left zero on exit except for
// the overflow buckets).
//
// Exact selection on the keys in two stages:
//  1. histogram rounds while many candidates remain: the bits above the
//     highest bit where the candidates differ are common to all of them, so
//     the next kHistWindow bits below it split the candidates into ordered
//     buckets; an LDS histogram and a prefix scan over the buckets give the
//     bucket holding the sought rank, and only its members are kept
//     (compacted in place).  The first round decides the sign from the
//     count of sign-clear keys and works on the magnitude bits (the keys of
//     negative values hold them complemented); keys of the other sign land
//     in the overflow bucket or past every bucket of the sought sign.
//  2. bitwise MSB radix select on the few survivors: split on the highest
//     differing bit, keep the side holding the rank, until all are equal.
// Lane g owns rows g, g+G, ...; its x-th candidate lives at base[x*STRIDE].
template <int T, int G>
__device__ __forceinline__ void select_tile(uint32_t *tile, uint32_t *hist, int n, int64_t k0,
                                            int64_t d, float *out, int stid) {
    constexpr int STRIDE = G * T;
    constexpr int BPL = kHistBuckets / G;   // buckets scanned per lane
    static_assert(BPL >= 2 && BPL % 2 == 0, "buckets per lane");
    const int g = stid % G;
    const int c = stid / G;
    uint32_t *base = tile + g * T + (c ^ tile_swz<T, G>(g));
    uint32_t *hcol = hist + c * kHistStride;
    int cnt = (n > g) ? (n - g + G - 1) / G : 0;
    int total = n;
    uint32_t m = (uint32_t)(n - 1) / 2;

    // first pass: common magnitude bits and the count of sign-clear keys
    uint32_t am = 0xFFFFFFFFu, om = 0u, z = 0u;
    for_each_candidate<STRIDE>(base, cnt, [&](uint32_t v) {
        const uint32_t mag = (v ^ ~(uint32_t)((int32_t)v >> 31)) & 0x7FFFFFFFu;
        am &= mag;
        om |= mag;
        z += v >> 31;
    });
    am = group_reduce<G, Op::And>(am);
    om = group_reduce<G, Op::Or>(om);
    z = (uint32_t)total - group_reduce<G, Op::Add>(z);   // keys with the top bit clear

    auto and_or = [&](uint32_t &a, uint32_t &o) {
        a = 0xFFFFFFFFu;
        o = 0u;
        for_each_candidate<STRIDE>(base, cnt, [&](uint32_t v) {
            a &= v;
            o |= v;
        });
        a = group_reduce<G, Op::And>(a);
        o = group_reduce<G, Op::Or>(o);
    };
    // one histogram round over the candidates whose keys lie in
    // [bias, bias + 2^(hb+1)); keeps the bucket holding rank m
    auto hist_round = [&](uint32_t bias, int hb) {
        const int sh = hb >= kHistWindow - 1 ? hb - (kHistWindow - 1) : 0;
        for_each_candidate<STRIDE>(base, cnt, [&](uint32_t v) {
            const uint32_t b = min((v - bias) >> sh, (uint32_t)kHistBuckets);
            atomicAdd(&hcol[b], 1u);
        });
        // bucket holding rank m: B = number of buckets whose inclusive
        // prefix count is <= m, below = the largest such prefix
        uint32_t h[BPL];
#pragma unroll
        for (int q = 0; q < BPL; q += 2) {
            const uint2 w2 = *reinterpret_cast<const uint2 *>(&hcol[g * BPL + q]);
            h[q] = w2.x;
            h[q + 1] = w2.y;
        }
#pragma unroll
        for (int q = 0; q < BPL; q += 2)
            *reinterpret_cast<uint2 *>(&hcol[g * BPL + q]) = make_uint2(0u, 0u);
        uint32_t tot = 0u;
#pragma unroll
        for (int q = 0; q < BPL; ++q) tot += h[q];
        uint32_t run = group_scan<G>(tot, g) - tot;
        uint32_t le = 0u, below = 0u;
#pragma unroll
        for (int q = 0; q < BPL; ++q) {
            run += h[q];
            const bool ok = run <= m;
            le += ok ? 1u : 0u;
            below = ok ? run : below;
        }
        le = group_reduce<G, Op::Add>(le);
        below = group_reduce<G, Op::Max>(below);
        m -= below;
        const uint32_t lo = bias + (le << sh);
        const uint32_t width = 1u << sh;
        cnt = compact<STRIDE>(base, cnt, [&](uint32_t v) { return v - lo < width; });
        total = (int)group_reduce<G, Op::Add>((uint32_t)cnt);
    };

    uint32_t a, o, varying;
    bool have_count = false;
    if (total > 2 * G) {
        uint32_t sgn = 0x80000000u;
        if (m < z) sgn = 0u;
        else m -= z;
        const uint32_t vm = am ^ om;
        if (vm == 0u) {   // every candidate has the same magnitude
            a = sgn ? (0x80000000u | am) : (~am & 0x7FFFFFFFu);
            varying = 0u;
        } else {
            const int hb = 31 - __clz(vm);
            const uint32_t hi = 0x7FFFFFFFu & ~((2u << hb) - 1u);
            hist_round(sgn ? (0x80000000u | (am & hi)) : (~am & hi), hb);
            and_or(a, o);
            varying = a ^ o;
            // the sign is settled now; every round settles the bits from the
            // highest differing one down to the window's lowest, so the next
            // round starts strictly lower (at most 31 / kHistWindow more)
            for (int round = 0; varying != 0u && total > 2 * G && round < 5; ++round) {
                const int hb2 = 31 - __clz(varying);
                hist_round(a & ~((2u << hb2) - 1u), hb2);
                and_or(a, o);
                varying = a ^ o;
            }
        }
    } else {
        and_or(a, o);
        varying = a ^ o;
        have_count = (varying >> 31) != 0u;   // z counts zeros of the top bit
    }

    // each step settles the highest differing bit: at most 32 steps
    for (int step = 0; varying != 0u && step < 32; ++step) {
        const uint32_t bit = 1u << (31 - __clz(varying));
        if (!have_count) {
            z = 0u;
            for_each_candidate<STRIDE>(base, cnt, [&](uint32_t v) { z += (v & bit) == 0u; });
            z = group_reduce<G, Op::Add>(z);
        }
        have_count = false;
        uint32_t want;
        if (m < z) {
            want = 0u;
        } else {
            want = bit;
            m -= z;
        }
        cnt = compact<STRIDE>(base, cnt, [&](uint32_t v) { return (v & bit) == want; });
        and_or(a, o);
        varying = a ^ o;
    }
    if (g == 0 && k0 + c < d) out[k0 + c] = __uint_as_float(from_key(a));
}

// ---------------------------------------------------------------------------
// Half-key tiles.  The LDS tile holds only the high 16 bits of every key,
// two rows per word, so a tile of the same LDS size is twice as wide (and
// the row segments read from HBM twice as long).  The high half of the
// sought key is selected exactly on the tile; the low halves are then read
// back from the replica rows, only for the rows whose high half equals it
// (about one row per column on continuous data; every row when all high
// halves of a column are equal, which costs speed, not exactness).
//
// Layout for a streaming role of RPI rows per sweep: rows j and j + RPI,
// which one lane loads in two consecutive sweeps, share the word of
// pair-row p = (j / 2RPI) * RPI + j % RPI (j / RPI even: low half), stored
// at p*T + (c ^ swz(p % G)), so a lane writes whole words.  Rows without a
// kept value (past the last row, or a dropped file) hold the largest key,
// 0xFFFF, as do the low halves read back for them: appending elements that
// are not below any other leaves every rank below the kept count in place.

constexpr int kHalfWindow = 6;                  // key bits per histogram round
constexpr int kHalfBuckets = 1 << kHalfWindow;
constexpr int kHalfStride = kHalfBuckets + 2;   // words per column block
constexpr uint32_t kHalfTop = 0xFFFFu;          // largest key: padding rows

__host__ __device__ constexpr int64_t half_hist_words(int T) { return (int64_t)T * kHalfStride; }
// streaming rows per sweep of a tile T columns wide, for `fill` streaming
// threads of four columns each
__host__ __device__ constexpr int half_rpi(int T, int fill) { return fill * 4 / T; }
// pair-rows of a tile of `rows` rows: whole pairs of sweeps
__host__ __device__ constexpr int64_t half_pair_rows(int64_t rows, int T, int fill) {
    return (rows + 2 * half_rpi(T, fill) - 1) / (2 * half_rpi(T, fill)) * half_rpi(T, fill);
}
__host__ __device__ constexpr int64_t half_tile_words(int64_t rows, int T, int fill) {
    return half_pair_rows(rows, T, fill) * T;
}

// Row held by half h of pair-row p.
template <int RPI>
__device__ __forceinline__ int half_row(int p, int h) {
    return (p / RPI) * 2 * RPI + h * RPI + p % RPI;
}

// The high halves of two full keys, packed (a's in the low 16 bits).
__device__ __forceinline__ uint32_t pack_high(uint32_t a, uint32_t b) {
    return (a >> 16) | (b & 0xFFFF0000u);
}

// Store pair-row p, columns 4cq..4cq+3, from the packed high halves of the
// even sweep (lo: columns 0,1 and 2,3 in two registers) and of the odd one.
template <int T, int G>
__device__ __forceinline__ void put_pairs(uint32_t *tile, int p, int cq, const uint32_t lo[2],
                                          const uint32_t hi[2]) {
    uint32_t w[4];
    w[0] = (lo[0] & 0xFFFFu) | (hi[0] << 16);
    w[1] = (lo[0] >> 16) | (hi[0] & 0xFFFF0000u);
    w[2] = (lo[1] & 0xFFFFu) | (hi[1] << 16);
    w[3] = (lo[1] >> 16) | (hi[1] & 0xFFFF0000u);
    const int sw = tile_swz<T, G>(p % G);
    if constexpr (T >= 64 && (32 / G) % 4 == 0) {
        // the swizzle keeps each aligned group of four columns together
        *reinterpret_cast<uint4 *>(&tile[p * T + ((4 * cq) ^ sw)]) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[p * T + ((4 * cq + e) ^ sw)] = w[e];
    }
}

// Lower median of each of the T columns of a half-key tile of np pair-rows
// holding nk kept values (1 <= nk, 2*np <= 65536), by the G lanes
// stid = c*G + g of column c, written to out[k0 + c] for k0 + c < d.
// row(j) gives the replica row of g behind tile row j, or -1 for a padding
// row.  hist: half_hist_words(T) words, zero on entry and on exit.  The
// tile is overwritten.  With REG > 0 (np a multiple of G, np / G <= REG)
// the lane's words are read from the tile once, into registers, and every
// later pass over the keys reads those (the median kernel measured 4-5 %
// faster at 455 rows; the single pass, whose registers are taken by its
// own state, keeps reading the tile).
//
//  1. one pass: the least key, the greatest key below 0xFFFF, the least
//     sign-set and the greatest sign-clear key, and the count of sign-set
//     keys (packed 16-bit min / max / add, two keys an instruction); settles
//     the sign and the window [lo, hi] of the keys of that sign;
//  2. histogram rounds over the window, each resolving kHalfWindow bits,
//     until the sought high half H is known (at most 3 rounds; H = 0xFFFF
//     when the rank falls past a sign-set window); nothing is compacted,
//     every round reads all keys;
//  3. one pass collecting the rows whose high half is H into the lane's
//     16-bit slots (in place), then their low halves are read from g;
//  4. bitwise radix select on those low halves for the remaining rank.
template <int T, int G, int RPI, int REG = 0, typename RowFn>
__device__ __forceinline__ void select_half_tile(uint32_t *tile, uint32_t *hist, int np, int nk,
                                                 int64_t k0, int64_t d, float *out, int stid,
                                                 const float *__restrict__ g, RowFn &&row) {
    constexpr int STRIDE = G * T;   // words between a lane's pair-rows
    constexpr int BPL = kHalfBuckets / G;
    static_assert(BPL >= 2 && BPL % 2 == 0, "buckets per lane");
    const int gl = stid % G;
    const int c = stid / G;
    uint32_t *base = tile + gl * T + (c ^ tile_swz<T, G>(gl));
    uint16_t *base16 = reinterpret_cast<uint16_t *>(base);
    uint32_t *hcol = hist + c * kHalfStride;
    const int cnt = np > gl ? (np - gl + G - 1) / G : 0;   // words of this lane
    uint32_t m = (uint32_t)(nk - 1) / 2;
    // REG > 0: the lane's words are read once, into registers.  The caller
    // passes np = half_pair_rows(...), a multiple of RPI = 4G, so every lane
    // of the wave holds the same count, a multiple of 4, at most REG
    static_assert(REG == 0 || RPI == 4 * G, "register mode needs RPI = 4G");
    uint32_t kw[REG > 0 ? REG : 1];
    const int cw = __builtin_amdgcn_readfirstlane(cnt);

    // every key of the lane: fn(key, word x, half h) for pair-row gl + x*G
    auto each = [&](auto &&fn) __attribute__((always_inline)) {
        if constexpr (REG > 0) {
            // cw is a multiple of 4 (np is a multiple of RPI = 4G)
#pragma unroll
            for (int xb = 0; xb < REG; xb += 4) {
                if (xb < cw) {
#pragma unroll
                    for (int x = xb; x < xb + 4 && x < REG; ++x) {
                        fn(kw[x] & 0xFFFFu, x, 0);
                        fn(kw[x] >> 16, x, 1);
                    }
                }
            }
            return;
        }
        int x = 0;
        for (; x + kSelBatch <= cnt; x += kSelBatch) {
            uint32_t v[kSelBatch];
#pragma unroll
            for (int u = 0; u < kSelBatch; ++u) v[u] = base[(x + u) * STRIDE];
#pragma unroll
            for (int u = 0; u < kSelBatch; ++u) {
                fn(v[u] & 0xFFFFu, x + u, 0);
                fn(v[u] >> 16, x + u, 1);
            }
        }
        for (; x < cnt; ++x) {
            const uint32_t v = base[x * STRIDE];
            fn(v & 0xFFFFu, x, 0);
            fn(v >> 16, x, 1);
        }
    };
    // the lane's x-th 16-bit slot (step 3 on)
    auto slot = [&](int x) __attribute__((always_inline)) -> uint16_t & {
        return base16[(x >> 1) * 2 * STRIDE + (x & 1)];
    };

    // 1. extremes and the sign count, both keys of a word at once in 16-bit
    //    lanes: the least key, the greatest key below 0xFFFF (the greatest
    //    key + 1, which wraps 0xFFFF to 0), and with the sign bit flipped the
    //    least sign-set key and the greatest sign-clear key; the number of
    //    sign-set keys
    uint32_t mn2 = 0xFFFFFFFFu, mt2 = 0u, ms2 = 0xFFFFFFFFu, mc2 = 0u, ns = 0u;
    auto stats = [&](uint32_t w) __attribute__((always_inline)) {
        const uint32_t x = w ^ 0x80008000u;
        mn2 = pk_min_u16(mn2, w);
        mt2 = pk_max_u16(mt2, pk_add_u16(w, 0x00010001u));
        ms2 = pk_min_u16(ms2, x);
        mc2 = pk_max_u16(mc2, x);
        ns += (uint32_t)__builtin_popcount(w & 0x80008000u);
    };
    if constexpr (REG > 0) {
#pragma unroll
        for (int xb = 0; xb < REG; xb += 4) {
            if (xb < cw) {
#pragma unroll
                for (int x = xb; x < xb + 4 && x < REG; ++x) kw[x] = base[x * STRIDE];
            }
        }
#pragma unroll
        for (int xb = 0; xb < REG; xb += 4) {
            if (xb < cw) {
#pragma unroll
                for (int x = xb; x < xb + 4 && x < REG; ++x) stats(kw[x]);
            }
        }
    } else {
        int x = 0;
        for (; x + kSelBatch <= cnt; x += kSelBatch) {
            uint32_t v[kSelBatch];
#pragma unroll
            for (int u = 0; u < kSelBatch; ++u) v[u] = base[(x + u) * STRIDE];
#pragma unroll
            for (int u = 0; u < kSelBatch; ++u) stats(v[u]);
        }
        for (; x < cnt; ++x) stats(base[x * STRIDE]);
    }
    auto lo16 = [](uint32_t v2, bool lower) __attribute__((always_inline)) {
        const uint32_t a = v2 & 0xFFFFu, b = v2 >> 16;
        return lower ? (a < b ? a : b) : (a > b ? a : b);
    };
    const uint32_t mn = group_reduce<G, Op::Min>(lo16(mn2, true));                // least key
    const uint32_t mt = group_reduce<G, Op::Max>(lo16(mt2, false));               // greatest below 0xFFFF, + 1
    const uint32_t ms = group_reduce<G, Op::Min>(lo16(ms2, true)) ^ 0x8000u;      // least sign-set
    const uint32_t mc = group_reduce<G, Op::Max>(lo16(mc2, false)) ^ 0x8000u;     // greatest sign-clear
    const uint32_t z = (uint32_t)(2 * np) - group_reduce<G, Op::Add>(ns);         // sign-clear count

    // 2. the window [lo, hi] of the keys of the sought key's sign (below
    //    0xFFFF); histogram rounds split it into kHalfBuckets buckets of
    //    2^sh keys and keep the one holding rank m, until sh = 0 (16 bits:
    //    three rounds at most).  A key above hi inside the window (0xFFFF, or
    //    a sign-set key in a sign-clear window) is counted like any other:
    //    it is above the sought key.  The rank past a sign-set window is a
    //    0xFFFF key.
    //    The round of single keys (sh = 0) also lists the lane's keys in its
    //    window as (word, half, bucket) codes in the lane's 16-bit slots, in
    //    place (the write cursor never passes the read cursor), and keeps
    //    those of the sought bucket as row numbers: step 3 then has its rows
    //    without another pass.  Not in a first round that may find the rank
    //    past a sign-set window (the tile must stay whole for the 0xFFFF
    //    pass), nor when a lane holds 512 words or more (9 bits of word).
    uint32_t H = kHalfTop;
    bool settled = false, collected = false;
    int w = 0;
    uint32_t lo, hi;
    const bool clear_sign = m < z;
    if (clear_sign) {
        lo = mn;
        hi = mc;
    } else {
        m -= z;
        lo = ms;
        hi = mt - 1u;
        if (mt == 0u || hi < lo) settled = true;   // no sign-set key below 0xFFFF
    }
    if (!settled) {
        uint32_t bias = lo;
        const int width = 32 - __clz(hi - lo);   // bits of hi - lo (0 when equal)
        int sh = width > kHalfWindow ? width - kHalfWindow : 0;
        for (int round = 0; round < 3; ++round) {
            const uint32_t span = (uint32_t)kHalfBuckets << sh;
            const bool list = sh == 0 && (round > 0 || clear_sign) && np <= 511 * G;
            if (list) {
                each([&](uint32_t k, int x, int hf) {
                    const uint32_t o = k - bias;
                    if (o < span) {
                        atomicAdd(&hcol[o], 1u);
                        slot(w) = (uint16_t)(((uint32_t)x << 7) | ((uint32_t)hf << 6) | o);
                        ++w;
                    }
                });
            } else {
                each([&](uint32_t k, int, int) {
                    const uint32_t o = k - bias;
                    if (o < span) atomicAdd(&hcol[o >> sh], 1u);
                });
            }
            uint32_t h[BPL];
#pragma unroll
            for (int q = 0; q < BPL; q += 2) {
                const uint2 w2 = *reinterpret_cast<const uint2 *>(&hcol[gl * BPL + q]);
                h[q] = w2.x;
                h[q + 1] = w2.y;
            }
#pragma unroll
            for (int q = 0; q < BPL; q += 2)
                *reinterpret_cast<uint2 *>(&hcol[gl * BPL + q]) = make_uint2(0u, 0u);
            uint32_t tot = 0u;
#pragma unroll
            for (int q = 0; q < BPL; ++q) tot += h[q];
            uint32_t run = group_scan<G>(tot, gl) - tot;
            uint32_t le = 0u, below = 0u;
#pragma unroll
            for (int q = 0; q < BPL; ++q) {
                run += h[q];
                const bool ok = run <= m;
                le += ok ? 1u : 0u;
                below = ok ? run : below;
            }
            le = group_reduce<G, Op::Add>(le);
            below = group_reduce<G, Op::Max>(below);
            m -= below;
            if (le == (uint32_t)kHalfBuckets) {   // past the window: a 0xFFFF key
                settled = true;
                break;
            }
            bias += le << sh;
            if (sh == 0) {
                if (list) {   // the listed keys of bucket le, as row numbers
                    int n2 = 0;
                    for (int j = 0; j < w; ++j) {
                        const uint32_t v = slot(j);
                        if ((v & 63u) == le) {
                            slot(n2) = (uint16_t)half_row<RPI>(gl + (int)(v >> 7) * G, (int)(v >> 6) & 1);
                            ++n2;
                        }
                    }
                    w = n2;
                    collected = true;
                }
                break;
            }
            sh = sh > kHalfWindow ? sh - kHalfWindow : 0;
        }
        if (!settled) H = bias;
    }

    // 3. rows whose high half is H, as row numbers in the lane's slots (the
    //    write cursor never passes the read cursor), then their low halves
    if (!collected) {
        w = 0;
        each([&](uint32_t k, int x, int hf) {
            if (k == H) {
                slot(w) = (uint16_t)half_row<RPI>(gl + x * G, hf);
                ++w;
            }
        });
    }
    const bool valid = k0 + c < d;
    constexpr int kGather = 4;   // row reads in flight per lane
    for (int x0 = 0; x0 < w; x0 += kGather) {
        uint32_t v[kGather];
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
            v[u] = 0xFFFFFFFFu;   // a padding row: the largest key
            if (x0 + u < w) {
                const int64_t rr = row(slot(x0 + u));
                if (rr >= 0 && valid) v[u] = to_key(__float_as_uint(g[rr * d + k0 + c]));
            }
        }
#pragma unroll
        for (int u = 0; u < kGather; ++u)
            if (x0 + u < w) slot(x0 + u) = (uint16_t)(v[u] & 0xFFFFu);
    }

    // 4. bitwise radix select of rank m among the low halves
    auto and_or = [&](uint32_t &a, uint32_t &o) __attribute__((always_inline)) {
        a = 0xFFFFu;
        o = 0u;
        for (int x = 0; x < w; ++x) {
            const uint32_t v = slot(x);
            a &= v;
            o |= v;
        }
        a = group_reduce<G, Op::And>(a);
        o = group_reduce<G, Op::Or>(o);
    };
    uint32_t a, o;
    and_or(a, o);
    uint32_t varying = a ^ o;
    for (int step = 0; varying != 0u && step < 16; ++step) {
        const uint32_t bit = 1u << (31 - __clz(varying));
        uint32_t zc = 0u;
        for (int x = 0; x < w; ++x) zc += (slot(x) & bit) == 0u;
        zc = group_reduce<G, Op::Add>(zc);
        uint32_t want;
        if (m < zc) {
            want = 0u;
        } else {
            want = bit;
            m -= zc;
        }
        int nw = 0;
        for (int x = 0; x < w; ++x) {
            const uint16_t v = slot(x);
            slot(nw) = v;
            nw += (v & bit) == want ? 1 : 0;
        }
        w = nw;
        and_or(a, o);
        varying = a ^ o;
    }
    if (gl == 0 && valid) out[k0 + c] = __uint_as_float(from_key((H << 16) | a));
}

// One 16-byte load (16-byte aligned) from a replica row that the pass
// reads once: a non-temporal load, which streams past the caches instead of
// filling them with lines nothing reads again (measured 3-6 % faster than a
// plain load on the 61 GB single pass).
__device__ __forceinline__ uint4 load_stream(const float *p) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Load four consecutive coordinates [k, k+4) of one row as bit patterns;
// coordinates at or beyond kend read as 0.
template <bool VEC>
__device__ __forceinline__ void load4(const float *row, int64_t k, int64_t kend,
                                      uint32_t v[4]) {
    if (VEC && k + 3 < kend) {
        const uint4 q = load_stream(row + k);
        v[0] = q.x;
        v[1] = q.y;
        v[2] = q.z;
        v[3] = q.w;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = (k + e < kend) ? __float_as_uint(row[k + e]) : 0u;
    }
}

// Row of replica (i,s): i*R+s in the file-major tensor, or row_of[i*R+s]
// when a row table is given.
__device__ __forceinline__ int64_t replica_row(const int32_t *row_of, int64_t i, int R, int s) {
    return row_of ? (int64_t)row_of[i * R + s] : i * R + s;
}

}  // namespace

// The tiles a median launch computes: every tile, or (a repair after a
// wrong guess) the tiles of the groups whose bit is set, bit b for tiles
// [b << gshift, (b + 1) << gshift).  Uniform per workgroup.
struct TileMask {
    const uint32_t *bits = nullptr;
    const int32_t *count = nullptr;   // groups set (no tile at all when 0)
    int gshift = 0;
    __device__ __forceinline__ bool has(int64_t t) const {
        const int64_t b = t >> gshift;
        return ((bits[b >> 5] >> (b & 31)) & 1u) != 0u;
    }
    // the first computed tile of t, t + step, ..., or one >= ntiles: t
    // itself when its bit is set, else the bits of eight candidates at once
    __device__ __forceinline__ int64_t next(int64_t t, int64_t step, int64_t ntiles) const {
        if (bits == nullptr || t >= ntiles) return t;
        if (*count == 0) return ntiles;
        if (has(t)) return t;
        for (t += step; t < ntiles; t += 8 * step) {
            uint32_t hit = 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t tu = t + u * step;
                if (tu < ntiles && has(tu)) hit |= 1u << u;
            }
            if (hit) return t + (int64_t)(__ffs(hit) - 1) * step;
        }
        return ntiles;
    }
};

}  // namespace aspis
