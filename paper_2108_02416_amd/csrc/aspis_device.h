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

// to_key on the high halves of two bit patterns packed in a word (the high
// half of a key depends on the high half of the pattern alone)
__device__ __forceinline__ uint32_t pk_high_keys(uint32_t w) {
    typedef short i16x2 __attribute__((ext_vector_type(2)));
    const uint32_t sgn = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, w) >> (short)15);
    return w ^ (sgn | 0x80008000u);
}
// the high halves of two bit patterns, packed (a's in the low 16 bits)
__device__ __forceinline__ uint32_t pack_high(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
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
// written to out[k] where k = col(c), unless that is negative.  hist: the workgroup's histogram
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
template <int T, int G, typename ColFn>
__device__ __forceinline__ void select_tile(uint32_t *tile, uint32_t *hist, int n, float *out,
                                            int stid, ColFn &&col) {
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
    if (g == 0) {
        const int64_t k = col(c);
        if (k >= 0) out[k] = __uint_as_float(from_key(a));
    }
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

// streaming rows per sweep of a tile T columns wide, for `fill` streaming
// threads of four columns each
__host__ __device__ constexpr int half_rpi(int T, int fill) { return fill * 4 / T; }
// words of a tile of `sweeps` sweeps (an even count), sweeps * rpi rows:
// padded to the sweeps of its kernel, so that the kernels have no bound of
// their own inside a tile
__host__ __device__ constexpr int64_t half_tile_words(int sweeps, int fill) {
    return (int64_t)sweeps * fill * 2;
}

// Row held by half h of pair-row p.
template <int RPI>
__device__ __forceinline__ int half_row(int p, int h) {
    return (p / RPI) * 2 * RPI + h * RPI + p % RPI;
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

// Lower median of each of the T columns of a half-key tile of NW*G pair-rows
// (NW words per lane, a multiple of 4) holding nk kept values (1 <= nk,
// 2*NW*G <= 65536), by the G lanes stid = c*G + g of column c, written to
// out[k] where k = col(c), unless that is negative.  row(j) gives the byte
// offset in g of the replica row behind tile row j, or -1 for a padding row.
// The tile may be overwritten.
//
//  1. the high byte of the sought key: the lane's high bytes, four to a
//     register, then eight binary-search steps.  A step needs the number of
//     keys below c, and v_sad_u8 sums |byte - c| over four bytes in one
//     instruction: with S(c) that sum over the column, S(c) - S(c-1) =
//     #(bytes <= c-1) - #(bytes >= c), so two of them give the count
//     exactly, half an instruction a key and step;
//  2. the low byte of the high half the same way: every 16-bit key clamped
//     to the settled high byte (a key below it becomes byte 0, above it
//     0xFF: neither changes the count below c for 1 <= c <= 0xFF);
//  3. one pass finding the rows whose high half is the sought one: a lane
//     keeps up to four in registers; when a lane of the wave finds more, the
//     rows are listed in the lanes' 16-bit slots of the tile (in place);
//     their low halves are read from g;
//  4. bitwise radix select on those low halves for the remaining rank.
//
// The pass is bound by the selecting waves' issue slots and by its chain of
// dependent steps, so it uses neither LDS atomics nor data-dependent rounds:
// about 14 VALU instructions a key, the tile read three times.  The LDS
// histograms it replaces took about 28 and waited for their atomics in every
// round: the median of 455 rows, d = 1.5M, 897 -> 640 us.
template <int T, int G, int RPI, int NW, typename RowFn, typename ColFn>
__device__ __forceinline__ void select_half_tile(uint32_t *tile, int nk, float *out, int stid,
                                                 const float *__restrict__ g, RowFn &&row,
                                                 ColFn &&column) {
    static_assert(RPI % (4 * G) == 0 && NW % 4 == 0, "whole blocks of four words per lane");
    constexpr int STRIDE = G * T;   // words between a lane's pair-rows
    const int gl = stid % G;
    const int c = stid / G;
    uint32_t *base = tile + gl * T + (c ^ tile_swz<T, G>(gl));
    const uint32_t m = (uint32_t)(nk - 1) / 2;

    // four keys' bytes to a register
    constexpr int NB = NW / 2;
    uint32_t kb[NB];
    auto load_bytes = [&](uint32_t sel, auto &&map) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NW; x += 2)
            kb[x / 2] = __builtin_amdgcn_perm(map(base[(x + 1) * STRIDE]), map(base[x * STRIDE]), sel);
    };
    // bytes of the column below c1 (1 <= c1 <= 0xFF)
    auto below_byte = [&](uint32_t c1) __attribute__((always_inline)) -> uint32_t {
        const uint32_t pc = c1 * 0x01010101u, pm = pc - 0x01010101u;
        uint32_t a0 = 0u, a1 = 0u, b0 = 0u, b1 = 0u;
#pragma unroll
        for (int x = 0; x < NB; x += 2) {
            a0 = __builtin_amdgcn_sad_u8(kb[x], pc, a0);
            b0 = __builtin_amdgcn_sad_u8(kb[x], pm, b0);
            a1 = __builtin_amdgcn_sad_u8(kb[x + 1], pc, a1);
            b1 = __builtin_amdgcn_sad_u8(kb[x + 1], pm, b1);
        }
        return (2u * NW * G + group_reduce<G, Op::Add>(a0 + a1 - b0 - b1)) >> 1;
    };
    uint32_t below = 0u;   // keys below the sought key's settled bits
    // the byte of the key of rank m: the greatest c with at most m bytes below
    auto search_byte = [&]() __attribute__((always_inline)) -> uint32_t {
        uint32_t b = 0u;
        for (uint32_t bit = 0x80u; bit != 0u; bit >>= 1) {
            const uint32_t n = below_byte(b | bit);
            if (n <= m) {
                b |= bit;
                below = n;
            }
        }
        return b;
    };
    // 1. the high byte
    load_bytes(0x07050301u, [](uint32_t w) __attribute__((always_inline)) { return w; });
    const uint32_t hb = search_byte();
    // 2. the low byte of the high half
    const uint32_t lo2 = hb * 0x01000100u, hi2 = lo2 | 0x00FF00FFu;
    load_bytes(0x06040200u, [&](uint32_t w) __attribute__((always_inline)) {
        return pk_min_u16(pk_max_u16(w, lo2), hi2);
    });
    const uint32_t H = (hb << 8) | search_byte();
    uint32_t rank = m - below;   // among the keys whose high half is H

    // 3. the rows whose high half is H, as codes 2x + half of the lane's
    //    words x, the last four found in h0 and h1
    const uint32_t H2 = H | (H << 16);
    uint32_t h0 = 0u, h1 = 0u;
    int w = 0;
    auto find = [&](uint32_t v, int x) __attribute__((always_inline)) {
        auto hit = [&](uint32_t code) __attribute__((always_inline)) {
            h1 = (h1 << 16) | (h0 >> 16);
            h0 = (h0 << 16) | code;
            ++w;
        };
        if ((v & 0xFFFFu) == 0u) hit((uint32_t)(2 * x));
        if (v < 0x10000u) hit((uint32_t)(2 * x + 1));
    };
#pragma unroll
    for (int x = 0; x < NW; x += 4) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = base[(x + u) * STRIDE] ^ H2;
#pragma unroll
        for (int u = 0; u < 4; u += 2) {
            // a zero half in either word: the minimum of both with 1 is not 1
            if (pk_min_u16(pk_min_u16(v[u], v[u + 1]), 0x00010001u) != 0x00010001u) {
                find(v[u], x + u);
                find(v[u + 1], x + u + 1);
            }
        }
    }
    const int64_t k = column(c);
    const char *col = reinterpret_cast<const char *>(g + (k >= 0 ? k : 0));
    auto low_half = [&](int j) __attribute__((always_inline)) -> uint32_t {
        const int64_t off = row(j);
        // a padding row: the largest key
        if (off < 0) return 0xFFFFu;
        return to_key(*reinterpret_cast<const uint32_t *>(col + off)) & 0xFFFFu;
    };
    uint32_t a, o;
    if (!__any(w > 4)) {
        // 4. bitwise radix select of that rank among the low halves, at most
        //    four a lane (in registers; bit u of act: value u still counts)
        uint32_t lv[4] = {0u, 0u, 0u, 0u};
        uint32_t act = (1u << w) - 1u;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < w) {
                const uint32_t code = ((u < 2 ? h0 : h1) >> (16 * (u & 1))) & 0xFFFFu;
                lv[u] = low_half(half_row<RPI>(gl + (int)(code >> 1) * G, (int)(code & 1u)));
            }
        for (int step = 0; step <= 16; ++step) {
            a = 0xFFFFu;
            o = 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (act >> u & 1u) {
                    a &= lv[u];
                    o |= lv[u];
                }
            a = group_reduce<G, Op::And>(a);
            o = group_reduce<G, Op::Or>(o);
            const uint32_t varying = a ^ o;
            if (varying == 0u) break;
            const uint32_t bit = 1u << (31 - __clz(varying));
            uint32_t zero = 0u;   // values with that bit clear
#pragma unroll
            for (int u = 0; u < 4; ++u) zero |= (lv[u] & bit) == 0u ? 1u << u : 0u;
            const uint32_t zc = group_reduce<G, Op::Add>((uint32_t)__popc(zero & act));
            if (rank < zc) {
                act &= zero;
            } else {
                act &= ~zero;
                rank -= zc;
            }
        }
    } else {
        // more: row numbers, then low halves, in the lane's slots (the write
        // cursor never passes the read cursor)
        uint16_t *base16 = reinterpret_cast<uint16_t *>(base);
        auto slot = [&](int x) __attribute__((always_inline)) -> uint16_t & {
            return base16[(x >> 1) * 2 * STRIDE + (x & 1)];
        };
        w = 0;
        for (int x = 0; x < NW; ++x) {
            const uint32_t v = base[x * STRIDE] ^ H2;
            if ((v & 0xFFFFu) == 0u) slot(w++) = (uint16_t)half_row<RPI>(gl + x * G, 0);
            if (v < 0x10000u) slot(w++) = (uint16_t)half_row<RPI>(gl + x * G, 1);
        }
        constexpr int kGather = 4;   // row reads in flight per lane
        for (int x0 = 0; x0 < w; x0 += kGather) {
            uint32_t v[kGather];
#pragma unroll
            for (int u = 0; u < kGather; ++u)
                if (x0 + u < w) v[u] = low_half(slot(x0 + u));
#pragma unroll
            for (int u = 0; u < kGather; ++u)
                if (x0 + u < w) slot(x0 + u) = (uint16_t)v[u];
        }
        auto and_or = [&]() __attribute__((always_inline)) {
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
        and_or();
        uint32_t varying = a ^ o;
        for (int step = 0; varying != 0u && step < 16; ++step) {
            const uint32_t bit = 1u << (31 - __clz(varying));
            uint32_t zc = 0u;
            for (int x = 0; x < w; ++x) zc += (slot(x) & bit) == 0u;
            zc = group_reduce<G, Op::Add>(zc);
            uint32_t want;
            if (rank < zc) {
                want = 0u;
            } else {
                want = bit;
                rank -= zc;
            }
            int nw = 0;
            for (int x = 0; x < w; ++x) {
                const uint16_t v = slot(x);
                slot(nw) = v;
                nw += (v & bit) == want ? 1 : 0;
            }
            w = nw;
            and_or();
            varying = a ^ o;
        }
    }
    if (gl == 0 && k >= 0) out[k] = __uint_as_float(from_key((H << 16) | a));
}

// One 16-byte load from a replica row that the pass reads once: a
// non-temporal load, which streams past the caches instead of filling them
// with lines nothing reads again (measured 3-6 % faster than a plain load on
// the 61 GB single pass), or (NT false) a plain load, where the lines a row
// segment straddles are read by another workgroup of the XCD as well
// (first_tile).  Any 4-byte alignment: global memory takes a 16-byte access
// at a dword boundary, so rows of any length are read this way (455 files,
// d = 2.5M + 1: 2.50 ms, against 5.63 ms with one 4-byte load a coordinate).
template <bool NT = true>
__device__ __forceinline__ uint4 load_stream(const float *p) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const u32x4 *q = reinterpret_cast<const u32x4 *>(p);
    u32x4 v;
    if constexpr (NT)
        v = __builtin_nontemporal_load(q);
    else
        v = *q;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Load four consecutive coordinates [k, k+4) of one row as bit patterns;
// coordinates at or beyond kend read as 0.
__device__ __forceinline__ void load4(const float *row, int64_t k, int64_t kend, uint32_t v[4]) {
    if (k + 3 < kend) {
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

// The first tile of a workgroup of a persistent grid of G (it takes every
// G-th tile from there).  Workgroups go to the 8 XCDs, each with its own L2,
// in turn, so in workgroup order neighbouring tiles are read by different
// XCDs; by_xcd gives the workgroups of one XCD a run of neighbouring tiles
// instead.  It pays where a row segment of a tile does
// not cover whole 128-byte lines (rows off line boundaries, or tiles of
// fewer than 32 columns): with plain loads the line two neighbouring tiles
// share then comes from the XCD's L2 the second time.  1,330 files, d =
// 1.25M (rows 64 bytes off every other time), 32 columns: 4.28 -> 3.34 ms
// (with non-temporal loads 4.02 ms); 455 files, d = 2.5M + 1, 128 columns:
// 2.50 -> 2.22 ms (2.37).  On whole lines it is slower: 455 files, d =
// 11.2M, 9.21 -> 9.37 ms, and with plain loads 9.99 ms.
__device__ __forceinline__ int64_t first_tile(bool by_xcd) {
    const unsigned b = blockIdx.x, G = gridDim.x;
    if (!by_xcd) return b;
    const unsigned x = b % 8, rest = G % 8;
    return x * (G / 8) + (x < rest ? x : rest) + b / 8;
}

// Column k0 + c of a tile whose lanes read whole 16-byte chunks: the chunk
// holding the end of rows of d coordinates (d >= 4) is read four coordinates
// before the end instead, so its tile columns hold those; -1 past the end.
__device__ __forceinline__ int64_t chunk_start(int64_t k, int64_t d) { return k < d - 4 ? k : d - 4; }
__device__ __forceinline__ int64_t chunk_col(int64_t k0, int c, int64_t d) {
    const int64_t k = k0 + (c & ~3);
    return k < d ? chunk_start(k, d) + (c & 3) : -1;
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
