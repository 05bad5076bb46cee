// aspis_ws.h -- the warp-specialised kernels (single pass and median), their
// plans, and the tables of the kernels built for each plan, which are spread
// over several sources (aspis_ws_*.hip) that compile in parallel.
#pragma once

#include <type_traits>

#include "aspis_device.h"

namespace aspis {

namespace {

// ---------------------------------------------------------------------------
// fused agreement + median, warp-specialised: waves 0-7 stream tile t+1 into
// registers (compare the r replicas, keep the guessed replica's keys) while
// waves 8-15 run the selection on tile t in LDS; the keys are handed over
// between two barriers.  The row loads and the selection overlap inside one
// workgroup, so a single [f x T] tile of LDS per CU is enough.

constexpr int kWsThreads = 1024;   // threads of a warp-specialised workgroup
constexpr int kWsFill = 512;       // threads of the streaming role (default split)

// The streaming role's loads run in a ring of B sweeps: a sweep is processed,
// its registers take the load of the sweep B further on (of the next tile
// past the end of this one), so B sweeps of loads are in flight at any time,
// over the hand-over between tiles too.  B divides the sweeps of a tile (a
// sweep's ring place is then the same in every tile) and is as large as the
// registers next to the tile's keys allow.  Measured:
// the file-major single pass is as fast as with bursts of two sweeps (9.20
// ms at 455 files, d = 11.2M, either way); three sweeps there spill 24
// registers (9.32 ms).  Through a row table the ring, the byte offsets
// (ws_offsets) and keys and addresses kept out of registers across sweeps
// take the spills from 27 to none and the pass at 455 files, d = 3M, from
// 2.78 to 2.51 ms (linear read 2.39 ms).
template <int R, int SW, bool HALF>
constexpr int ws_ring() {
    if (R != 3) return R == 5 && SW < 24 && SW % 2 == 0 ? 2 : 1;
    if (SW > 32) return 1;
    if (SW <= (HALF ? 16 : 8) && SW % 4 == 0) return 4;
    return SW <= 24 && SW % 3 == 0 ? 3 : SW % 2 == 0 ? 2 : 1;
}

// Sweeps of loads that stay in flight over the hand-over between two tiles: the
// whole ring, but one sweep for 64-column full-key tiles of 16 sweeps.  There 64
// key registers, the put's addresses and two sweeps of loads spill 21 registers:
// 455 files, d = 11.2M, 10.05 ms, 9.76 with one sweep carried (3 spills), 9.84
// with none and 10.22 with a ring of one; d = 2.5M + 1, 3.02 -> 2.51, d = 3M
// through a row table 2.84 -> 2.74.
// Narrower full-key tiles of 16 sweeps spill 11 to 13 and keep the ring: 2,300
// files on 8 columns, d = 0.3M, 2.37 ms, 2.47 with one carried.
template <int T, int R, int SW, bool HALF>
constexpr int ws_carry() {
    return R == 3 && !HALF && T == 64 && SW == 16 ? 1 : ws_ring<R, SW, HALF>();
}

// Row tables in LDS hold byte offsets (8 bytes a row: a row's address is one
// addition then, no 64-bit product a load) in half-key tiles of 32 columns
// or more, row numbers (4 bytes) where that room would cost tile width.
constexpr bool ws_offsets(int T, bool half) { return half && T >= 32; }

// LDS words before the row table of the single pass: histograms and key tile,
// and the per-file words (half keys: slot nibbles, and pair-difference
// nibbles at r = 3 or words; full keys: two words a file); rounded up to an
// even count
__host__ __device__ constexpr int64_t ws_words_before_table(int64_t f, int r, int T, int sweeps,
                                                            bool half, int fill) {
    const int64_t w = half ? half_tile_words(sweeps, fill) + (f + 7) / 8 + (r == 3 ? (f + 7) / 8 : f)
                           : hist_words(T) + f * (int64_t)T + 2 * f;
    return (w + 1) & ~int64_t{1};
}

// NT: tiles of whole 128-byte lines, non-temporal loads, workgroup order;
// else plain loads, each XCD a run of neighbouring tiles (first_tile).
template <int T, int R, int SW, bool IND, bool HALF, int FILL, bool RTG, bool NT>
__global__ void __launch_bounds__(kWsThreads)
fused_ws_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f, int64_t d,
                const int32_t *__restrict__ sel, const int32_t *__restrict__ pos,
                const int32_t *__restrict__ n_sel, int64_t ntiles,
                uint32_t *__restrict__ pair_diff, float *__restrict__ out, PathGate gate) {
    if (gate.closed()) return;
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int G = (kWsThreads - FILL) / T;   // selection lanes per column
    constexpr int CPR = T / 4;           // float4 chunks per row segment
    constexpr int RPI = FILL / CPR;      // rows per sweep of the streaming role
    constexpr int B = ws_ring<R, SW, HALF>();   // sweeps of loads in flight
    constexpr int CARRY = ws_carry<T, R, SW, HALF>();   // of them over a hand-over
    static_assert(SW % B == 0 && CARRY <= B, "the ring divides the tile");
    // key registers per sweep: 4 keys, or (HALF) 4 high halves packed in 2;
    // a half-key tile's rows are the files themselves
    constexpr int KW = HALF ? 2 : 4;
    static_assert(!HALF || (SW % 2 == 0 && RPI == half_rpi(T, FILL) && RPI % 8 == 0 && R <= 7),
                  "half-key sweeps");
    // a file's pair-difference bits fit a nibble only at r = 3 (3 bits)
    constexpr bool PDN = HALF && R == 3;
    const int n = *n_sel;
    const int64_t hwords = HALF ? 0 : hist_words(T);   // full keys only
    const int64_t f8 = (f + 7) / 8;
    uint32_t *hist = smem;               // selection histograms
    uint32_t *tile = smem + hwords;
    // per-file words.  Full keys: pd [f] pair-difference bits, ps [f]
    // (tile row << 3) | slot or -1.  Half keys (tile row = file): ps [f/8],
    // one nibble per file, 8 | slot or 0; pd [f/8] pair-difference nibbles
    // at r = 3, else pd [f] words
    uint32_t *pd = tile + (HALF ? half_tile_words(SW, FILL) : f * T);
    int32_t *ps = reinterpret_cast<int32_t *>(pd + (PDN ? f8 : f));
    // IND: the row table [f*R], staged in LDS, or (RTG) read from global
    // memory, where it stays cached, when LDS is needed for a wider tile
    constexpr bool OFFS = ws_offsets(T, HALF);
    uint32_t *rt_lds = smem + ws_words_before_table(f, R, T, SW, HALF, FILL);
    // byte offset of the row of replica e = i*R + s
    auto row_offset = [&](int e) __attribute__((always_inline)) -> int64_t {
        if constexpr (RTG) return (int64_t)row_of[e] * d * 4;
        if constexpr (OFFS) return reinterpret_cast<const int64_t *>(rt_lds)[e];
        return (int64_t)(int32_t)rt_lds[e] * d * 4;
    };
    const int tid = threadIdx.x;
    if constexpr (HALF) {
        for (int64_t w = tid; w < f8; w += kWsThreads) {
            uint32_t v = 0u;
            for (int e = 0; e < 8; ++e) {
                const int64_t i = 8 * w + e;
                if (i < f && pos[i] >= 0) v |= (8u | (uint32_t)sel[i]) << (4 * e);
            }
            ps[w] = (int32_t)v;
        }
        for (int64_t w = tid; w < (PDN ? f8 : f); w += kWsThreads) pd[w] = 0u;
    } else {
        for (int64_t i = tid; i < f; i += kWsThreads) {
            pd[i] = 0u;
            ps[i] = pos[i] >= 0 ? (pos[i] << 3) | sel[i] : -1;
        }
    }
    // the slot nibble of file i (HALF): 8 | slot when kept, else 0
    auto nib = [&](int i) __attribute__((always_inline)) {
        return ((uint32_t)ps[i >> 3] >> ((i & 7) * 4)) & 15u;
    };
    if constexpr (IND && !RTG)
        for (int64_t i = tid; i < f * R; i += kWsThreads) {
            if constexpr (OFFS)
                reinterpret_cast<int64_t *>(rt_lds)[i] = (int64_t)row_of[i] * d * 4;
            else
                rt_lds[i] = (uint32_t)row_of[i];
        }
    for (int i = tid; i < hwords; i += kWsThreads) hist[i] = 0u;
    __syncthreads();
    // roles are whole waves: the first FILL/64 waves stream, the rest
    // select; every wave executes the same number of barriers (1 + 2 per
    // tile)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < FILL / 64) {
        const int cq = tid % CPR, j0 = tid / CPR;
        const int64_t sweep = (int64_t)RPI * R * d;   // elements between sweeps
        const int f32 = (int)f;
        uint32_t keys[SW][KW];
        // pair-difference bits of the lane's files.  r = 3 and 5: sweep x's
        // in bits NP*(x % PER) of word x / PER, ORed over every tile in
        // registers and merged into LDS once at the end.  r = 7 (21 bits a
        // file) has no registers for that and adds new bits to the files'
        // LDS words (at r = 5 that is 3 % slower: 462 files, d = 1M, 1.447
        // against 1.400 ms)
        constexpr int NPB = R * (R - 1) / 2;
        constexpr int PER = 32 / NPB;
        uint32_t pdacc[R <= 5 ? (SW + PER - 1) / PER : 1];
        if constexpr (R <= 5)
#pragma unroll
            for (int a = 0; a < (SW + PER - 1) / PER; ++a) pdacc[a] = 0u;
        // the r replica chunks of one sweep, kept in registers (a value
        // type, so that no per-lane indexing can turn it into memory)
        struct Chunks {
            uint4 q[R];
        };
        // issue the row loads of sweep x of tile t.  Every load is in bounds:
        // a lane at or past the end of the rows reads the last four
        // coordinates of its row instead (chunk_col; repeated ones change
        // neither the agreement bits nor any written median), and a lane past
        // the last file loads nothing (proc_sweep ignores it).
        // the lane's chunk of tile t in row 0 (IND) or in its first file's
        // first row
        auto tile_base = [&](int64_t t) __attribute__((always_inline)) -> const float * {
            const int64_t col = chunk_start(t * T + 4 * cq, d);
            return g + (IND ? col : (int64_t)j0 * R * d + col);
        };
        // RTG: the rows of the sweep to be loaded next.  A lane's global loads
        // return in order, so a sweep that read its own rows would wait for
        // every load before it; read one sweep ahead, they are there when the
        // loads before the last sweep are.  2,300 files, d = 0.6M, 3.13 -> 2.80
        // ms a step, d = 2M 10.43 -> 9.29; on another allocation d = 2M 10.07 ->
        // 8.95, with bursts of two and three sweeps 9.51 and 9.10.
        int32_t rows_ahead[RTG ? R : 1];
        auto fetch_rows = [&](int x) __attribute__((always_inline)) {
            int i = j0;
            asm volatile("" : "+v"(i));
            i = min(i + x * RPI, f32 - 1);   // past the last file: in bounds, unused
#pragma unroll
            for (int s = 0; s < R; ++s) rows_ahead[RTG ? s : 0] = row_of[i * R + s];
        };
        auto load_sweep = [&](const float *base, int x) __attribute__((always_inline)) {
            // opaque copies of the lane's first file and the sweep stride:
            // every row address and check below is recomputed from them,
            // instead of the compiler carrying one pointer, one lane mask and
            // one offset per sweep across tiles
            int i = j0;
            int64_t stride = sweep;
            asm volatile("" : "+v"(i), "+s"(stride));
            i += x * RPI;
            Chunks c;
            int32_t row[RTG ? R : 1];
            if constexpr (RTG) {
#pragma unroll
                for (int s = 0; s < R; ++s) row[s] = rows_ahead[s];
                fetch_rows((x + 1) % SW);
            }
            if (i < f32) {
                const float *rows = base + x * stride;
#pragma unroll
                for (int s = 0; s < R; ++s)
                    c.q[s] = load_stream<NT>(
                        RTG   ? base + (int64_t)row[RTG ? s : 0] * d
                        : IND ? reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) +
                                                                row_offset(i * R + s))
                              : rows + s * d);
            } else {
#pragma unroll
                for (int s = 0; s < R; ++s) c.q[s] = make_uint4(0u, 0u, 0u, 0u);
            }
            return c;
        };
        // compare the replicas of sweep x and keep the guessed replica's keys
        // (HALF: its high key halves, packed two to a register, 0xFFFF for a
        // file past the last or dropped)
        auto proc_sweep = [&](int x, Chunks c) __attribute__((always_inline)) {
            const int i = j0 + x * RPI;
            if constexpr (HALF) {
                keys[x][0] = 0xFFFFFFFFu;
                keys[x][1] = 0xFFFFFFFFu;
            }
            if (i < f32) {
                uint32_t diff = 0u;
                int p = 0;
#pragma unroll
                for (int s = 0; s < R; ++s)
#pragma unroll
                    for (int u = s + 1; u < R; ++u) {
                        const uint32_t y = (c.q[s].x ^ c.q[u].x) | (c.q[s].y ^ c.q[u].y) |
                                           (c.q[s].z ^ c.q[u].z) | (c.q[s].w ^ c.q[u].w);
                        diff |= (y != 0u ? 1u : 0u) << p;
                        ++p;
                    }
                if constexpr (R <= 5) {
                    pdacc[x / PER] |= diff << (NPB * (x % PER));
                } else {
                    if (diff & ~pd[i]) atomicOr(&pd[i], diff);
                }
                // HALF: file i's nibble, word (j0 >> 3) + x*RPI/8 (RPI is a
                // multiple of 8), shift (j0 & 7) * 4 in every sweep
                const int w8 = (j0 >> 3) + x * (RPI / 8), sh = (j0 & 7) * 4;
                const int q = HALF ? (int)(((uint32_t)ps[w8] >> sh) & 15u) : ps[i];
                const int s_sel = q & 7;
                uint4 w = c.q[0];
#pragma unroll
                for (int s = 1; s < R; ++s)
                    if (s_sel == s) w = c.q[s];
                if constexpr (HALF) {
                    if (q & 8) {
                        keys[x][0] = pk_high_keys(pack_high(w.x, w.y));
                        keys[x][1] = pk_high_keys(pack_high(w.z, w.w));
                    }
                    // computed here: the compiler would sink it to the put
                    // and hold the loaded words until then
                    asm volatile("" : "+v"(keys[x][0]), "+v"(keys[x][1]));
                } else {
                    keys[x][0] = to_key(w.x);
                    keys[x][1] = to_key(w.y);
                    keys[x][2] = to_key(w.z);
                    keys[x][3] = to_key(w.w);
                }
            }
        };
        Chunks c[B];
        // tile t from the ring, which holds its sweeps [0, held); refilled with
        // t's later sweeps and then with the first CARRY ones of tile tn
        auto stream_tile = [&](int64_t t, int64_t tn, int held) __attribute__((always_inline)) {
            const float *base = tile_base(t);
#pragma unroll
            for (int x = 0; x < B; ++x)
                if (x >= held) c[x] = load_sweep(base, x);
#pragma unroll
            for (int x = 0; x < SW; ++x) {
                proc_sweep(x, c[x % B]);
                __builtin_amdgcn_sched_barrier(0);
                if (x == SW - B) base = tile_base(tn);
                if (x + B < SW || (x + B - SW < CARRY && tn < ntiles))
                    c[x % B] = load_sweep(base, (x + B) % SW);
                // no scheduling across sweeps, which would hold more loads in
                // registers than fit
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto put_tile = [&]() __attribute__((always_inline)) {
            if constexpr (HALF) {
                // pair-rows j0 + k*RPI
#pragma unroll
                for (int k = 0; k < SW / 2; ++k)
                    put_pairs<T, G>(tile, j0 + k * RPI, cq, keys[2 * k], keys[2 * k + 1]);
            } else {
#pragma unroll
                for (int x = 0; x < SW; ++x) {
                    const int i = j0 + x * RPI;
                    if (i < f) {
                        const int q = ps[i];
                        if (q >= 0) put_keys<T, G>(tile, q >> 3, cq, keys[x]);
                    }
                }
            }
        };
        int64_t t = first_tile(!NT);
        if (t < ntiles) {
            if constexpr (RTG) fetch_rows(0);
            stream_tile(t, t + gridDim.x, 0);
            put_tile();
        }
        __syncthreads();
        for (; t < ntiles; t += gridDim.x) {
            const int64_t tn = t + gridDim.x;
            if (tn < ntiles) stream_tile(tn, tn + gridDim.x, CARRY);
            __syncthreads();
            if (tn < ntiles) put_tile();
            __syncthreads();
        }
        // the lane's pair-difference bits into the workgroup's words
        if constexpr (R <= 5)
#pragma unroll
            for (int x = 0; x < SW; ++x) {
                const int i = j0 + x * RPI;
                const uint32_t b = (pdacc[x / PER] >> (NPB * (x % PER))) & ((1u << NPB) - 1u);
                if (i < f && b) {
                    if constexpr (PDN)
                        atomicOr(&pd[i >> 3], b << ((i & 7) * 4));
                    else
                        atomicOr(&pd[i], b);
                }
            }
    } else {
        __syncthreads();
        for (int64_t t = first_tile(!NT); t < ntiles; t += gridDim.x) {
            auto col = [&](int c) __attribute__((always_inline)) { return chunk_col(t * T, c, d); };
            if (n > 0) {
                if constexpr (HALF) {
                    // tile row j is file j: its guessed replica's row of g
                    auto row = [&](int j) __attribute__((always_inline)) -> int64_t {
                        const uint32_t q = j < f ? nib(j) : 0u;
                        if (!(q & 8u)) return -1;
                        if constexpr (IND) return row_offset(j * R + (int)(q & 7));
                        return ((int64_t)j * R + (q & 7)) * d * 4;
                    };
                    select_half_tile<T, G, RPI, RPI / G * SW / 2>(tile, n, out, tid - FILL, g, row, col);
                } else {
                    select_tile<T, G>(tile, hist, n, out, tid - FILL, col);
                }
            }
            __syncthreads();
            __syncthreads();
        }
    }
    __syncthreads();
    for (int64_t i = tid; i < f; i += kWsThreads) {
        const uint32_t b = PDN ? ((pd[i >> 3] >> ((i & 7) * 4)) & 15u) : pd[i];
        if (b) atomicOr(&pair_diff[i], b);
    }
}

// ---------------------------------------------------------------------------
// median of the kept rows, warp-specialised like fused_ws_kernel: waves 0-7
// stream the kept rows of tile t+1 (one row per kept file, through the row
// list of the selection) into registers while waves 8-15 select on tile t.
// Used by the two-pass path and after a wrong guess of the single pass.
// Its loads are plain ones: 455 kept files, d = 1.5M, 625 us, against 641 with
// non-temporal ones; by_xcd as in the single pass (first_tile).

// the ring of the streaming role's loads (ws_ring), one 16-byte load a
// sweep: six sweeps (10 measured 1 % slower at 455 kept files)
template <int SW, bool HALF>
constexpr int mws_ring() {
    constexpr int cap = (128 - 28 - SW * (HALF ? 2 : 4)) / 4;
    constexpr int most = HALF ? 6 : 4;
    for (int b = cap < most ? cap : most; b > 1; --b)
        if (SW % b == 0) return b;
    return 1;
}

template <int T, int SW, bool HALF>
__global__ void __launch_bounds__(kWsThreads)
median_ws_kernel(const float *__restrict__ g, int64_t d, const int32_t *__restrict__ rows,
                 const int32_t *__restrict__ n_sel, int64_t ntiles, bool by_xcd,
                 float *__restrict__ out, TileMask mask) {
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int FILL = kWsFill;        // threads of the streaming role
    constexpr int G = (kWsThreads - FILL) / T;   // selection lanes per column
    constexpr int CPR = T / 4;           // float4 chunks per row segment
    constexpr int RPI = FILL / CPR;      // rows per sweep of the streaming role
    constexpr int B = mws_ring<SW, HALF>();   // sweeps of loads in flight
    // key registers per sweep: 4 keys, or (HALF) 4 high halves packed in 2
    constexpr int KW = HALF ? 2 : 4;
    static_assert(!HALF || (SW % 2 == 0 && RPI == half_rpi(T, FILL)), "half-key sweeps");
    const int n = *n_sel;
    if (n <= 0) return;                  // uniform: no workgroup reaches a barrier
    const int64_t hwords = HALF ? 0 : hist_words(T);   // full keys only
    uint32_t *hist = smem;
    uint32_t *tile = smem + hwords;
    // [n] kept rows (ws_offsets; the words before them: an even count)
    using Row = std::conditional_t<ws_offsets(T, HALF), int64_t, int32_t>;
    constexpr bool OFFS = ws_offsets(T, HALF);
    Row *rl = reinterpret_cast<Row *>(tile + (HALF ? half_tile_words(SW, FILL) : (int64_t)n * T));
    auto row_offset = [&](int j) __attribute__((always_inline)) -> int64_t {
        return OFFS ? (int64_t)rl[j] : (int64_t)rl[j] * d * 4;
    };
    const int tid = threadIdx.x;
    for (int i = tid; i < n; i += kWsThreads) rl[i] = OFFS ? (Row)((int64_t)rows[i] * d * 4) : (Row)rows[i];
    for (int i = tid; i < hwords; i += kWsThreads) hist[i] = 0u;
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < FILL / 64) {
        const int cq = tid % CPR, j0 = tid / CPR;
        uint32_t keys[SW][KW];
        // one 16-byte chunk of a kept row (a lane past the last kept row
        // re-reads that row, which is never put again; past the end of the
        // rows it re-reads the row's last chunk, whose median is never
        // written)
        auto load_row = [&](int64_t t, int x) __attribute__((always_inline)) {
            const int64_t col = chunk_start(t * T + 4 * cq, d);
            int j = j0;
            asm volatile("" : "+v"(j));   // offsets read per tile, not held
            j = min(j + x * RPI, n - 1);
            return load_stream<false>(reinterpret_cast<const float *>(
                reinterpret_cast<const char *>(g + col) + row_offset(j)));
        };
        auto to_keys = [&](int x, uint4 q) __attribute__((always_inline)) {
            if constexpr (HALF) {
                // high key halves; 0xFFFF past the last kept row
                const bool keep = j0 + x * RPI < n;
                keys[x][0] = keep ? pk_high_keys(pack_high(q.x, q.y)) : 0xFFFFFFFFu;
                keys[x][1] = keep ? pk_high_keys(pack_high(q.z, q.w)) : 0xFFFFFFFFu;
                // computed here: the compiler would sink it to the put and
                // hold the four loaded words until then
                asm volatile("" : "+v"(keys[x][0]), "+v"(keys[x][1]));
            } else {
                keys[x][0] = to_key(q.x);
                keys[x][1] = to_key(q.y);
                keys[x][2] = to_key(q.z);
                keys[x][3] = to_key(q.w);
            }
        };
        uint4 c[B];
        auto stream_tile = [&](int64_t t, int64_t tn) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < SW; ++x) {
                to_keys(x, c[x % B]);
                __builtin_amdgcn_sched_barrier(0);
                if (x + B < SW)
                    c[x % B] = load_row(t, x + B);
                else if (tn < ntiles)
                    c[x % B] = load_row(tn, x + B - SW);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto put_tile = [&]() __attribute__((always_inline)) {
            if constexpr (HALF) {
#pragma unroll
                for (int k = 0; k < SW / 2; ++k)
                    put_pairs<T, G>(tile, j0 + k * RPI, cq, keys[2 * k], keys[2 * k + 1]);
            } else {
#pragma unroll
                for (int x = 0; x < SW; ++x) {
                    int j = j0 + x * RPI;
                    asm volatile("" : "+v"(j));   // as above
                    if (j < n) put_keys<T, G>(tile, j, cq, keys[x]);
                }
            }
        };
        // the workgroup's tiles: t, then tn (whose first sweeps are loaded
        // before the hand-over of t), then tnn
        const int64_t G0 = gridDim.x;
        int64_t t = mask.next(first_tile(by_xcd), G0, ntiles);
        int64_t tn = mask.next(t + G0, G0, ntiles);
        if (t < ntiles) {
#pragma unroll
            for (int x = 0; x < B; ++x) c[x] = load_row(t, x);
            stream_tile(t, tn);
            put_tile();
        }
        __syncthreads();
        while (t < ntiles) {
            const int64_t tnn = mask.next(tn + G0, G0, ntiles);
            if (tn < ntiles) stream_tile(tn, tnn);
            __syncthreads();
            if (tn < ntiles) put_tile();
            __syncthreads();
            t = tn;
            tn = tnn;
        }
    } else {
        __syncthreads();
        for (int64_t t = mask.next(first_tile(by_xcd), gridDim.x, ntiles); t < ntiles;
             t = mask.next(t + gridDim.x, gridDim.x, ntiles)) {
            auto col = [&](int c) __attribute__((always_inline)) { return chunk_col(t * T, c, d); };
            if constexpr (HALF) {
                auto row = [&](int j) __attribute__((always_inline)) -> int64_t {
                    return j < n ? row_offset(j) : -1;
                };
                select_half_tile<T, G, RPI, RPI / G * SW / 2>(tile, n, out, tid - FILL, g, row, col);
            } else {
                select_tile<T, G>(tile, hist, n, out, tid - FILL, col);
            }
            __syncthreads();
            __syncthreads();
        }
    }
}

}  // namespace

// Warp-specialised plans.  Full keys: the widest tile (8..64 columns) whose
// key block fits in LDS and whose rows fit the streaming role's registers
// (at most 16 sweeps of 4 key registers).  Half keys: a wider tile (16..128
// columns) with up to 36 sweeps of 2 key registers, taken only when it is wider
// than the full-key tile, from kHalfMinRows rows on (the single pass at r = 3 in
// long vectors: from kHalfFewRows).  The single pass's half keys try the even
// split of streaming and selecting waves first, then 12 streaming waves and 4
// selecting ones (kWsFillWide): 1.5x the rows per sweep, so that thousands of
// rows fit the registers of a 32- or 64-column tile.
struct WsPlan {
    int r = 3;
    int T = 0;
    int sweeps = 0;
    bool half = false;
    int fill = kWsFill;
    bool rtg = false;   // row table read from global memory (not in LDS)
    // row segments of whole 128-byte lines (the single pass's NT)
    bool lines = true;
};

constexpr int kWsFillWide = 768;

// ---------------------------------------------------------------------------
// The kernels built for each plan.  A launcher looks its kernel up here; a
// plan with no entry is a planning error (reported by aspis_plan and the
// launchers alike, never launched).

// a plan's kernel in the tables: tile columns, sweeps, half keys
constexpr int ws_key(int T, int sweeps, bool half) { return T * 1000 + sweeps * 10 + (half ? 1 : 0); }

// the kernel of plan p for tiles of whole 128-byte lines or not
#define ASPIS_NT(kernel, ...) (p.lines ? &kernel<__VA_ARGS__, true> : &kernel<__VA_ARGS__, false>)

using FusedWsFn = void (*)(const float *, const int32_t *, int64_t, int64_t, const int32_t *,
                           const int32_t *, const int32_t *, int64_t, uint32_t *, float *,
                           PathGate);
using MedianWsFn = void (*)(const float *, int64_t, const int32_t *, const int32_t *, int64_t,
                            bool, float *, TileMask);

// nullptr: not built.  fused_ws_fn looks in the family of the plan.
FusedWsFn fused_ws_fn(const WsPlan &p, bool ind);
FusedWsFn fused_ws_r5_fn(const WsPlan &p, bool ind);       // r = 5
FusedWsFn fused_ws_r7_fn(const WsPlan &p, bool ind);       // r = 7
FusedWsFn fused_ws_r3_fn(const WsPlan &p);                 // r = 3, file-major
FusedWsFn fused_ws_r3_table_fn(const WsPlan &p);           // r = 3, row table
MedianWsFn median_ws_fn(const WsPlan &p);

}  // namespace aspis
