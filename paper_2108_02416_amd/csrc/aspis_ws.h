// aspis_ws.h -- the warp-specialised kernels (single pass and median), their
// plans, and the tables of the kernels built for each plan, which are spread
// over several sources (aspis_ws_*.hip) that compile in parallel.
#pragma once

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

// sweeps per burst of loads: as many as the streaming role's registers hold
// next to the tile's keys (SW x 4 registers, or SW x 2 with half keys).  The
// 36-sweep tile spills either way; one sweep per burst spills least
template <int R, int SW>
constexpr int ws_batch() { return R == 3 ? (SW > 32 ? 1 : SW > 12 ? 2 : 3) : 1; }

template <int T, int R, int SW, bool IND, bool HALF, int FILL, bool RTG = false>
__global__ void __launch_bounds__(kWsThreads)
fused_ws_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f, int64_t d,
                const int32_t *__restrict__ sel, const int32_t *__restrict__ pos,
                const int32_t *__restrict__ n_sel, int64_t ntiles,
                uint32_t *__restrict__ pair_diff, float *__restrict__ out) {
    extern __shared__ uint32_t smem[];
    constexpr int G = (kWsThreads - FILL) / T;   // selection lanes per column
    constexpr int CPR = T / 4;           // float4 chunks per row segment
    constexpr int RPI = FILL / CPR;      // rows per sweep of the streaming role
    constexpr int B = ws_batch<R, SW>(); // sweeps per burst of loads
    // key registers per sweep: 4 keys, or (HALF) 4 high halves packed in 2;
    // a half-key tile's rows are the files themselves
    constexpr int KW = HALF ? 2 : 4;
    static_assert(!HALF || (SW % 2 == 0 && RPI == half_rpi(T, FILL) && RPI % 8 == 0 && R <= 7),
                  "half-key sweeps");
    // a file's pair-difference bits fit a nibble only at r = 3 (3 bits)
    constexpr bool PDN = HALF && R == 3;
    const int n = *n_sel;
    const int64_t hwords = HALF ? half_hist_words(T) : hist_words(T);
    const int64_t f8 = (f + 7) / 8;
    uint32_t *hist = smem;               // selection histograms
    uint32_t *tile = smem + hwords;
    // per-file words.  Full keys: pd [f] pair-difference bits, ps [f]
    // (tile row << 3) | slot or -1.  Half keys (tile row = file): ps [f/8],
    // one nibble per file, 8 | slot or 0; pd [f/8] pair-difference nibbles
    // at r = 3, else pd [f] words
    uint32_t *pd = tile + (HALF ? half_tile_words(f, T, FILL) : f * T);
    int32_t *ps = reinterpret_cast<int32_t *>(pd + (PDN ? f8 : f));
    // [f*R] row table (IND): staged in LDS, or (RTG) read from global
    // memory, where it stays cached, when LDS is needed for a wider tile
    int32_t *rt_lds = ps + (HALF ? f8 : f);
    const int32_t *rt = RTG ? row_of : rt_lds;
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
        for (int64_t i = tid; i < f * R; i += kWsThreads) rt_lds[i] = row_of[i];
    for (int i = tid; i < hwords; i += kWsThreads) hist[i] = 0u;
    __syncthreads();
    // roles are whole waves: the first FILL/64 waves stream, the rest
    // select; every wave executes the same number of barriers (1 + 2 per
    // tile)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < FILL / 64) {
        const int cq = tid % CPR, j0 = tid / CPR;
        const int64_t sweep = (int64_t)RPI * R * d;   // elements between sweeps
        uint32_t keys[SW][KW];
        // pair-difference bits of the lane's files (sweep x: bits
        // NP*(x % PER) of word x / PER), ORed over every tile in registers
        // and merged into LDS once at the end
        constexpr int NPB = R * (R - 1) / 2;
        constexpr int PER = 32 / NPB;
        uint32_t pdacc[(SW + PER - 1) / PER];
#pragma unroll
        for (int a = 0; a < (SW + PER - 1) / PER; ++a) pdacc[a] = 0u;
        // the r replica chunks of one sweep, kept in registers (a value
        // type, so that no per-lane indexing can turn it into memory)
        struct Chunks {
            uint4 q[R];
        };
        // issue the row loads of sweep x of tile t.  Every load is in bounds:
        // a lane past the end of the rows (tail tile; d % 4 == 0) reads the
        // last chunk of its row instead (a repeated chunk changes neither
        // the agreement bits nor any written median), and a lane past the
        // last file loads nothing (proc_sweep ignores it).
        auto load_sweep = [&](int64_t t, int x) __attribute__((always_inline)) {
            const int64_t col = min(t * T + 4 * cq, d - 4);
            if constexpr (IND) {
                int i = j0 + x * RPI;
                asm volatile("" : "+v"(i));   // row addresses recomputed per tile
                Chunks c;
                if (i < f) {
#pragma unroll
                    for (int s = 0; s < R; ++s)
                        c.q[s] = load_stream(g + (int64_t)rt[i * R + s] * d + col);
                } else {
#pragma unroll
                    for (int s = 0; s < R; ++s) c.q[s] = make_uint4(0u, 0u, 0u, 0u);
                }
                return c;
            }
            const float *base = g + (int64_t)j0 * R * d + col;
            int lim = (int)(f - j0);   // sweeps x with x * RPI < lim hold a file
            // opaque copies of the tile's base address, the limit and the
            // sweep stride: every row address and check below is recomputed
            // from them, instead of the compiler carrying one pointer, one
            // lane mask and one offset per sweep across tiles
            int64_t stride = sweep;
            asm volatile("" : "+v"(base), "+v"(lim), "+s"(stride));
            Chunks c;
            if (x * RPI < lim) {
                const float *rows = base + x * stride;
#pragma unroll
                for (int s = 0; s < R; ++s) c.q[s] = load_stream(rows + s * d);
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
            const int i = j0 + x * RPI;   // f <= C(64,3) here
            if constexpr (HALF) {
                keys[x][0] = 0xFFFFFFFFu;
                keys[x][1] = 0xFFFFFFFFu;
            }
            if (i < f) {
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
                pdacc[x / PER] |= diff << (NPB * (x % PER));
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
                        keys[x][0] = pack_high(to_key(w.x), to_key(w.y));
                        keys[x][1] = pack_high(to_key(w.z), to_key(w.w));
                    }
                } else {
                    keys[x][0] = to_key(w.x);
                    keys[x][1] = to_key(w.y);
                    keys[x][2] = to_key(w.z);
                    keys[x][3] = to_key(w.w);
                }
            }
        };
        // sweep 0 of the next tile, loaded early: before the barrier and the
        // hand-over, so that loads stay in flight meanwhile.  The 36-sweep
        // tile, the row-table reads and r = 5 (five chunks a sweep) have no
        // registers to spare for it and load it with their tile
        constexpr bool kEarly0 = SW <= 32 && !IND && R == 3;
        Chunks c0;
        // tile t from its sweep 0 (already in c0, or loaded first); the
        // other sweeps go in bursts of B, all loads of a burst issued first
        auto stream_rest = [&](int64_t t) __attribute__((always_inline)) {
            if constexpr (!kEarly0) c0 = load_sweep(t, 0);
            proc_sweep(0, c0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int xb = 1; xb < SW; xb += B) {
                Chunks c[B];
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (xb + b < SW) c[b] = load_sweep(t, xb + b);
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (xb + b < SW) proc_sweep(xb + b, c[b]);
                // keep each burst's loads together: no scheduling across
                // bursts, which would hold more loads in registers than fit
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto put_tile = [&]() __attribute__((always_inline)) {
            if constexpr (HALF) {
                // pair-rows j0 + k*RPI of the sweep pairs holding a file
                int64_t fo = f;   // opaque: compared per tile, not held per pair
                asm volatile("" : "+s"(fo));
#pragma unroll
                for (int k = 0; k < SW / 2; ++k)
                    if (k * 2 * RPI < fo)
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
        int64_t t = blockIdx.x;
        if (t < ntiles) {
            if constexpr (kEarly0) c0 = load_sweep(t, 0);
            stream_rest(t);
        }
        if (kEarly0 && t + gridDim.x < ntiles) c0 = load_sweep(t + gridDim.x, 0);
        if (t < ntiles) put_tile();
        __syncthreads();
        for (; t < ntiles; t += gridDim.x) {
            const int64_t tn = t + gridDim.x;
            if (tn < ntiles) stream_rest(tn);
            if (kEarly0 && tn + gridDim.x < ntiles) c0 = load_sweep(tn + gridDim.x, 0);
            __syncthreads();
            if (tn < ntiles) put_tile();
            __syncthreads();
        }
        // the lane's pair-difference bits into the workgroup's words
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
        for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
            if (n > 0) {
                if constexpr (HALF) {
                    // tile row j is file j: its guessed replica's row of g
                    auto row = [&](int j) __attribute__((always_inline)) -> int64_t {
                        const uint32_t q = j < f ? nib(j) : 0u;
                        if (!(q & 8u)) return -1;
                        return IND ? (int64_t)rt[j * R + (q & 7)] : (int64_t)j * R + (q & 7);
                    };
                    select_half_tile<T, G, RPI>(tile, hist, (int)half_pair_rows(f, T, FILL), n,
                                                t * T, d, out, tid - FILL, g, row);
                } else {
                    select_tile<T, G>(tile, hist, n, t * T, d, out, tid - FILL);
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

template <int SW>
constexpr int mws_batch() { return SW >= 16 ? 4 : (SW < 6 ? SW : 6); }

template <int T, int SW, bool HALF, int FILL>
__global__ void __launch_bounds__(kWsThreads)
median_ws_kernel(const float *__restrict__ g, int64_t d, const int32_t *__restrict__ rows,
                 const int32_t *__restrict__ n_sel, int64_t ntiles, float *__restrict__ out,
                 TileMask mask) {
    extern __shared__ uint32_t smem[];
    constexpr int G = (kWsThreads - FILL) / T;   // selection lanes per column
    constexpr int CPR = T / 4;           // float4 chunks per row segment
    constexpr int RPI = FILL / CPR;      // rows per sweep of the streaming role
    constexpr int B = mws_batch<SW>();   // sweeps per burst of loads
    // key registers per sweep: 4 keys, or (HALF) 4 high halves packed in 2
    constexpr int KW = HALF ? 2 : 4;
    static_assert(!HALF || (SW % 2 == 0 && RPI == half_rpi(T, FILL)), "half-key sweeps");
    const int n = *n_sel;
    if (n <= 0) return;                  // uniform: no workgroup reaches a barrier
    const int64_t hwords = HALF ? half_hist_words(T) : hist_words(T);
    uint32_t *hist = smem;
    uint32_t *tile = smem + hwords;
    int32_t *rl = reinterpret_cast<int32_t *>(tile + (HALF ? half_tile_words(n, T, FILL)
                                                           : (int64_t)n * T));   // [n] kept rows
    const int tid = threadIdx.x;
    for (int i = tid; i < n; i += kWsThreads) rl[i] = rows[i];
    for (int i = tid; i < hwords; i += kWsThreads) hist[i] = 0u;
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < FILL / 64) {
        const int cq = tid % CPR, j0 = tid / CPR;
        uint32_t keys[SW][KW];
        // one 16-byte chunk of kept row j (a lane past the last kept row
        // re-reads row 0, which is never put; past the end of the rows it
        // re-reads the row's last chunk, whose median is never written)
        auto load_row = [&](int64_t t, int x) __attribute__((always_inline)) {
            const int64_t col = min(t * T + 4 * cq, d - 4);
            int j = j0 + x * RPI < n ? j0 + x * RPI : 0;
            asm volatile("" : "+v"(j));   // row address recomputed per tile
            return load_stream(g + (int64_t)rl[j] * d + col);
        };
        auto to_keys = [&](int x, uint4 q) __attribute__((always_inline)) {
            if constexpr (HALF) {
                // high key halves; 0xFFFF past the last kept row
                const bool keep = j0 + x * RPI < n;
                keys[x][0] = keep ? pack_high(to_key(q.x), to_key(q.y)) : 0xFFFFFFFFu;
                keys[x][1] = keep ? pack_high(to_key(q.z), to_key(q.w)) : 0xFFFFFFFFu;
            } else {
                keys[x][0] = to_key(q.x);
                keys[x][1] = to_key(q.y);
                keys[x][2] = to_key(q.z);
                keys[x][3] = to_key(q.w);
            }
        };
        uint4 c0;   // sweep 0 of the next tile, loaded early
        auto stream_rest = [&](int64_t t) __attribute__((always_inline)) {
            to_keys(0, c0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int xb = 1; xb < SW; xb += B) {
                uint4 c[B];
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (xb + b < SW) c[b] = load_row(t, xb + b);
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (xb + b < SW) to_keys(xb + b, c[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto put_tile = [&]() __attribute__((always_inline)) {
            if constexpr (HALF) {
                int no = n;   // opaque: compared per tile, not held per pair
                asm volatile("" : "+s"(no));
#pragma unroll
                for (int k = 0; k < SW / 2; ++k) {
                    int p = j0 + k * RPI;
                    // opaque: the LDS addresses are recomputed per tile
                    // instead of being held in registers for every pair
                    asm volatile("" : "+v"(p));
                    if (k * 2 * RPI < no) put_pairs<T, G>(tile, p, cq, keys[2 * k], keys[2 * k + 1]);
                }
            } else {
#pragma unroll
                for (int x = 0; x < SW; ++x) {
                    int j = j0 + x * RPI;
                    asm volatile("" : "+v"(j));   // as above
                    if (j < n) put_keys<T, G>(tile, j, cq, keys[x]);
                }
            }
        };
        // the workgroup's tiles: t, then tn (whose sweep 0 is loaded early)
        const int64_t G0 = gridDim.x;
        int64_t t = mask.next(blockIdx.x, G0, ntiles);
        int64_t tn = mask.next(t + G0, G0, ntiles);
        if (t < ntiles) {
            c0 = load_row(t, 0);
            stream_rest(t);
        }
        if (tn < ntiles) c0 = load_row(tn, 0);
        if (t < ntiles) put_tile();
        __syncthreads();
        while (t < ntiles) {
            const int64_t tnn = mask.next(tn + G0, G0, ntiles);
            if (tn < ntiles) stream_rest(tn);
            if (tnn < ntiles) c0 = load_row(tnn, 0);
            __syncthreads();
            if (tn < ntiles) put_tile();
            __syncthreads();
            t = tn;
            tn = tnn;
        }
    } else {
        __syncthreads();
        for (int64_t t = mask.next(blockIdx.x, gridDim.x, ntiles); t < ntiles;
             t = mask.next(t + gridDim.x, gridDim.x, ntiles)) {
            if constexpr (HALF) {
                auto row = [&](int j) __attribute__((always_inline)) -> int64_t {
                    return j < n ? (int64_t)rl[j] : -1;
                };
                // FILL = 512: RPI = 4G, so every lane holds the same number of
                // words, at most 2 SW
                constexpr int REG = (FILL == kWsFill && RPI == 4 * G) ? 2 * SW : 0;
                select_half_tile<T, G, RPI, REG>(tile, hist, (int)half_pair_rows(n, T, FILL), n,
                                                 t * T, d, out, tid - FILL, g, row);
            } else {
                select_tile<T, G>(tile, hist, n, t * T, d, out, tid - FILL);
            }
            __syncthreads();
            __syncthreads();
        }
    }
}

}  // namespace

// Warp-specialised plans.  Full keys: the widest tile (8..64 columns) whose
// key block fits in LDS and whose rows fit the streaming role's registers
// (at most 16 sweeps of 4 key registers).  Half keys, for many rows: a wider
// tile (16..128 columns) with up to 32 sweeps of 2 key registers; taken
// only when it is wider than the full-key tile, since below kHalfMinRows
// rows a tile is streamed too quickly to hide the reads of the low halves.
// Half keys try the even split of streaming and selecting waves first, then
// 12 streaming waves and 4 selecting ones (kWsFillWide): 1.5x the rows per
// sweep, so that thousands of rows fit the registers of a 32- or 64-column
// tile.
struct WsPlan {
    int r = 3;
    int T = 0;
    int sweeps = 0;
    bool half = false;
    int fill = kWsFill;
    bool rtg = false;   // row table read from global memory (not in LDS)
};

constexpr int kWsFillWide = 768;

// ---------------------------------------------------------------------------
// The kernels built for each plan.  A launcher looks its kernel up here; a
// plan with no entry is a planning error (reported by aspis_plan and the
// launchers alike, never launched).

// a plan's kernel in the tables: tile columns, sweeps, half keys
constexpr int ws_key(int T, int sweeps, bool half) { return T * 1000 + sweeps * 10 + (half ? 1 : 0); }

using FusedWsFn = void (*)(const float *, const int32_t *, int64_t, int64_t, const int32_t *,
                           const int32_t *, const int32_t *, int64_t, uint32_t *, float *);
using MedianWsFn = void (*)(const float *, int64_t, const int32_t *, const int32_t *, int64_t,
                            float *, TileMask);

// nullptr: not built.  fused_ws_fn looks in the family of the plan.
FusedWsFn fused_ws_fn(const WsPlan &p, bool ind);
FusedWsFn fused_ws_r5_fn(const WsPlan &p);                 // r = 5
FusedWsFn fused_ws_r3_fn(const WsPlan &p);                 // r = 3, file-major
FusedWsFn fused_ws_r3_table_fn(const WsPlan &p);           // r = 3, row table
MedianWsFn median_ws_fn(const WsPlan &p);

}  // namespace aspis
