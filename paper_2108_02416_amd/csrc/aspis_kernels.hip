// aspis_kernels.hip -- gfx950 kernels of the Aspis detect-and-aggregate step.
//
// The replicas are float32 rows of d coordinates: row (i,s) holds the
// gradient the worker in slot s returned for file i, either at row i*r+s of
// a file-major [f][r][d] tensor or through a row table (the workers' own
// [K][l][d] uploads).  Everything here is integer work on the 32-bit
// patterns (bitwise comparison, order-preserving keys) except the fp64 sums
// of the mean, so nothing is a dense contraction and no MFMA is used; the
// kernels are bound by HBM reads.
//
//   agree_kernel       Eq. (4): per file, OR over coordinates of "slot pair p
//                      differs"; one coalesced stream over the r rows.
//   probe_kernel       the same over the probe's blocks, with the tie probe
//                      (agree_file_kernel and tie_probe_kernel: each alone).
//   guess_kernel       the probe's votes, clique search and selection, and
//                      the reduction it calls for, in one workgroup.
//   vote_kernel        Eq. (3) majority per file and the K x K disagreement
//                      rows (Section 4: edge iff the pair agrees on all
//                      common files).
//   vote_rows_kernel   the same in one workgroup, rows built in LDS and
//                      staged for the host (the single pass).
//   select_kernel      Algorithm 1 selection (Case 1 honest replica / Case 2
//                      majority) and the ordered list of kept rows.
//   median_kernel      Algorithm 1 Case 2 coordinate-wise median: a tile of T
//                      coordinates x all kept rows is staged in LDS as
//                      totalOrder keys, and each column's lower median is
//                      found by G lanes of one wave (select_tile: one LDS
//                      histogram round, then a bitwise radix finish).
//   median_ws_kernel   the same median, warp-specialised like the single
//                      pass (two-pass path, and the rerun after a wrong guess).
//   fused_ws_kernel    agreement + median in one read, warp-specialised: some
//                      waves stream the next tile while the others select on
//                      the current one (the headline path).  Where it gives a
//                      wider tile, the LDS tile keeps only the high 16 bits of
//                      each key (select_half_tile); the low halves of the rows
//                      that tie with the median's high half are read back.
//   fused_kernel       agreement + median in one read, load then select per
//                      tile, where no warp-specialised plan exists (rows of
//                      fewer than four coordinates, more files than its tiles
//                      hold, full keys of more than 128 files at r = 5 and 7).
//   fused_mean_kernel  agreement + Case 1 mean in one read.
//   mean_kernel        Algorithm 1 Case 1 mean, fp64 accumulation in file
//                      order.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "aspis_guess.h"
#include "aspis_ws.h"

namespace aspis {

namespace {

// ---------------------------------------------------------------------------
// utility kernels

__global__ void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void fill_u64_kernel(uint64_t *p, int64_t n, uint64_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// agreement: Eq. (4) for every file and slot pair, over coordinates [0,kend)

constexpr int kAgreeUnroll = 4;                       // float4 per thread
constexpr int64_t kAgreeChunk = (int64_t)kBlock * 4 * kAgreeUnroll;

template <int R>
__global__ void __launch_bounds__(kBlock)
agree_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f,
             int64_t d, int64_t kend, int64_t nchunks, uint32_t *__restrict__ pair_diff) {
    const int64_t nwork = f * nchunks;
    for (int64_t w = blockIdx.x; w < nwork; w += gridDim.x) {
        const int64_t i = w / nchunks;
        const int64_t chunk = w - i * nchunks;
        const float *rows[R];
#pragma unroll
        for (int s = 0; s < R; ++s) rows[s] = g + replica_row(row_of, i, R, s) * d;
        uint32_t diff = 0u;
#pragma unroll
        for (int u = 0; u < kAgreeUnroll; ++u) {
            const int64_t k = chunk * kAgreeChunk + (int64_t)u * kBlock * 4 +
                              (int64_t)threadIdx.x * 4;
            if (k < kend) {
                uint32_t v[R][4];
#pragma unroll
                for (int s = 0; s < R; ++s) load4(rows[s], k, kend, v[s]);
                int p = 0;
#pragma unroll
                for (int s = 0; s < R; ++s)
#pragma unroll
                    for (int t = s + 1; t < R; ++t) {
                        const uint32_t x = (v[s][0] ^ v[t][0]) | (v[s][1] ^ v[t][1]) |
                                           (v[s][2] ^ v[t][2]) | (v[s][3] ^ v[t][3]);
                        diff |= (x != 0u ? 1u : 0u) << p;
                        ++p;
                    }
            }
        }
        // OR over the wave; one atomic per wave only when something differs
        uint32_t wdiff = 0u;
        constexpr int P = R * (R - 1) / 2;
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (__ballot((diff >> p) & 1u)) wdiff |= 1u << p;
        // the word already holds the bits after the first chunks of a file
        // that differs: read it first, so that the other chunks' waves of
        // that file do not all queue atomics on one address
        if ((threadIdx.x & 63) == 0 && wdiff && (wdiff & ~__atomic_load_n(&pair_diff[i], __ATOMIC_RELAXED)))
            atomicOr(&pair_diff[i], wdiff);
    }
}

// Agreement of file i over blocks first, first + step, ... of the probe, by
// one workgroup: returns the file's bits there to thread 0.
template <int R>
__device__ __forceinline__ uint32_t probe_agreement(const float *g, const int32_t *row_of, int64_t i,
                                                    int64_t d, const ProbeSet &probe, int64_t first,
                                                    int64_t step) {
    static_assert(kProbeBlockCols == kBlock * 4, "one float4 per thread and probe block");
    __shared__ uint32_t wave_bits[kBlock / 64];
    constexpr int P = R * (R - 1) / 2;
    const float *rows[R];
#pragma unroll
    for (int s = 0; s < R; ++s) rows[s] = g + replica_row(row_of, i, R, s) * d;
    uint32_t diff = 0u;
    for (int64_t j0 = first; j0 < probe.nb; j0 += kAgreeUnroll * step) {
        uint32_t v[kAgreeUnroll][R][4];
#pragma unroll
        for (int u = 0; u < kAgreeUnroll; ++u) {
            // block j0 + u*step: the thread's four coordinates (none past its end)
            int64_t k = 0, kend = 0;
            if (j0 + u * step < probe.nb) {
                const int64_t b = probe.block_start(j0 + u * step);
                k = b + (int64_t)threadIdx.x * 4;
                kend = probe.block_end(b);
            }
#pragma unroll
            for (int s = 0; s < R; ++s) {
                if (k < kend)
                    load4(rows[s], k, kend, v[u][s]);
                else
                    v[u][s][0] = v[u][s][1] = v[u][s][2] = v[u][s][3] = 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < kAgreeUnroll; ++u) {
            int p = 0;
#pragma unroll
            for (int s = 0; s < R; ++s)
#pragma unroll
                for (int t = s + 1; t < R; ++t) {
                    const uint32_t x = (v[u][s][0] ^ v[u][t][0]) | (v[u][s][1] ^ v[u][t][1]) |
                                       (v[u][s][2] ^ v[u][t][2]) | (v[u][s][3] ^ v[u][t][3]);
                    diff |= (x != 0u ? 1u : 0u) << p;
                    ++p;
                }
        }
    }
    uint32_t wdiff = 0u;
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (__ballot((diff >> p) & 1u)) wdiff |= 1u << p;
    if ((threadIdx.x & 63) == 0) wave_bits[threadIdx.x >> 6] = wdiff;
    __syncthreads();
    uint32_t bits = 0u;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) bits |= wave_bits[w];
    }
    __syncthreads();
    return bits;
}

// Agreement over the probed coordinates, one file per workgroup: stores the
// file's word, so pair_diff needs no zero fill and no atomics.
template <int R>
__global__ void __launch_bounds__(kBlock)
agree_file_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f,
                  int64_t d, ProbeSet probe, uint32_t *__restrict__ pair_diff) {
    for (int64_t i = blockIdx.x; i < f; i += gridDim.x) {
        const uint32_t b = probe_agreement<R>(g, row_of, i, d, probe, 0, 1);
        if (threadIdx.x == 0) pair_diff[i] = b;
    }
}

// ---------------------------------------------------------------------------
// vote and disagreement rows

// Eq. (3) for one file from its pair-difference word: the lowest slot of the
// largest class of bitwise-equal replicas and that class's size.  Calls
// differ(s, t) for every slot pair whose replicas differ.
template <int R, typename DiffFn>
__device__ __forceinline__ void file_vote(uint32_t pd, int *vote_slot, int *class_size,
                                          DiffFn differ) {
    // same[s] = bitmask of slots whose replica equals slot s's
    uint32_t same[R];
#pragma unroll
    for (int s = 0; s < R; ++s) same[s] = 1u << s;
    int p = 0;
#pragma unroll
    for (int s = 0; s < R; ++s)
#pragma unroll
        for (int t = s + 1; t < R; ++t, ++p) {
            if (pd >> p & 1u) {
                differ(s, t);
            } else {
                same[s] |= 1u << t;
                same[t] |= 1u << s;
            }
        }
    int best = 0, best_n = 0;
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const int c = __popc(same[s]);
        if (c > best_n) {
            best_n = c;
            best = s;
        }
    }
    *vote_slot = best;
    *class_size = best_n;
}

template <int R>
__global__ void vote_kernel(const uint32_t *__restrict__ pair_diff,
                            const int32_t *__restrict__ subsets, int64_t f,
                            int8_t *__restrict__ vote,
                            uint8_t *__restrict__ has_majority,
                            uint64_t *__restrict__ disagree) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < f;
         i += (int64_t)gridDim.x * blockDim.x) {
        int best = 0, best_n = 0;
        file_vote<R>(pair_diff[i], &best, &best_n, [&](int s, int t) {
            const int us = subsets[i * R + s], ut = subsets[i * R + t];
            atomicOr((unsigned long long *)&disagree[us], 1ull << ut);
            atomicOr((unsigned long long *)&disagree[ut], 1ull << us);
        });
        vote[i] = (int8_t)best;
        has_majority[i] = (uint8_t)(best_n >= (R + 1) / 2);
    }
}

// The same in one workgroup, for the single pass (f is at most a few
// thousand there): the K rows are built in LDS and stored whole (no zero
// fill), and a copy goes to stage[0..K) for the host, with stage[64] = 1 if
// any file's vote differs from the one vote[] held before the call.  sel_out,
// when not NULL, receives a copy of sel (the guessed selection, which the
// host finds to be the final one in nearly every step).
template <int R>
__global__ void __launch_bounds__(1024)
vote_rows_kernel(const uint32_t *__restrict__ pair_diff, const int32_t *__restrict__ subsets,
                 int64_t f, int K, int8_t *__restrict__ vote,
                 uint8_t *__restrict__ has_majority, uint64_t *__restrict__ disagree,
                 uint64_t *__restrict__ stage, const int32_t *__restrict__ sel,
                 int32_t *__restrict__ sel_out) {
    __shared__ unsigned long long rows[64];
    __shared__ int changed;
    const int tid = threadIdx.x;
    if (tid < 64) rows[tid] = 0ull;
    if (tid == 0) changed = 0;
    __syncthreads();
    for (int64_t i = tid; i < f; i += blockDim.x) {
        int best = 0, best_n = 0;
        file_vote<R>(pair_diff[i], &best, &best_n, [&](int s, int t) {
            const int us = subsets[i * R + s], ut = subsets[i * R + t];
            atomicOr(&rows[us], 1ull << ut);
            atomicOr(&rows[ut], 1ull << us);
        });
        if (sel_out) sel_out[i] = sel[i];
        if (vote[i] != (int8_t)best) changed = 1;
        vote[i] = (int8_t)best;
        has_majority[i] = (uint8_t)(best_n >= (R + 1) / 2);
    }
    __syncthreads();
    if (tid < K) {
        disagree[tid] = rows[tid];
        stage[tid] = rows[tid];
    }
    if (tid == 0) stage[64] = (uint64_t)changed;
}

// ---------------------------------------------------------------------------
// selection (one workgroup of 1024 threads; f is at most a few thousand)

__device__ __forceinline__ void select_files(const int32_t *subsets, const int8_t *vote, int64_t f,
                                             int r, int success, uint64_t honest,
                                             const int32_t *row_of, int32_t *sel, int32_t *pos,
                                             int32_t *rows, int32_t *n_sel, int32_t *sel_out) {
    __shared__ int wave_tot[16];
    __shared__ int carry;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int64_t b = 0; b < f; b += 1024) {
        const int64_t i = b + tid;
        int s = -1;
        if (i < f) {
            if (success) {
                for (int x = 0; x < r; ++x)
                    if (honest >> subsets[i * r + x] & 1ull) {
                        s = x;
                        break;
                    }
            } else {
                s = vote[i];
            }
        }
        const bool keep = s >= 0;
        const uint64_t bal = __ballot(keep);
        const int in_wave = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wave_tot[wave] = __popcll(bal);
        __syncthreads();
        int before = carry;
        for (int w = 0; w < wave; ++w) before += wave_tot[w];
        if (i < f) {
            const int p = keep ? before + in_wave : -1;
            sel[i] = s;
            pos[i] = p;
            if (sel_out) sel_out[i] = s;
            if (keep) rows[p] = row_of ? row_of[i * r + s] : (int32_t)(i * r + s);
        }
        __syncthreads();
        if (tid == 0) {
            int tot = 0;
            for (int w = 0; w < 16; ++w) tot += wave_tot[w];
            carry += tot;
        }
        __syncthreads();
    }
    if (tid == 0) *n_sel = carry;
}

__global__ void __launch_bounds__(1024)
select_kernel(const int32_t *__restrict__ subsets,
              const int8_t *__restrict__ vote, int64_t f, int r,
              int success, uint64_t honest, const int32_t *__restrict__ row_of,
              int32_t *__restrict__ sel, int32_t *__restrict__ pos, int32_t *__restrict__ rows,
              int32_t *__restrict__ n_sel, int32_t *__restrict__ sel_out,
              uint32_t *__restrict__ zero, int64_t n_zero) {
    if (zero)
        for (int64_t i = threadIdx.x; i < n_zero; i += 1024) zero[i] = 0u;
    select_files(subsets, vote, f, r, success, honest, row_of, sel, pos, rows, n_sel, sel_out);
}

// ---------------------------------------------------------------------------
// the guess of the single pass, on the device: the host's clique search
// would cost the step a copy, a synchronisation and a launch before its main
// kernel can start

// The operations of guess_clique by one wave, whose 64 lanes all run in step:
// lane u holds the workers that disagree with worker u (0 from K on) and, at
// lane d, the open branch of depth d.  Everything else is the same in every
// lane, so it stays in scalar registers.
struct GuessWave {
    uint32_t dis, stack, lane;
    __device__ void pairs(uint32_t C, uint32_t bits[5]) const {
        const uint32_t n = (C >> (lane & 31u)) & 1u ? (uint32_t)__popc(C & dis) : 0u;
#pragma unroll
        for (int b = 0; b < 5; ++b) bits[b] = (uint32_t)__ballot((n >> b) & 1u);
    }
    __device__ uint32_t against(int v) const {
        return (uint32_t)__builtin_amdgcn_readlane((int)dis, v);
    }
    __device__ void push(int depth, uint32_t C) {
        stack = lane == (uint32_t)depth ? C : stack;
    }
    __device__ uint32_t pop(int depth) const {
        return (uint32_t)__builtin_amdgcn_readlane((int)stack, depth);
    }
};

// The probe's outcome in one workgroup: votes and disagreement rows from the
// files' partial words (split: how many a file has, file i's at part[s*f +
// i]), the clique search, the guessed selection into the workspace, the
// reduction the guess calls for (path_out, a kPath value), and pair_diff zeroed
// for the main pass.  stage: as vote_rows_kernel's, without the flag;
// stage[kStageGuess] = success | path << 8, stage[kStageGuess + 1] = the
// honest mask.
template <int R>
__global__ void __launch_bounds__(1024)
guess_kernel(const uint32_t *__restrict__ part, int split, const int32_t *__restrict__ subsets,
             int64_t f, int K, int need, int mode, int keys,
             const uint32_t *__restrict__ tie_counts, int n_tie,
             const int32_t *__restrict__ row_of, int8_t *__restrict__ vote,
             uint8_t *__restrict__ has_majority, uint64_t *__restrict__ disagree,
             uint64_t *__restrict__ stage, uint32_t *__restrict__ pair_diff,
             int32_t *__restrict__ sel, int32_t *__restrict__ pos, int32_t *__restrict__ rows,
             int32_t *__restrict__ n_sel, int32_t *__restrict__ path_out) {
    __shared__ unsigned long long dis_rows[64];
    __shared__ int success;
    __shared__ uint64_t honest;
    const int tid = threadIdx.x;
    if (tid < 64) dis_rows[tid] = 0ull;
    __syncthreads();
    for (int64_t i = tid; i < f; i += 1024) {
        uint32_t pd = 0u;
        for (int s = 0; s < split; ++s) pd |= part[(int64_t)s * f + i];
        int best = 0, best_n = 0;
        file_vote<R>(pd, &best, &best_n, [&](int s, int t) {
            const int us = subsets[i * R + s], ut = subsets[i * R + t];
            atomicOr(&dis_rows[us], 1ull << ut);
            atomicOr(&dis_rows[ut], 1ull << us);
        });
        vote[i] = (int8_t)best;
        has_majority[i] = (uint8_t)(best_n >= (R + 1) / 2);
        pair_diff[i] = 0u;
    }
    __syncthreads();
    if (tid < 64) {
        const uint64_t dis = dis_rows[tid];
        if (tid < K) {
            disagree[tid] = dis;
            stage[tid] = dis;
        }
        GuessWave wave{tid < K ? (uint32_t)dis : 0u, 0u, (uint32_t)tid};
        uint32_t h = 0u;
        const bool ok = guess_clique(wave, K, need, &h);
        // the tie estimate: the mean count, rounded up
        uint32_t full = keys == kKeysFull ? 1u : 0u;
        if (keys == kKeysProbe) {
            const uint32_t sum = group_reduce<64, Op::Add>(tid < n_tie ? tie_counts[tid] : 0u);
            full = (sum + (uint32_t)n_tie - 1u) / (uint32_t)n_tie >= kTieFullKeys ? 1u : 0u;
        }
        const bool mean = mode == kModeMean || (mode == kModePaper && ok);
        const int path = mean ? kPathMean : full ? kPathFullKeys : kPathHalfKeys;
        if (tid == 0) {
            success = ok ? 1 : 0;
            honest = h;
            *path_out = path;
            stage[kStageGuess] = (uint64_t)(ok ? 1 : 0) | (uint64_t)path << 8;
            stage[kStageGuess + 1] = h;
        }
    }
    __syncthreads();
    select_files(subsets, vote, f, R, success, honest, row_of, sel, pos, rows, n_sel, nullptr);
}

// Row of every replica in a worker-major upload: replica (i,s) is row u*l + k
// of worker u = slot s's worker, i the k-th file of u.  The files holding u,
// u taken out, are the (r-1)-subsets of the K-1 others in lexicographic
// order, so k is the rank of file i's other workers among those.
__global__ void __launch_bounds__(kBlock)
worker_rows_kernel(int K, int r, int64_t f, int32_t *__restrict__ row_of) {
    __shared__ uint32_t binom[64][8];   // C(n, k); C(63, 7) fits 32 bits
    for (int e = threadIdx.x; e < 64 * 8; e += kBlock) {
        const int n = e / 8, k = e % 8;
        uint64_t v = k <= n ? 1u : 0u;
        for (int j = 0; j < k && k <= n; ++j) v = v * (uint64_t)(n - j) / (uint64_t)(j + 1);
        binom[n][k] = (uint32_t)v;
    }
    __syncthreads();
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i >= f) return;
    // file i's workers: the subset of rank i
    int c[8];
    int64_t rest = i;
    int u = 0;
    for (int s = 0; s < r; ++s, ++u) {
        // subsets whose next worker is u
        for (; rest >= (int64_t)binom[K - 1 - u][r - 1 - s]; ++u) rest -= binom[K - 1 - u][r - 1 - s];
        c[s] = u;
    }
    const int64_t l = binom[K - 1][r - 1];
    for (int s = 0; s < r; ++s) {
        int64_t k = 0;
        int next = 0;   // the least label the next worker may have
        for (int t = 0, m = 0; t < r; ++t) {
            if (t == s) continue;
            const int w = c[t] - (t > s ? 1 : 0);   // label without worker c[s]
            for (int x = next; x < w; ++x) k += binom[K - 2 - x][r - 2 - m];
            next = w + 1;
            ++m;
        }
        row_of[i * r + s] = (int32_t)(c[s] * l + k);
    }
}

// ---------------------------------------------------------------------------
// median of the kept rows

constexpr int kMedianBatch = 8;   // row loads per thread issued as one burst

template <int T>
__global__ void __launch_bounds__(tile_block<T>())
median_kernel(const float *__restrict__ g, int64_t d,
              const int32_t *__restrict__ rows, const int32_t *__restrict__ n_sel,
              int64_t ntiles, float *__restrict__ out, TileMask mask) {
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int BLOCK = tile_block<T>();
    uint32_t *hist = smem;
    uint32_t *tile = smem + hist_words(T);
    constexpr int G = BLOCK / T;
    constexpr int CPR = T / 4;           // float4 chunks per row segment
    constexpr int RPI = BLOCK / CPR;     // rows filled per sweep
    const int n = *n_sel;
    if (n <= 0) return;
    const int tid = threadIdx.x;
    for (int i = tid; i < hist_words(T); i += BLOCK) hist[i] = 0u;
    const int cq = tid % CPR, j0 = tid / CPR;
    for (int64_t t = mask.next(blockIdx.x, gridDim.x, ntiles); t < ntiles;
         t = mask.next(t + gridDim.x, gridDim.x, ntiles)) {
        const int64_t k0 = t * T;
        auto col = [&](int c) { return k0 + c < d ? k0 + c : (int64_t)-1; };
        for (int jb = 0; jb < n; jb += RPI * kMedianBatch) {
            uint32_t v[kMedianBatch][4];
#pragma unroll
            for (int b = 0; b < kMedianBatch; ++b) {
                const int j = jb + b * RPI + j0;
                if (j < n) load4(g + (int64_t)rows[j] * d, k0 + 4 * cq, d, v[b]);
            }
#pragma unroll
            for (int b = 0; b < kMedianBatch; ++b) {
                const int j = jb + b * RPI + j0;
                if (j < n) {
                    uint32_t k[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) k[e] = to_key(v[b][e]);
                    put_keys<T, G>(tile, j, cq, k);
                }
            }
        }
        __syncthreads();
        select_tile<T, G>(tile, hist, n, out, tid, col);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// fused agreement + median (one read of all r replicas)

template <int R>
constexpr int fused_batch() { return R == 3 ? 4 : (R == 5 ? 2 : 1); }

template <int T, int R>
__global__ void __launch_bounds__(tile_block<T>())
fused_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f, int64_t d,
             const int32_t *__restrict__ sel, const int32_t *__restrict__ pos,
             const int32_t *__restrict__ n_sel, int64_t ntiles,
             uint32_t *__restrict__ pair_diff, float *__restrict__ out, PathGate gate) {
    if (gate.closed()) return;
    extern __shared__ __align__(16) uint32_t smem[];
    constexpr int BLOCK = tile_block<T>();
    constexpr int G = BLOCK / T;
    constexpr int CPR = T / 4;
    constexpr int RPI = BLOCK / CPR;
    constexpr int B = fused_batch<R>();
    const int n = *n_sel;
    uint32_t *hist = smem;
    uint32_t *tile = smem + hist_words(T);
    uint32_t *pd = tile + f * T;         // [f] per-workgroup pair-difference bits
    const int tid = threadIdx.x;
    for (int64_t i = tid; i < f; i += BLOCK) pd[i] = 0u;
    for (int i = tid; i < hist_words(T); i += BLOCK) hist[i] = 0u;
    __syncthreads();
    const int cq = tid % CPR, j0 = tid / CPR;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t k0 = t * T;
        auto col = [&](int c) { return k0 + c < d ? k0 + c : (int64_t)-1; };
        for (int64_t ib = 0; ib < f; ib += (int64_t)RPI * B) {
            uint32_t v[B][R][4];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int64_t i = ib + b * RPI + j0;
                if (i < f) {
#pragma unroll
                    for (int s = 0; s < R; ++s)
                        load4(g + replica_row(row_of, i, R, s) * d, k0 + 4 * cq, d, v[b][s]);
                }
            }
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int64_t i = ib + b * RPI + j0;
                if (i >= f) continue;
                uint32_t diff = 0u;
                int p = 0;
#pragma unroll
                for (int s = 0; s < R; ++s)
#pragma unroll
                    for (int u = s + 1; u < R; ++u) {
                        const uint32_t x = (v[b][s][0] ^ v[b][u][0]) | (v[b][s][1] ^ v[b][u][1]) |
                                           (v[b][s][2] ^ v[b][u][2]) | (v[b][s][3] ^ v[b][u][3]);
                        diff |= (x != 0u ? 1u : 0u) << p;
                        ++p;
                    }
                if (diff) atomicOr(&pd[i], diff);
                const int j = pos[i];
                if (j >= 0) {
                    const int s_sel = sel[i];
                    uint32_t w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        w[e] = v[b][0][e];
#pragma unroll
                        for (int s = 1; s < R; ++s) w[e] = (s_sel == s) ? v[b][s][e] : w[e];
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = to_key(w[e]);
                    put_keys<T, G>(tile, j, cq, w);
                }
            }
        }
        __syncthreads();
        if (n > 0) select_tile<T, G>(tile, hist, n, out, tid, col);
        __syncthreads();
    }
    for (int64_t i = tid; i < f; i += BLOCK)
        if (pd[i]) atomicOr(&pair_diff[i], pd[i]);
}

// ---------------------------------------------------------------------------
// fused agreement + mean (one read of all r replicas): each thread owns four
// coordinates and walks every file in ascending order, comparing the r
// replicas and adding the guessed replica to an fp64 sum -- the file order
// of the sum is the mean kernel's and the oracle's.  A wave reads 1 KiB of
// one row per load.  The pair-difference bits of a wave are combined with
// ballots into per-workgroup LDS words, merged into pair_diff at the end.

// Bound by HBM.  A lane's loads run in a ring of B files (a file is processed,
// its registers take the load of the file B further on), so that few waves
// keep the memory busy: 455 files, d = 1M 0.97 -> 0.85 ms, d = 0.2M 0.71 ->
// 0.20 ms (linear reads 0.77 and 0.17); 462 files at r = 5, d = 4M 6.83 -> 5.82
// ms; 120 files at r = 7, d = 0.4M 0.55 -> 0.23 ms, all against bursts of
// loads waited for together.  At r = 3 those bursts (62 registers, 8
// workgroups per CU) stay where the vector gives each CU at least 5 and at
// most 8 workgroups, which then run as one full round.  Kernel times of bursts
// and ring at 35, 120, 455 and 1,140 files, both layouts: d = 1.31M to 2.09M (5
// to 8 workgroups) bursts 1 to 12 % faster (455 files, d = 1.6M, 1.29 against
// 1.41 ms); d = 1.06M and 1,234,567 (4 to 5) ring 1 to 6 % faster (1,140 files, d =
// 1.06M, 2.45 against 2.61 ms), d = 1.15M within 2 % either way.
constexpr int64_t kMeanBurstMin = 5, kMeanBurstMax = 8;   // workgroups per CU

// IND: rows through the table row_of.  SHORT: rows of fewer than four
// coordinates.
template <int R, int B, bool IND, bool SHORT>
__global__ void __launch_bounds__(kBlock)
fused_mean_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f,
                  int64_t d, const int32_t *__restrict__ sel, const int32_t *__restrict__ n_sel,
                  uint32_t *__restrict__ pair_diff, float *__restrict__ out, PathGate gate) {
    if (gate.closed()) return;
    extern __shared__ uint32_t pdw[];   // [f]
    const int tid = threadIdx.x;
    const int nf = (int)f;
    for (int i = tid; i < nf; i += kBlock) pdw[i] = 0u;
    __syncthreads();
    const int n = *n_sel;
    const int64_t nq = (d + 3) / 4;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    // every lane of a workgroup runs the same iterations (the ballots need
    // whole waves); a lane at or past the end of the rows reads their last
    // four coordinates
    for (int64_t q0 = (int64_t)blockIdx.x * kBlock; q0 < nq; q0 += stride) {
        const int64_t k = (q0 + tid) * 4;
        const int64_t col = SHORT ? 0 : chunk_start(k, d);
        const float *at = g + col;
        struct Chunks {
            uint4 q[R];
        };
        auto load_file = [&](int i) __attribute__((always_inline)) {
            Chunks c;
#pragma unroll
            for (int s = 0; s < R; ++s) {
                const float *row = at + (IND ? (int64_t)row_of[i * R + s] : (int64_t)i * R + s) * d;
                if constexpr (SHORT) {
                    uint32_t v[4];
                    load4(row, 0, d, v);
                    c.q[s] = make_uint4(v[0], v[1], v[2], v[3]);
                } else {
                    c.q[s] = load_stream(row);
                }
            }
            return c;
        };
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        Chunks c[B];
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (b < nf) c[b] = load_file(b);
        for (int ib = 0; ib < nf; ib += B) {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int i = ib + b;
                if (i >= nf) break;
                uint32_t wdiff = 0u;   // of the wave
                int p = 0;
#pragma unroll
                for (int s = 0; s < R; ++s)
#pragma unroll
                    for (int u = s + 1; u < R; ++u) {
                        const uint4 x = c[b].q[s], y = c[b].q[u];
                        const uint32_t z = (x.x ^ y.x) | (x.y ^ y.y) | (x.z ^ y.z) | (x.w ^ y.w);
                        if (__ballot(z != 0u)) wdiff |= 1u << p;
                        ++p;
                    }
                if ((tid & 63) == 0 && wdiff) atomicOr(&pdw[i], wdiff);
                const int s_sel = sel[i];
                if (s_sel >= 0) {
                    uint4 w = c[b].q[0];
#pragma unroll
                    for (int s = 1; s < R; ++s)
                        if (s_sel == s) w = c[b].q[s];
                    acc[0] += (double)__uint_as_float(w.x);
                    acc[1] += (double)__uint_as_float(w.y);
                    acc[2] += (double)__uint_as_float(w.z);
                    acc[3] += (double)__uint_as_float(w.w);
                }
                // each ring place refilled before the next file is processed
                __builtin_amdgcn_sched_barrier(0);
                if (i + B < nf) c[b] = load_file(i + B);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (k < d && n > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < d) out[col + e] = (float)(acc[e] / (double)n);
        }
    }
    __syncthreads();
    for (int i = tid; i < nf; i += kBlock)
        if (pdw[i]) atomicOr(&pair_diff[i], pdw[i]);
}

// The same at r = 3 in bursts of three files (R rows each), all loads of a burst
// issued first: 62 VGPRs, 8 workgroups per CU.
constexpr int kMeanFiles = 3;

template <int R>
__global__ void __launch_bounds__(kBlock)
fused_mean_burst_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f,
                  int64_t d, const int32_t *__restrict__ sel, const int32_t *__restrict__ pos,
                  const int32_t *__restrict__ n_sel, uint32_t *__restrict__ pair_diff,
                  float *__restrict__ out, PathGate gate) {
    if (gate.closed()) return;
    extern __shared__ uint32_t pdw[];   // [f]
    const int tid = threadIdx.x;
    for (int64_t i = tid; i < f; i += kBlock) pdw[i] = 0u;
    __syncthreads();
    const int n = *n_sel;
    const int64_t nq = (d + 3) / 4;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    // every lane of a workgroup runs the same iterations (the ballots need
    // whole waves); lanes past the end of the rows read and write nothing
    for (int64_t q0 = (int64_t)blockIdx.x * kBlock; q0 < nq; q0 += stride) {
        const int64_t k = (q0 + tid) * 4;
        const int64_t kend = q0 + tid < nq ? d : 0;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        for (int64_t ib = 0; ib < f; ib += kMeanFiles) {
            uint32_t v[kMeanFiles][R][4];
#pragma unroll
            for (int b = 0; b < kMeanFiles; ++b) {
                const int64_t i = ib + b;
                if (i < f) {
#pragma unroll
                    for (int s = 0; s < R; ++s)
                        load4(g + replica_row(row_of, i, R, s) * d, k, kend, v[b][s]);
                }
            }
#pragma unroll
            for (int b = 0; b < kMeanFiles; ++b) {
                const int64_t i = ib + b;
                if (i >= f) break;
                uint32_t diff = 0u;
                int p = 0;
#pragma unroll
                for (int s = 0; s < R; ++s)
#pragma unroll
                    for (int u = s + 1; u < R; ++u) {
                        const uint32_t x = (v[b][s][0] ^ v[b][u][0]) | (v[b][s][1] ^ v[b][u][1]) |
                                           (v[b][s][2] ^ v[b][u][2]) | (v[b][s][3] ^ v[b][u][3]);
                        diff |= (x != 0u ? 1u : 0u) << p;
                        ++p;
                    }
                uint32_t wdiff = 0u;
#pragma unroll
                for (int q = 0; q < R * (R - 1) / 2; ++q)
                    if (__ballot((diff >> q) & 1u)) wdiff |= 1u << q;
                if ((tid & 63) == 0 && wdiff) atomicOr(&pdw[i], wdiff);
                if (pos[i] >= 0) {
                    const int s_sel = sel[i];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t w = v[b][0][e];
#pragma unroll
                        for (int s = 1; s < R; ++s) w = (s_sel == s) ? v[b][s][e] : w;
                        acc[e] += (double)__uint_as_float(w);
                    }
                }
            }
        }
        if (kend != 0 && n > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + e < d) out[k + e] = (float)(acc[e] / (double)n);
        }
    }
    __syncthreads();
    for (int64_t i = tid; i < f; i += kBlock)
        if (pdw[i]) atomicOr(&pair_diff[i], pdw[i]);
}

// ---------------------------------------------------------------------------
// mean of the kept rows (fp64, file order)

constexpr int kMeanRows = 8;
constexpr int64_t kMeanTileCols = kBlock * 4;   // coordinates per mean tile: four per thread

__global__ void __launch_bounds__(kBlock)
mean_kernel(const float *__restrict__ g, int64_t d,
            const int32_t *__restrict__ rows, const int32_t *__restrict__ n_sel,
            float *__restrict__ out, TileMask mask) {
    const int n = *n_sel;
    if (n <= 0) return;
    // tiles of kMeanTileCols coordinates, four per thread
    const int64_t ntiles = (d + kMeanTileCols - 1) / kMeanTileCols;
    for (int64_t t = mask.next(blockIdx.x, gridDim.x, ntiles); t < ntiles;
         t = mask.next(t + gridDim.x, gridDim.x, ntiles)) {
        const int64_t k = t * kMeanTileCols + 4 * (int64_t)threadIdx.x;
        if (k >= d) continue;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        // bursts of kMeanRows loads, then the additions in row order
        for (int j0 = 0; j0 < n; j0 += kMeanRows) {
            uint32_t v[kMeanRows][4];
#pragma unroll
            for (int b = 0; b < kMeanRows; ++b)
                if (j0 + b < n) load4(g + (int64_t)rows[j0 + b] * d, k, d, v[b]);
#pragma unroll
            for (int b = 0; b < kMeanRows; ++b)
                if (j0 + b < n) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] += (double)__uint_as_float(v[b][e]);
                }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k + e < d) out[k + e] = (float)(acc[e] / (double)n);
    }
}

// ---------------------------------------------------------------------------
// median of any number of kept rows: an MSB-first radix select over the
// 32-bit keys in four rounds of 8 bits, whose histograms live in LDS while
// the keys are read from HBM again in every round.  It takes over when not
// even a narrow tile of every kept row's keys fits in LDS (beyond about
// 10,000 kept files); it reads the kept rows four times, trading bandwidth
// for capacity.  Lane c of every wave owns column c of a 64-column tile and
// wave w reads rows w, w + 4, ... (256-byte row segments per wave load).

constexpr int kRadixCols = 64;
constexpr int kRadixThreads = 256;
constexpr int kRadixWaves = kRadixThreads / kRadixCols;
constexpr int kRadixBuckets = 256;
constexpr int kRadixStride = kRadixBuckets + 1;   // bucket b of column c at c*257 + b:
                                                  // bank (c + b) % 64
constexpr int kRadixBatch = 8;                    // row loads in flight per lane
constexpr int kRadixQuarter = kRadixBuckets / kRadixWaves;

__global__ void __launch_bounds__(kRadixThreads)
median_radix_kernel(const float *__restrict__ g, int64_t d, const int32_t *__restrict__ rows,
                    const int32_t *__restrict__ n_sel, int64_t ntiles, float *__restrict__ out,
                    TileMask mask) {
    __shared__ uint32_t hist[kRadixCols * kRadixStride];
    __shared__ uint32_t part[kRadixWaves][kRadixCols];   // bucket counts per quarter
    __shared__ uint32_t prefix[kRadixCols], rank[kRadixCols];
    const int n = *n_sel;
    if (n <= 0) return;   // uniform: no workgroup reaches a barrier
    const int tid = threadIdx.x, c = tid % kRadixCols, w = tid / kRadixCols;
    for (int64_t t = mask.next(blockIdx.x, gridDim.x, ntiles); t < ntiles;
         t = mask.next(t + gridDim.x, gridDim.x, ntiles)) {
        const int64_t k = t * kRadixCols + c;
        const bool valid = k < d;
        if (tid < kRadixCols) {
            prefix[tid] = 0u;
            rank[tid] = (uint32_t)(n - 1) / 2;
        }
        // round x settles key bits [24 - 8x, 32 - 8x) among the keys whose
        // higher bits equal the prefix settled so far
        for (int round = 0; round < 4; ++round) {
            for (int i = tid; i < kRadixCols * kRadixStride; i += kRadixThreads) hist[i] = 0u;
            __syncthreads();
            const int sh = 24 - 8 * round;
            const uint32_t pre = prefix[c];
            uint32_t *hc = hist + c * kRadixStride;
            auto count = [&](uint32_t v) __attribute__((always_inline)) {
                const uint32_t key = to_key(v);
                if (round == 0 || (key >> (sh + 8)) == pre) atomicAdd(&hc[(key >> sh) & 255u], 1u);
            };
            if (valid) {
                const float *col = g + k;
                int j = w;
                for (; j + (kRadixBatch - 1) * kRadixWaves < n; j += kRadixBatch * kRadixWaves) {
                    uint32_t v[kRadixBatch];
#pragma unroll
                    for (int u = 0; u < kRadixBatch; ++u)
                        v[u] = __float_as_uint(col[(int64_t)rows[j + u * kRadixWaves] * d]);
#pragma unroll
                    for (int u = 0; u < kRadixBatch; ++u) count(v[u]);
                }
                for (; j < n; j += kRadixWaves) count(__float_as_uint(col[(int64_t)rows[j] * d]));
            }
            __syncthreads();
            // the bucket holding the sought rank: wave w sums its quarter of
            // the column's buckets, then one lane per column walks the
            // quarters and the buckets of the quarter that holds it
            uint32_t sum = 0u;
#pragma unroll 8
            for (int b = 0; b < kRadixQuarter; ++b) sum += hc[w * kRadixQuarter + b];
            part[w][c] = sum;
            __syncthreads();
            if (tid < kRadixCols) {
                uint32_t m = rank[c], run = 0u;
                int qt = 0;
                for (; qt < kRadixWaves - 1; ++qt) {
                    if (run + part[qt][c] > m) break;
                    run += part[qt][c];
                }
                int b = qt * kRadixQuarter;
                for (; b < (qt + 1) * kRadixQuarter - 1; ++b) {
                    if (run + hc[b] > m) break;
                    run += hc[b];
                }
                rank[c] = m - run;
                prefix[c] = (prefix[c] << 8) | (uint32_t)b;
            }
            __syncthreads();
        }
        if (w == 0 && valid) out[k] = __uint_as_float(from_key(prefix[c]));
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// tie probe: how many values share the median's high 16 key bits.  The
// half-key tiles read back the low halves of every row tied with the
// median's high half, so heavily tied data (quantised gradients, values on
// a grid) is better served by full-key tiles.  For kTieCols coordinates
// spread over the probed prefix, one workgroup takes each file's value at
// that coordinate -- the value of its largest class of equal replicas, the
// file's vote on that coordinate alone, which is what the selection keeps
// in most files -- finds the high half H of their lower median (two
// 8-bit histogram rounds in LDS) and stores how many files have high half
// H.  It needs no selection, so it runs with the probe.

constexpr int kTieThreads = 256;

// Probed coordinate c (c < min(kTieCols, probe.coords())): the prefix
// split in kTieCols equal steps, or offsets spread over the blocks.
__device__ __forceinline__ int64_t tie_coord(const ProbeSet &probe, int c) {
    if (probe.seed == 0) {
        const int64_t kstep = probe.kend >= kTieCols ? probe.kend / kTieCols : 1;
        return (int64_t)c * kstep;
    }
    const int64_t per = (kTieCols + probe.nb - 1) / probe.nb;   // coordinates per block
    const int64_t step = kProbeBlockCols / per;
    return probe.block_start(c % probe.nb) + (c / probe.nb) * step;
}
constexpr int kTieMaxFiles = 4096;   // files looked at per coordinate (the first ones)
static_assert(kTieThreads == 256, "one histogram bucket per thread");

template <int R>
__device__ __forceinline__ void tie_count(const float *g, const int32_t *row_of, int64_t f, int64_t d,
                                          const ProbeSet &probe, int coord, uint32_t *out) {
    __shared__ uint16_t h[kTieMaxFiles];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t wsum[kTieThreads / 64];
    __shared__ uint32_t pick[2];   // bucket, rank within it
    const int tid = threadIdx.x;
    const int64_t k = tie_coord(probe, coord);
    const int n = (int)(f < kTieMaxFiles ? f : kTieMaxFiles);
    for (int i = tid; i < n; i += kTieThreads) {
        uint32_t v[R];
#pragma unroll
        for (int s = 0; s < R; ++s) v[s] = __float_as_uint(g[replica_row(row_of, i, R, s) * d + k]);
        // the value of the largest class of equal replicas, the lower slot
        // on a tie (Eq. (3) on this one coordinate)
        uint32_t val = v[0];
        int best = 0;
#pragma unroll
        for (int s = 0; s < R; ++s) {
            int c = 0;
#pragma unroll
            for (int t = 0; t < R; ++t) c += v[s] == v[t] ? 1 : 0;
            if (c > best) {
                best = c;
                val = v[s];
            }
        }
        h[i] = (uint16_t)(to_key(val) >> 16);
    }
    // round 0 counts the high bytes; round 1 the low bytes of the keys whose
    // high byte is the median's; the median's bucket count then is the number
    // of files tied with it
    uint32_t rank = (uint32_t)(n - 1) / 2, hi = 0u;
    for (int round = 0; round < 2; ++round) {
        hist[tid] = 0u;   // kTieThreads == 256 buckets
        __syncthreads();
        for (int i = tid; i < n; i += kTieThreads) {
            const uint32_t x = h[i];
            if (round == 0)
                atomicAdd(&hist[x >> 8], 1u);
            else if ((x >> 8) == hi)
                atomicAdd(&hist[x & 255u], 1u);
        }
        __syncthreads();
        // the bucket holding the rank: a prefix sum over the 256 buckets,
        // one per thread (wave scans, then the waves' totals)
        const uint32_t c = hist[tid];
        uint32_t incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
            incl += (tid & 63) >= o ? y : 0u;
        }
        if ((tid & 63) == 63) wsum[tid >> 6] = incl;
        __syncthreads();
        for (int w = 0; w < (tid >> 6); ++w) incl += wsum[w];
        if (incl - c <= rank && rank < incl) {   // exactly one bucket
            pick[0] = (uint32_t)tid;
            pick[1] = rank - (incl - c);
        }
        __syncthreads();
        const uint32_t b = pick[0];
        if (round == 0) {
            hi = b;
            rank = pick[1];
        } else if (tid == 0) {
            out[coord] = hist[b];
        }
        __syncthreads();
    }
}

template <int R>
__global__ void __launch_bounds__(kTieThreads)
tie_probe_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f,
                 int64_t d, ProbeSet probe, uint32_t *__restrict__ out) {
    tie_count<R>(g, row_of, f, d, probe, (int)blockIdx.x, out);
}

// The whole probe in one launch: workgroups [0, f*split) compare file b % f
// over every split-th block of the probe (from block b / f on) into part[b],
// the rest run the tie probe.  A file alone leaves a small cluster's probe to
// a few workgroups: K = 7, d = 0.1M, 29 us without the split, 13 us with it and
// the guess (guess_kernel).
template <int R>
__global__ void __launch_bounds__(kBlock)
probe_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f, int split,
             int64_t d, ProbeSet probe, uint32_t *__restrict__ part, uint32_t *__restrict__ tie_out) {
    static_assert(kTieThreads == kBlock, "one workgroup size");
    const int64_t b = blockIdx.x, n = f * split;
    if (b < n) {
        const uint32_t bits = probe_agreement<R>(g, row_of, b % f, d, probe, b / f, split);
        if (threadIdx.x == 0) part[b] = bits;
    } else {
        tie_count<R>(g, row_of, f, d, probe, (int)(b - n), tie_out);
    }
}

// ---------------------------------------------------------------------------
// repair after a wrong guess (the guess kept the same files as the final
// selection and reduced them with the same median): the median computed with
// the guess already is the final one wherever each moved file's two
// replicas are equal, so only the tiles holding a coordinate where they
// differ are recomputed.

__global__ void save_sel_kernel(const int32_t *__restrict__ sel, int64_t f,
                                int8_t *__restrict__ sel_prev, int32_t *__restrict__ repair) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < f) sel_prev[i] = (int8_t)sel[i];
    if (i < 4) repair[i] = 0;
}

constexpr int kDirtyMaxMoved = 2048;   // moved files a workgroup lists (LDS)
constexpr int kDirtyBatch = 4;         // moved files per burst of loads

// Every workgroup lists the moved files (replica rows of the guess and of the
// final selection, where the two differ somewhere in the vector), then sets
// the bits of its words: bit b of word w for the columns [b' << cshift,
// (b' + 1) << cshift), b' = 32w + b, when a listed pair differs there --
// every bit when the kept files differ or more files moved than the list
// holds.
template <int R>
__global__ void __launch_bounds__(kBlock)
dirty_tiles_kernel(const float *__restrict__ g, const int32_t *__restrict__ row_of, int64_t f,
                   int64_t d, int cshift, int64_t nbits,
                   const int8_t *__restrict__ sel_prev, const int32_t *__restrict__ sel,
                   const uint32_t *__restrict__ pair_diff, uint32_t *__restrict__ dirty,
                   int32_t *__restrict__ repair) {
    __shared__ int32_t moved[2 * kDirtyMaxMoved];
    __shared__ int32_t n_moved, every;
    __shared__ uint32_t word;
    const int tid = threadIdx.x;
    if (tid == 0) {
        n_moved = 0;
        every = 0;
        word = 0u;
    }
    __syncthreads();
    for (int64_t i = tid; i < f; i += kBlock) {
        const int a = sel_prev[i], b = sel[i];
        if ((a < 0) != (b < 0)) {
            atomicOr(&every, 1);
            continue;
        }
        if (a < 0 || a == b) continue;
        // bit of the slot pair (lo, hi) in the pair-difference word
        const int lo = a < b ? a : b, hi = a < b ? b : a;
        const int p = lo * (2 * R - lo - 1) / 2 + (hi - lo - 1);
        if (((pair_diff[i] >> p) & 1u) == 0u) continue;   // bitwise equal replicas
        const int x = atomicAdd(&n_moved, 1);
        if (x < kDirtyMaxMoved) {
            moved[2 * x] = (int32_t)replica_row(row_of, i, R, a);
            moved[2 * x + 1] = (int32_t)replica_row(row_of, i, R, b);
        } else {
            atomicOr(&every, 1);
        }
    }
    __syncthreads();
    const bool all = every != 0;
    const int n = n_moved < kDirtyMaxMoved ? n_moved : kDirtyMaxMoved;
    const int64_t nwords = (nbits + 31) / 32;
    for (int64_t w = blockIdx.x; w < nwords; w += gridDim.x) {
        const int64_t nb = nbits - 32 * w < 32 ? nbits - 32 * w : 32;
        const uint32_t full = nb == 32 ? 0xFFFFFFFFu : (1u << nb) - 1u;
        if (all) {
            if (tid == 0) {
                dirty[w] = full;
                atomicAdd(&repair[0], __popc(full));
            }
            continue;
        }
        const int64_t c0 = (w * 32) << cshift;
        const int64_t c1 = c0 + (nb << cshift) < d ? c0 + (nb << cshift) : d;
        uint32_t mine = 0u;
        for (int64_t k = c0 + 4 * tid; k < c1; k += 4 * kBlock) {
            const uint32_t bit = 1u << ((k - c0) >> cshift);
            if (mine & bit) continue;
            for (int x0 = 0; x0 < n; x0 += kDirtyBatch) {
                uint32_t va[kDirtyBatch][4], vb[kDirtyBatch][4];
#pragma unroll
                for (int u = 0; u < kDirtyBatch; ++u) {
                    if (x0 + u < n) {
                        load4(g + (int64_t)moved[2 * (x0 + u)] * d, k, d, va[u]);
                        load4(g + (int64_t)moved[2 * (x0 + u) + 1] * d, k, d, vb[u]);
                    }
                }
                uint32_t diff = 0u;
#pragma unroll
                for (int u = 0; u < kDirtyBatch; ++u)
                    if (x0 + u < n)
                        diff |= (va[u][0] ^ vb[u][0]) | (va[u][1] ^ vb[u][1]) |
                                (va[u][2] ^ vb[u][2]) | (va[u][3] ^ vb[u][3]);
                if (diff != 0u) {
                    mine |= bit;
                    break;
                }
            }
        }
        if (mine) atomicOr(&word, mine);
        __syncthreads();
        if (tid == 0) {
            dirty[w] = word;
            atomicAdd(&repair[0], __popc(word));
            word = 0u;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// read-bandwidth probe

constexpr int kProbeBlocks = 2048;

__global__ void __launch_bounds__(kBlock)
read_probe_kernel(const uint4 *__restrict__ p, int64_t n16, uint32_t *sink) {
    uint32_t acc = 0u;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint4 v = load_stream(reinterpret_cast<const float *>(p + i));
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    sink[blockIdx.x * (int64_t)blockDim.x + threadIdx.x] = acc;
}

// Compute units of each device, looked up once per device (relaxed atomics:
// concurrent first calls store the same value).
constexpr int kMaxDevices = 64;
std::atomic<int> g_num_cus[kMaxDevices];

int num_cus() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
    int cus = g_num_cus[dev].load(std::memory_order_relaxed);
    if (cus == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        g_num_cus[dev].store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// Row segments of T columns cover whole 128-byte lines: no line is shared by
// neighbouring tiles.
bool whole_lines(const float *g, int64_t d, int T) {
    return (uintptr_t)g % 128 == 0 && d % 32 == 0 && T % 32 == 0;
}

int64_t grid_for(int64_t work, int64_t cap) { return work < cap ? (work < 1 ? 1 : work) : cap; }

// widest tile T whose [rows x T] key block (plus extra bytes) fits in LDS
int pick_tile(int64_t rows, int64_t extra_bytes) {
    for (int T : {64, 32, 16, 8, 4})
        if (rows * 4 * (int64_t)T + hist_words(T) * 4 + extra_bytes <= kLdsBytes) return T;
    return 0;
}

// workgroups per CU that the LDS allows, for the grid of a tile kernel
int64_t tile_grid(int64_t ntiles, size_t lds) {
    int per_cu = (int)(kLdsBytes / (int64_t)(lds ? lds : 1));
    per_cu = per_cu < 1 ? 1 : (per_cu > 2 ? 2 : per_cu);
    return grid_for(ntiles, (int64_t)num_cus() * per_cu);
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers

// sel, pos, rows: int32 [f] each; 256 bytes of counters; 1,024 bytes of
// staged rows; the row table int32 [f*r].  Each part starts 256-aligned.
constexpr size_t kWsCounters = 256, kWsStage = 1024;

size_t workspace_bytes(int64_t f, int r) {
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    return up((size_t)f * 4) * 3 + kWsCounters + kWsStage + up((size_t)f * r * 4) + up((size_t)f) +
           (size_t)kDirtyWords * 4 + kWsCounters;
}

Workspace carve_workspace(void *base, int64_t f, int r) {
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    char *p = static_cast<char *>(base);
    Workspace w;
    w.sel = reinterpret_cast<int32_t *>(p);
    p += up((size_t)f * 4);
    w.pos = reinterpret_cast<int32_t *>(p);
    p += up((size_t)f * 4);
    w.rows = reinterpret_cast<int32_t *>(p);
    p += up((size_t)f * 4);
    w.n_sel = reinterpret_cast<int32_t *>(p);
    p += kWsCounters;
    w.stage = reinterpret_cast<uint64_t *>(p);
    p += kWsStage;
    w.row_of = reinterpret_cast<int32_t *>(p);
    p += up((size_t)f * r * 4);
    w.sel_prev = reinterpret_cast<int8_t *>(p);
    p += up((size_t)f);
    w.dirty = reinterpret_cast<uint32_t *>(p);
    p += (size_t)kDirtyWords * 4;
    w.repair = reinterpret_cast<int32_t *>(p);
    return w;
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    fill_u32_kernel<<<(unsigned)grid_for((n + 255) / 256, 1024), 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}
hipError_t launch_fill_u64(uint64_t *p, int64_t n, uint64_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    fill_u64_kernel<<<(unsigned)grid_for((n + 255) / 256, 1024), 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_agree(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                        int64_t kend, uint32_t *pair_diff, hipStream_t s) {
    if (kend <= 0 || f <= 0) return hipSuccess;
    const int64_t nchunks = (kend + kAgreeChunk - 1) / kAgreeChunk;
    const unsigned grid = (unsigned)grid_for(f * nchunks, (int64_t)num_cus() * 16);
#define ASPIS_AGREE(RR) \
    agree_kernel<RR><<<grid, kBlock, 0, s>>>(g, row_of, f, d, kend, nchunks, pair_diff);
    switch (r) {
    case 3: ASPIS_AGREE(3) break;
    case 5: ASPIS_AGREE(5) break;
    case 7: ASPIS_AGREE(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_AGREE
    return hipGetLastError();
}

hipError_t launch_vote(const uint32_t *pair_diff, const int32_t *subsets, int64_t f,
                       int r, int8_t *vote, uint8_t *has_majority, uint64_t *disagree,
                       hipStream_t s) {
    const unsigned grid = (unsigned)grid_for((f + 255) / 256, 64);
#define ASPIS_VOTE(RR) \
    vote_kernel<RR><<<grid, 256, 0, s>>>(pair_diff, subsets, f, vote, has_majority, disagree);
    switch (r) {
    case 3: ASPIS_VOTE(3) break;
    case 5: ASPIS_VOTE(5) break;
    case 7: ASPIS_VOTE(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_VOTE
    return hipGetLastError();
}

namespace {
hipError_t vote_rows(const uint32_t *pair_diff, const int32_t *subsets, int64_t f, int r, int K,
                     int8_t *vote, uint8_t *has_majority, uint64_t *disagree, uint64_t *stage,
                     const int32_t *sel, int32_t *sel_out, hipStream_t s) {
#define ASPIS_VOTE(RR)                                                                           \
    vote_rows_kernel<RR><<<1, 1024, 0, s>>>(pair_diff, subsets, f, K, vote, has_majority, disagree, \
                                            stage, sel, sel_out);
    switch (r) {
    case 3: ASPIS_VOTE(3) break;
    case 5: ASPIS_VOTE(5) break;
    case 7: ASPIS_VOTE(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_VOTE
    return hipGetLastError();
}
}  // namespace

hipError_t launch_vote_rows(const uint32_t *pair_diff, const int32_t *subsets, int64_t f,
                            int r, int K, int8_t *vote, uint8_t *has_majority,
                            uint64_t *disagree, uint64_t *stage, hipStream_t s) {
    if (f > kVoteRowsMaxFiles || K < 1 || K > 64) return hipErrorInvalidValue;
    return vote_rows(pair_diff, subsets, f, r, K, vote, has_majority, disagree, stage, nullptr,
                     nullptr, s);
}

// Every probed coordinate inside [0, d), the blocks within their count.
bool probe_valid(const ProbeSet &p, int64_t d) {
    if (p.nb <= 0 || p.nb > kProbeMaxBlocks) return false;
    if (p.seed == 0) return p.kend > 0 && p.kend <= d && p.kend <= p.nb * kProbeBlockCols;
    for (int64_t j = 0; j < p.nb; ++j)
        if (p.start[j] < 0 || p.start[j] + kProbeBlockCols > d || p.start[j] % 4 != 0) return false;
    return true;
}

hipError_t launch_agree_file(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                             const ProbeSet &probe, uint32_t *pair_diff, hipStream_t s) {
    if (f <= 0) return hipSuccess;
    if (!probe_valid(probe, d)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)grid_for(f, (int64_t)num_cus() * 8);
#define ASPIS_AGREE_FILE(RR) \
    agree_file_kernel<RR><<<grid, kBlock, 0, s>>>(g, row_of, f, d, probe, pair_diff);
    switch (r) {
    case 3: ASPIS_AGREE_FILE(3) break;
    case 5: ASPIS_AGREE_FILE(5) break;
    case 7: ASPIS_AGREE_FILE(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_AGREE_FILE
    return hipGetLastError();
}

hipError_t launch_select(const int32_t *subsets, const int8_t *vote, int64_t f, int r,
                         int success, uint64_t honest, const int32_t *row_of, const Workspace &ws,
                         int32_t *sel_out, uint32_t *zero, int64_t n_zero, hipStream_t s) {
    select_kernel<<<1, 1024, 0, s>>>(subsets, vote, f, r, success, honest, row_of, ws.sel,
                                     ws.pos, ws.rows, ws.n_sel, sel_out, zero, n_zero);
    return hipGetLastError();
}

namespace {

constexpr int64_t kHalfMinRows = 128;
// The single pass at r = 3 takes half-key tiles of 128 columns from 24 files
// on where the vector gives every CU of an MI355X one (256; a constant, not the
// device's count, so that aspis_plan needs no device): their selection costs a
// quarter of the full keys' a column, K = 7 (35 files) d = 1M 133 against
// 203 us, d = 0.1M 26 against 32 us, K = 10 (120 files) d = 1M 237 against 336 us;
// shorter vectors spread over more CUs in tiles of 64 columns (K = 7, d =
// 7,850: 13.1 against 10.6 us).
constexpr int64_t kHalfFewRows = 24, kHalfFewCols = 128 * 256;
constexpr int64_t kHalfMaxRows = 60000;   // row numbers (with padding) fit 16 bits

// Most sweeps a half-key plan may take: 32, and 36 for the 32-column tile with
// the even split (2,300 files file-major; 2 to 4 spills).  Against the wide
// split: kernel 8.97 ms either way at d = 2M, 2.69 against 2.48 ms at d = 0.6M,
// where the wide one would be better.  Not with a row table, which 36 sweeps
// leave to global memory: 9.29 against 8.98 ms, and 2.90 against 2.61 ms.
constexpr int max_half_sweeps(int T, int fill) { return T == 32 && fill == kWsFill ? 36 : 32; }

// Sweep counts built for each plan.  A half-key tile is padded to them (the
// selection works on the padding too), so they are multiples of 4 apart,
// with 30 for the 128-column tile (455 files) and 36 for the 32-column tile
// of the even split (2,300); 20 is not built for 16 columns.
int round_sweeps(int64_t sw, bool half, int T, int fill) {
    if (half) {
        if (fill == kWsFillWide) return 24;
        if (T == 128 && (sw == 29 || sw == 30)) return 30;
        if (T == 16 && sw > 16 && sw <= 24) return 24;
        return (int)((sw + 3) / 4 * 4);
    }
    return sw <= 2 ? 2 : sw <= 4 ? 4 : sw <= 8 ? 8 : sw <= 12 ? 12 : 16;
}

// The half-key plan wider than `narrower` columns, or none; lds(T, fill)
// gives the kernel's LDS bytes.  The wide split serves 64 columns file-major
// (1,140 files) and 32 with the row table in global memory (2,024 and 2,300).
// It is not built for a row table in LDS (455 files take 128 columns of the even
// split with one: d = 3M 2.61 ms a step, 2.73 on the 64-column full-key tile);
// a table in global memory (rtg) takes it only: 2,024 files, d = 0.6M, 2.47 ms
// a step, 2.73 with the even split's 32 sweeps.
// r = 7: at most 16 sweeps of 64 or 128 columns, 28 of 32 or 16 (seven chunks
// a sweep; the keys of more sweeps spill): 330 files, d = 0.4M, 64 columns of
// 12 sweeps 0.58 ms, 128 of 24 0.66 ms; 792 files, d = 0.2M, 32 of 16 0.71,
// 64 of 28 0.88 ms; 1,716 files, d = 0.1M, 32 of 28 0.87, 16 of 16 0.91 ms.
template <typename LdsFn>
WsPlan half_plan(int64_t f, int narrower, bool ind, bool rtg, LdsFn &&lds, int r = 3,
                 int64_t min_rows = kHalfMinRows, bool wide = true) {
    WsPlan p;
    if (f < min_rows || f > kHalfMaxRows) return p;
    for (int T : {128, 64, 32, 16}) {
        if (T <= narrower) break;
        for (int fill : {kWsFill, kWsFillWide}) {
            if (fill == kWsFillWide && (!wide || (ind && !rtg) || T == 128 || T == 16 || r != 3)) continue;
            if (rtg && fill != kWsFillWide) continue;
            const int64_t rpi = half_rpi(T, fill);
            const int64_t sw = (f + rpi - 1) / rpi;
            const int64_t max_sw = fill == kWsFillWide ? 24
                                   : r == 7            ? (T > 32 ? 16 : 28)
                                   : (ind || r != 3)   ? 32
                                                       : max_half_sweeps(T, fill);
            if (sw > max_sw) continue;
            const int sweeps = round_sweeps(sw, true, T, fill);
            if (lds(T, sweeps, fill) > kLdsBytes) continue;
            p.T = T;
            p.sweeps = sweeps;
            p.half = true;
            p.fill = fill;
            p.rtg = rtg;
            return p;
        }
    }
    return p;
}

// LDS of the warp-specialised median: histograms, key tile, row list.
int64_t mws_lds_bytes(int64_t f, int T, int sweeps, bool half) {
    return half ? half_tile_words(sweeps, kWsFill) * 4 + f * (ws_offsets(T, half) ? 8 : 4)
                : (hist_words(T) + f * (int64_t)T) * 4 + f * 4;
}

WsPlan mws_plan(int64_t f, bool vec, bool full_keys = false) {
    WsPlan p;
    if (!vec) return p;
    for (int T : {64, 32, 16, 8}) {
        if (mws_lds_bytes(f, T, 0, false) > kLdsBytes) continue;
        const int64_t rpi = kWsFill / (T / 4);
        const int64_t sw = (f + rpi - 1) / rpi;
        // 16 sweeps fit the registers only next to the 64-column selection
        if (sw > (T == 64 ? 16 : 12)) continue;
        p.T = T;
        p.sweeps = sw <= 4 ? 4 : sw <= 8 ? 8 : sw <= 12 ? 12 : 16;
        break;
    }
    if (full_keys) return p;
    // The even split only: the wide one would give 1,140 files 64 columns instead
    // of 32, but halves the selecting waves, which bound the median (the two-pass
    // step at d = 1M 3.43 against 3.24 ms, at d = 200,003 0.82 against 0.76).  The
    // single pass, bound by its stream, gains from it (d = 200,003 0.61 against
    // 0.65 ms, d = 3M 6.40 against 6.50).
    const WsPlan h = half_plan(
        f, p.T, false, false,
        [&](int T, int sweeps, int) { return mws_lds_bytes(f, T, sweeps, true); }, 3, kHalfMinRows,
        false);
    return h.T != 0 ? h : p;
}

// LDS of the warp-specialised single pass: histograms, key tile, per-file
// words (half keys: two nibbles per file) and, with a row table in LDS, the
// table.
int64_t ws_lds_bytes(int64_t f, int r, int T, int sweeps, bool table_in_lds, bool half, int fill) {
    return ws_words_before_table(f, r, T, sweeps, half, fill) * 4 +
           (table_in_lds ? f * r * (ws_offsets(T, half) ? 8 : 4) : 0);
}

// Warp-specialised single pass (rows of four coordinates or more): plans as for the
// median above (the wide split without a row table in LDS).  r = 5 and 7: the
// even split.
WsPlan ws_plan(int64_t f, int r, int64_t d, bool ind, bool full_keys = false) {
    WsPlan p;
    if (d < 4) return p;
    p.r = r;
    if (r != 3) {
        // full keys: 64 columns and up to four sweeps (128 files), what the
        // registers hold next to five or seven chunks a sweep; half keys
        // beyond
        if (ws_lds_bytes(f, r, 64, 0, ind, false, kWsFill) <= kLdsBytes && f <= 4 * kWsFill / 16) {
            p.T = 64;
            p.sweeps = f <= 2 * kWsFill / 16 ? 2 : 4;
        }
        if (full_keys) return p;
        WsPlan h = half_plan(f, p.T, ind, false, [&](int T, int sweeps, int fill) {
            return ws_lds_bytes(f, r, T, sweeps, ind, true, fill);
        }, r);
        h.r = r;
        return h.T != 0 ? h : p;
    }
    for (int T : {64, 32, 16, 8}) {
        if (ws_lds_bytes(f, r, T, 0, ind, false, kWsFill) > kLdsBytes) continue;
        const int64_t rpi = kWsFill / (T / 4);
        const int64_t sw = (f + rpi - 1) / rpi;
        if (sw > 16) continue;
        p.T = T;
        p.sweeps = round_sweeps(sw, false, T, kWsFill);
        break;
    }
    if (full_keys) return p;
    const WsPlan h = half_plan(f, p.T, ind, false, [&](int T, int sweeps, int fill) {
        return ws_lds_bytes(f, r, T, sweeps, ind, true, fill);
    }, 3, d > kHalfFewCols ? kHalfFewRows : kHalfMinRows);
    WsPlan best = h.T != 0 ? h : p;
    if (ind) {
        // a 32-column tile when the row table, read from global memory (where
        // it stays cached), leaves LDS to the keys, instead of 16 columns with
        // the table in LDS (1,540 and 1,771 files, d = 0.8M: 2.76 against
        // 3.40 ms and 3.11 against 3.71 ms).  Not 64 columns instead of 32:
        // 1,140 files, d = 1M, 2.47 against 2.19 ms
        const WsPlan wide = half_plan(f, best.T, true, true, [&](int T, int sweeps, int fill) {
            return ws_lds_bytes(f, r, T, sweeps, false, true, fill);
        });
        if (wide.T != 0 && best.T <= 16) best = wide;
    }
    return best;
}

}  // namespace

FusedWsFn fused_ws_fn(const WsPlan &p, bool ind) {
    if (p.r != 3) return p.r == 5 ? fused_ws_r5_fn(p, ind) : fused_ws_r7_fn(p, ind);
    return ind ? fused_ws_r3_table_fn(p) : fused_ws_r3_fn(p);
}

namespace {

KernelPlan ws_kernel_plan(int kind, const WsPlan &p, int64_t lds, int table) {
    KernelPlan k;
    k.kind = kind;
    k.tile_cols = p.T;
    k.sweeps = p.sweeps;
    k.half_keys = p.half ? 1 : 0;
    k.stream_threads = p.fill;
    k.row_table = table;
    k.lds_bytes = lds;
    k.block = kWsThreads;
    return k;
}

}  // namespace

bool plan_median(int64_t f, bool vec, KernelPlan *out, bool full_keys) {
    const WsPlan p = mws_plan(f, vec, full_keys);
    if (p.T != 0) {
        *out = ws_kernel_plan(median_ws_fn(p) ? kKernelMedianWs : kKernelUnbuilt, p,
                              mws_lds_bytes(f, p.T, p.sweeps, p.half), 0);
        return out->kind == kKernelMedianWs;
    }
    KernelPlan k;
    const int T = pick_tile(f, 0);
    if (T != 0) {
        k.kind = kKernelMedianTile;
        k.tile_cols = T;
        k.lds_bytes = f * 4 * T + hist_words(T) * 4;
        k.block = (T >= 16 ? 1024 : 64 * T);
    } else {
        k.kind = kKernelMedianRadix;
        k.tile_cols = kRadixCols;
        k.lds_bytes = 0;   // static
        k.block = kRadixThreads;
    }
    *out = k;
    return true;
}

bool plan_single_pass(int64_t f, int r, int64_t d, bool ind, KernelPlan *out, bool full_keys) {
    *out = KernelPlan{};
    const WsPlan p = ws_plan(f, r, d, ind, full_keys);
    if (p.T != 0) {
        const int table = ind ? (p.rtg ? 2 : 1) : 0;
        *out = ws_kernel_plan(fused_ws_fn(p, ind) ? kKernelFusedWs : kKernelUnbuilt, p,
                              ws_lds_bytes(f, r, p.T, p.sweeps, ind && !p.rtg, p.half, p.fill), table);
        return out->kind == kKernelFusedWs;
    }
    if (r != 3 && r != 5 && r != 7) return false;
    const int T = pick_tile(f, f * 4);
    if (T == 0) return false;
    out->kind = kKernelFused;
    out->tile_cols = T;
    out->row_table = ind ? 2 : 0;
    out->lds_bytes = f * 4 * T + f * 4 + hist_words(T) * 4;
    out->block = (T >= 16 ? 1024 : 64 * T);
    return true;
}

bool fused_supported(int64_t f, int r) {
    KernelPlan k;
    return plan_single_pass(f, r, 4, false, &k, false) || plan_single_pass(f, r, 1, false, &k, false);
}

hipError_t launch_median(const float *g, int64_t d, const Workspace &ws, int64_t f,
                         float *out, hipStream_t s, TileUse *use, bool full_keys, bool repair) {
    const bool vec = d >= 4;
    KernelPlan k;
    if (!plan_median(f, vec, &k, full_keys)) return hipErrorInvalidValue;
    if (use) *use = TileUse{k.tile_cols, k.half_keys};
    const int T = k.tile_cols;
    const int64_t ntiles = (d + T - 1) / T;
    TileMask mask;
    if (repair) {
        mask.bits = ws.dirty;
        mask.count = ws.repair;
        mask.gshift = dirty_gran_shift(ntiles);
    }
    if (k.kind == kKernelMedianWs) {
        const unsigned grid = (unsigned)grid_for(ntiles, (int64_t)num_cus());
        const MedianWsFn fn = median_ws_fn(mws_plan(f, vec, full_keys));
        fn<<<grid, kWsThreads, (size_t)k.lds_bytes, s>>>(g, d, ws.rows, ws.n_sel, ntiles,
                                                         !whole_lines(g, d, T), out, mask);
        return hipGetLastError();
    }
    if (k.kind == kKernelMedianRadix) {
        // LDS: 66 KB of histograms, two workgroups per CU
        const unsigned grid = (unsigned)grid_for(ntiles, (int64_t)num_cus() * 2);
        median_radix_kernel<<<grid, kRadixThreads, 0, s>>>(g, d, ws.rows, ws.n_sel, ntiles, out,
                                                           mask);
        return hipGetLastError();
    }
    const size_t lds = (size_t)k.lds_bytes;
    const unsigned grid = (unsigned)tile_grid(ntiles, lds);
#define ASPIS_MED(TT)                                                                        \
    median_kernel<TT><<<grid, tile_block<TT>(), lds, s>>>(g, d, ws.rows, ws.n_sel, ntiles, out, mask);
    switch (T) {
    case 64: ASPIS_MED(64) break;
    case 32: ASPIS_MED(32) break;
    case 16: ASPIS_MED(16) break;
    case 8: ASPIS_MED(8) break;
    case 4: ASPIS_MED(4) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_MED
    return hipGetLastError();
}

hipError_t launch_save_sel(const Workspace &ws, int64_t f, hipStream_t s) {
    if (f <= 0) return hipErrorInvalidValue;
    save_sel_kernel<<<(unsigned)((f + kBlock - 1) / kBlock), kBlock, 0, s>>>(ws.sel, f, ws.sel_prev,
                                                                            ws.repair);
    return hipGetLastError();
}

hipError_t launch_dirty_tiles(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                              const Workspace &ws, const uint32_t *pair_diff, int tile_cols,
                              hipStream_t s) {
    if (f <= 0 || d <= 0 || tile_cols < 4 || (tile_cols & (tile_cols - 1)) != 0)
        return hipErrorInvalidValue;
    const int64_t ntiles = (d + tile_cols - 1) / tile_cols;
    const int gshift = dirty_gran_shift(ntiles);
    const int64_t nbits = (ntiles + (int64_t(1) << gshift) - 1) >> gshift;
    int cshift = gshift;   // columns per bit: tile_cols << gshift
    for (int c = tile_cols; c > 1; c >>= 1) ++cshift;
    const unsigned grid = (unsigned)grid_for((nbits + 31) / 32, (int64_t)num_cus() * 8);
#define ASPIS_DIRTY(RR)                                                                       \
    dirty_tiles_kernel<RR><<<grid, kBlock, 0, s>>>(g, row_of, f, d, cshift, nbits, ws.sel_prev, \
                                                   ws.sel, pair_diff, ws.dirty, ws.repair);
    switch (r) {
    case 3: ASPIS_DIRTY(3) break;
    case 5: ASPIS_DIRTY(5) break;
    case 7: ASPIS_DIRTY(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_DIRTY
    return hipGetLastError();
}

hipError_t launch_fused(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                        const Workspace &ws, uint32_t *pair_diff, float *out, hipStream_t s,
                        TileUse *use, bool full_keys) {
    return launch_fused_if(g, row_of, f, r, d, ws, pair_diff, out, s, use, full_keys, PathGate{});
}

hipError_t launch_fused_if(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                           const Workspace &ws, uint32_t *pair_diff, float *out, hipStream_t s,
                           TileUse *use, bool full_keys, PathGate gate) {
    const bool ind = row_of != nullptr;
    KernelPlan k;
    if (!plan_single_pass(f, r, d, ind, &k, full_keys)) return hipErrorInvalidValue;
    if (use) *use = TileUse{k.tile_cols, k.half_keys};
    const int T = k.tile_cols;
    const int64_t ntiles = (d + T - 1) / T;
    const size_t lds = (size_t)k.lds_bytes;
    if (k.kind == kKernelFusedWs) {
        const unsigned grid = (unsigned)grid_for(ntiles, (int64_t)num_cus());
        WsPlan p = ws_plan(f, r, d, ind, full_keys);
        p.lines = whole_lines(g, d, T);
        const FusedWsFn fn = fused_ws_fn(p, ind);
        fn<<<grid, kWsThreads, lds, s>>>(g, ind ? row_of : nullptr, f, d, ws.sel, ws.pos, ws.n_sel,
                                         ntiles, pair_diff, out, gate);
        return hipGetLastError();
    }
    const unsigned grid = (unsigned)tile_grid(ntiles, lds);
#define ASPIS_FUSED(TT, RR)                               \
    fused_kernel<TT, RR><<<grid, tile_block<TT>(), lds, s>>>( \
        g, row_of, f, d, ws.sel, ws.pos, ws.n_sel, ntiles, pair_diff, out, gate);
#define ASPIS_FUSED_R(TT)                     \
    switch (r) {                              \
    case 3: ASPIS_FUSED(TT, 3) break;         \
    case 5: ASPIS_FUSED(TT, 5) break;         \
    case 7: ASPIS_FUSED(TT, 7) break;         \
    default: return hipErrorInvalidValue;     \
    }
    switch (T) {
    case 64: ASPIS_FUSED_R(64) break;
    case 32: ASPIS_FUSED_R(32) break;
    case 16: ASPIS_FUSED_R(16) break;
    case 8: ASPIS_FUSED_R(8) break;
    case 4: ASPIS_FUSED_R(4) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_FUSED_R
#undef ASPIS_FUSED
    return hipGetLastError();
}

bool fused_mean_supported(int64_t f, int r) {
    return (r == 3 || r == 5 || r == 7) && f * 4 <= kFusedMeanLds;
}

hipError_t launch_fused_mean(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                             const Workspace &ws, uint32_t *pair_diff, float *out,
                             hipStream_t s) {
    return launch_fused_mean_if(g, row_of, f, r, d, ws, pair_diff, out, s, PathGate{});
}

hipError_t launch_fused_mean_if(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                                const Workspace &ws, uint32_t *pair_diff, float *out, hipStream_t s,
                                PathGate gate) {
    if (!fused_mean_supported(f, r)) return hipErrorInvalidValue;
    const int64_t nq = (d + 3) / 4;
    // up to 8 workgroups per CU: each wave's loads follow one another file
    // after file, so more resident waves keep more rows in flight (4 per CU
    // left K=21, d=5M 7 % slower)
    const unsigned grid = (unsigned)grid_for((nq + kBlock - 1) / kBlock, (int64_t)num_cus() * 8);
    const size_t lds = (size_t)f * 4;
#define ASPIS_FMEAN_(RR, BB, IND, SHORT)                                            \
    fused_mean_kernel<RR, BB, IND, SHORT><<<grid, kBlock, lds, s>>>(                \
        g, row_of, f, d, ws.sel, ws.n_sel, pair_diff, out, gate);
#define ASPIS_FMEAN(RR, BB)                   \
    if (d < 4 && row_of) {                    \
        ASPIS_FMEAN_(RR, 1, true, true)       \
    } else if (d < 4) {                       \
        ASPIS_FMEAN_(RR, 1, false, true)      \
    } else if (row_of) {                      \
        ASPIS_FMEAN_(RR, BB, true, false)     \
    } else {                                  \
        ASPIS_FMEAN_(RR, BB, false, false)    \
    }
    const int64_t blocks = (nq + kBlock - 1) / kBlock;
    switch (r) {
    case 3:
        if (blocks >= kMeanBurstMin * num_cus() && blocks <= kMeanBurstMax * num_cus()) {
            fused_mean_burst_kernel<3><<<grid, kBlock, lds, s>>>(g, row_of, f, d, ws.sel, ws.pos,
                                                                 ws.n_sel, pair_diff, out, gate);
        } else {
            ASPIS_FMEAN(3, 6)
        }
        break;
    case 5: ASPIS_FMEAN(5, 3) break;
    case 7: ASPIS_FMEAN(7, 3) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_FMEAN_
#undef ASPIS_FMEAN
    return hipGetLastError();
}

hipError_t launch_mean(const float *g, int64_t d, const Workspace &ws, float *out,
                       hipStream_t s, bool repair) {
    const int64_t ntiles = (d + kMeanTileCols - 1) / kMeanTileCols;
    const unsigned grid = (unsigned)grid_for(ntiles, (int64_t)num_cus() * 8);
    TileMask mask;
    if (repair) {
        mask.bits = ws.dirty;
        mask.count = ws.repair;
        mask.gshift = dirty_gran_shift(ntiles);
    }
    mean_kernel<<<grid, kBlock, 0, s>>>(g, d, ws.rows, ws.n_sel, out, mask);
    return hipGetLastError();
}

int reduce_tile_cols(const float *g, int64_t f, int64_t d, bool mean, bool full_keys) {
    if (mean) return (int)kMeanTileCols;
    const bool vec = d >= 4;
    KernelPlan k;
    return plan_median(f, vec, &k, full_keys) ? k.tile_cols : 0;
}

// The workspace of the allocation-free entry point: a static device array,
// one copy per device, whose device address is looked up once per device
// with that device current (in host code the array's name is a host-side
// stand-in, never a device address).
__device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
std::atomic<void *> g_scratch[kMaxDevices];
}  // namespace

hipError_t scratch_ptr(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *p = g_scratch[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return hipSuccess;
}

hipError_t launch_tie_probe(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                            const ProbeSet &probe, uint32_t *out, hipStream_t s) {
    const int64_t n = probe.coords();
    if (f <= 0 || n <= 0 || !probe_valid(probe, d)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)(n >= kTieCols ? kTieCols : n);
    switch (r) {
    case 3: tie_probe_kernel<3><<<grid, kTieThreads, 0, s>>>(g, row_of, f, d, probe, out); break;
    case 5: tie_probe_kernel<5><<<grid, kTieThreads, 0, s>>>(g, row_of, f, d, probe, out); break;
    case 7: tie_probe_kernel<7><<<grid, kTieThreads, 0, s>>>(g, row_of, f, d, probe, out); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_probe(const float *g, const int32_t *row_of, int64_t f, int r, int64_t d,
                        const ProbeSet &probe, const Workspace &ws, int n_tie, int *split,
                        hipStream_t s) {
    // the partial words share the workspace of the repair's tile-group bits,
    // which are written after them
    if (f <= 0 || f > kDirtyWords || !probe_valid(probe, d) || n_tie < 0 || n_tie > kTieCols ||
        n_tie > probe.coords())
        return hipErrorInvalidValue;
    int64_t most = kDirtyWords / f;
    const int64_t bursts = (probe.nb + kAgreeUnroll - 1) / kAgreeUnroll;
    if (most > bursts) most = bursts;
    *split = (int)(most > 8 ? 8 : most);
    const unsigned grid = (unsigned)(f * *split + n_tie);
    uint32_t *tie_out = reinterpret_cast<uint32_t *>(ws.stage + kStageTie);
#define ASPIS_PROBE(RR) \
    probe_kernel<RR><<<grid, kBlock, 0, s>>>(g, row_of, f, *split, d, probe, ws.dirty, tie_out);
    switch (r) {
    case 3: ASPIS_PROBE(3) break;
    case 5: ASPIS_PROBE(5) break;
    case 7: ASPIS_PROBE(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_PROBE
    return hipGetLastError();
}

hipError_t launch_guess(const int32_t *subsets, const int32_t *row_of, int64_t f, int r, int K, int q,
                        int mode, int keys, int n_tie, int split, int8_t *vote,
                        uint8_t *has_majority, uint64_t *disagree, uint32_t *pair_diff,
                        const Workspace &ws, hipStream_t s) {
    if (f <= 0 || f > kDirtyWords || K < 1 || K > kGuessMaxK || q < 0 || q >= K ||
        (keys == kKeysProbe && n_tie < 1))
        return hipErrorInvalidValue;
    const uint32_t *ties = reinterpret_cast<const uint32_t *>(ws.stage + kStageTie);
#define ASPIS_GUESS(RR)                                                                          \
    guess_kernel<RR><<<1, 1024, 0, s>>>(ws.dirty, split, subsets, f, K, K - q, mode, keys, ties,  \
                                        n_tie, row_of, vote, has_majority, disagree, ws.stage,   \
                                        pair_diff, ws.sel, ws.pos, ws.rows, ws.n_sel, ws.n_sel + 1);
    switch (r) {
    case 3: ASPIS_GUESS(3) break;
    case 5: ASPIS_GUESS(5) break;
    case 7: ASPIS_GUESS(7) break;
    default: return hipErrorInvalidValue;
    }
#undef ASPIS_GUESS
    return hipGetLastError();
}

hipError_t launch_finish(const uint32_t *pair_diff, const int32_t *subsets, int64_t f, int r, int K,
                         int8_t *vote, uint8_t *has_majority, uint64_t *disagree,
                         const Workspace &ws, int32_t *sel_out, hipStream_t s) {
    if (f > kVoteRowsMaxFiles || K < 1 || K > 64) return hipErrorInvalidValue;
    return vote_rows(pair_diff, subsets, f, r, K, vote, has_majority, disagree, ws.stage, ws.sel,
                     sel_out, s);
}

hipError_t launch_worker_rows(int K, int r, int64_t f, int32_t *row_of, hipStream_t s) {
    if (K < 2 || K > 64 || r < 2 || r > 7 || f <= 0) return hipErrorInvalidValue;
    worker_rows_kernel<<<(unsigned)((f + kBlock - 1) / kBlock), kBlock, 0, s>>>(K, r, f, row_of);
    return hipGetLastError();
}

size_t read_probe_sink_words() { return (size_t)kProbeBlocks * kBlock; }

hipError_t launch_read_probe(const void *buf, size_t nbytes, uint32_t *sink, hipStream_t s) {
    read_probe_kernel<<<kProbeBlocks, kBlock, 0, s>>>(static_cast<const uint4 *>(buf),
                                                      (int64_t)(nbytes / 16), sink);
    return hipGetLastError();
}

}  // namespace aspis
