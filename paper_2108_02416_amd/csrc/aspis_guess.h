// aspis_guess.h -- the clique search of the single pass's guess, written over
// a set of wave operations so that host code can run it too.  Not part of the
// ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace aspis {

// Most workers the search takes: one 32-bit mask.  The device guess has at
// most 4,096 files, so K <= 30 there (r = 3; less at r = 5 and 7).
constexpr int kGuessMaxK = 32;

// Whether the detection graph has exactly one maximum clique and it holds at
// least `need` workers (>= 1), as aspis_clique decides it; that clique to
// *honest.
//
// A clique is what is left after every disagreeing pair has lost a worker, so
// the search branches on the candidates C alone: the worker v with the most
// disagreements inside C is dropped, or it stays and those workers are
// dropped.  The two subtrees share no clique, and a clique the first one
// leaves non-maximal is met again, larger, in the second: at the maximum size
// each clique is met once.  Where nobody disagrees with more than one worker
// the maximum is known: one of each pair is dropped, and a pair gives two.
// Cut where C cannot reach thr, the least size that would still change the
// answer: with k = |C| - thr workers to spare, dropping k workers of at most
// `top` disagreements each settles at most k * top pairs.
//
// It ends after at most 1,596 nodes for K <= 30: a branch spares one worker
// less, or at least two less, out of the K - need = q <= 14 at the root, so
// N(k) = 1 + N(k-1) + N(k-2) bounds the nodes.  An honest cluster takes one
// node, q plain adversaries about 2q, and 14 adversaries who each disagree with
// three of 16 honest workers 77 (131 at most of 200 such graphs; a hill climb
// over graphs of 30 workers found none above 819).  A node is about 0.3 us: the
// probe and the guess of that cluster take 98 us, 75 us when all are honest.
// A search for maximal cliques (Bron-Kerbosch with Tomita's pivot, cut at the
// same size) takes 1,400 branches there, 0.36 us each.
//
// Wave: pairs(C, bits) sets bits[b] to the workers of C with bit b set in
// their number of disagreements inside C; against(v) gives the workers that
// disagree with v; push(depth, C) and pop(depth) keep the open branches.
template <class Wave>
__host__ __device__ inline bool guess_clique(Wave &wave, int K, int need, uint32_t *honest) {
    uint32_t C = K >= 32 ? ~0u : (1u << K) - 1u;
    int thr = need, best = 0, count = 0, depth = 0;
    uint32_t found = 0u;
    for (;;) {
        // a node: |C| >= thr
        uint32_t bits[5];
        wave.pairs(C, bits);
        int twice = 0, top = 0;   // twice the disagreeing pairs; the most of one worker
        uint32_t most = C;
        for (int b = 4; b >= 0; --b) {
            twice += __builtin_popcount(bits[b]) << b;
            if (most & bits[b]) {
                most &= bits[b];
                top |= 1 << b;
            }
        }
        const int spare = __builtin_popcount(C) - thr;
        bool down = false;
        if (top <= 1) {
            const int size = thr + spare - twice / 2;
            if (size >= thr) {
                if (top == 0 && (count == 0 || size > best)) {
                    count = 1;
                    found = C;
                    thr = size;
                } else {
                    count = 2;
                    thr = size + 1;
                }
                best = size;
            }
        } else if (twice <= 2 * spare * top) {
            const int v = __builtin_ctz(most);
            if (spare >= top) wave.push(depth++, C & ~wave.against(v));
            C &= ~(1u << v);
            down = spare >= 1;
        }
        while (!down) {
            if (depth == 0) {
                *honest = found;
                return count == 1;
            }
            C = wave.pop(--depth);
            down = __builtin_popcount(C) >= thr;   // thr may have grown
        }
    }
}

}  // namespace aspis
