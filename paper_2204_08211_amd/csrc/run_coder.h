// Coder of h_Hf (Sec. II-B (iii), Sec. IV-A (ii); Algorithm 1 line 9) for wavefronts that share a chunk: a thread codes a
// run of 16 consecutive symbols, which it holds in registers, straight to its place in the chunk's words.
//
// A run's code lengths are known before its place is (the table's entries are looked up first and kept), so one prefix sum
// over the runs says where each begins, and the codewords are ORed into the chunk's words in LDS from there on: no row per
// lane, nothing shifted afterwards.  A thread's chain is a quarter of that of pack_core.h, whose lanes take 64 symbols, and
// all wavefronts of the chunk share it.
//
// Entries in LDS are the table's turned round: the codeword (up to 24 bits) from the top bit on, its length in the low
// byte; kFastSlow alone for a longer code or none.  A run that has one, or two neighbours of more than 32 bits together,
// is coded symbol by symbol from the full table (run_append_exact); so is a chunk of more words than the window holds,
// window by window.
#pragma once

#include "co3_internal.h"
#include "wave_ops.h"

namespace co3 {

constexpr int kRun = 16;                      // symbols per thread
constexpr int kRunWindow = 2048;              // words: 16 bits per symbol of a chunk
constexpr int kRunWindowStride = kRunWindow + 4;   // a run without bits behind a full window ORs nothing into the word behind it

__device__ inline uint32_t run_entry(uint32_t fast)
{
    const uint32_t len = fast >> 24;
    return len == kFastSlow ? kFastSlow : (len ? fast << (32u - len) : 0u) | len;
}

// in[r] of lane j of a quad becomes out[j] of lane r
__device__ inline void quad_transpose(uint32_t (&a)[4], uint32_t lane)
{
    const bool b0 = lane & 1u, b1 = lane & 2u;
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b0 ? a[k] : a[k + 1]), 0xb1, 0xf, 0xf, true);
        a[k] = b0 ? x : a[k];
        a[k + 1] = b0 ? a[k + 1] : x;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b1 ? a[k] : a[k + 2]), 0x4e, 0xf, 0xf, true);
        a[k] = b1 ? x : a[k];
        a[k + 2] = b1 ? a[k + 2] : x;
    }
}

__device__ inline uint32_t quad_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xb1, 0xf, 0xf, true);
    x += (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4e, 0xf, 0xf, true);
    return x;
}

__device__ inline uint32_t run_symbol(const uint32_t (&w)[4], int j) { return (w[j >> 2] >> (8 * (j & 3))) & 0xffu; }

// Bits of symbols from .. to - 1 of a run, any code length; those without a code have none and count in nocode.
__device__ inline uint32_t run_bits_exact(const uint32_t (&w)[4], int from, int to, const uint32_t *entry, const BookDev &book,
                                          uint32_t &nocode)
{
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t x = w[k];
#pragma unroll 1
        for (int j = 4 * k; j < 4 * k + 4; ++j, x >>= 8) {
            if (j < from || j >= to) continue;
            uint32_t L = entry[x & 0xffu] & 0xffu;
            if (L == kFastSlow) {
                L = book.len[x & 0xffu];
                nocode += L == 0u ? 1u : 0u;
            }
            bits += L;
        }
    }
    return bits;
}

// Codewords of a run's entries (pairs of up to 32 bits) from bit pos on; 0 stands for no symbol.  A word is ORed in with every
// pair: what it holds so far is in its place already.
template <int kN>
__device__ inline void run_append(const uint32_t (&e)[kN], uint32_t pos, uint32_t *win)
{
    static_assert(kN % 2 == 0, "pairs");
    uint32_t *at = win + (pos >> 5);
    uint32_t np = pos & 31u, cur = 0u;   // bits of *at that are taken, and those of this run
#pragma unroll
    for (int j = 0; j < kN; j += 2) {
        const uint32_t c = (e[j] & 0xffffff00u) | ((e[j + 1] & 0xffffff00u) >> (e[j] & 31u));
        cur |= c >> np;
        atomicOr(at, cur);
        const uint32_t rest = __builtin_amdgcn_alignbit(c, 0u, np);
        np += (e[j] & 0xffu) + (e[j + 1] & 0xffu);
        cur = np >= 32u ? rest : cur;
        at += np >> 5;
        np &= 31u;
    }
    atomicOr(at, cur);
}

// The same for any code length: of symbols from .. to - 1, the words wbase .. wbase + wn - 1 of the chunk, to win[0 ..].
__device__ inline void run_append_exact(const uint32_t (&w)[4], int from, int to, const uint32_t *entry, const BookDev &book,
                                        uint32_t pos, uint32_t *win, uint32_t wbase, uint32_t wn)
{
    uint32_t wi = (pos >> 5) - wbase, np = pos & 31u;   // (below the window wi is huge)
    uint64_t acc = 0;
    auto append = [&](uint64_t code, uint32_t L) {   // L <= 32, np < 32
        acc = (acc << L) | code;
        np += L;
        if (np >= 32u) {
            np -= 32u;
            if (wi < wn) atomicOr(&win[wi], (uint32_t)(acc >> np));
            ++wi;
        }
    };
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t x = w[k];
#pragma unroll 1
        for (int j = 4 * k; j < 4 * k + 4; ++j, x >>= 8) {
            if (j < from || j >= to) continue;
            const uint32_t e = entry[x & 0xffu];
            uint32_t L = e & 0xffu;
            uint64_t code = L ? e >> (32u - (L & 31u)) : 0u;
            if (L == kFastSlow) {
                L = book.len[x & 0xffu];
                code = book.code[x & 0xffu];
                if (L > 32u) {
                    append(code >> 32, L - 32u);
                    code &= 0xffffffffull;
                    L = 32u;
                }
            }
            if (L) append(code, L);
        }
    }
    if (np && wi < wn) atomicOr(&win[wi], (uint32_t)(acc << (32u - np)));
}

}  // namespace co3
