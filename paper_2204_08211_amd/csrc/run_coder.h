// Coder of h_Hf (Sec. II-B (iii), Sec. IV-A (ii); Algorithm 1 line 9) for four wavefronts that share a chunk: a thread codes a
// run of 16 consecutive symbols, which it holds in registers, straight to its place in the chunk's words.  Of the single-sweep
// encoder (k_fused.hip) and of the coder for stored symbols (k_pack.hip).
//
// A run's code lengths are known before its place is (the table's entries are looked up first and kept), so one prefix sum
// over the runs says where each begins, and the codewords are ORed into the chunk's words in LDS from there on: no row per
// lane, nothing shifted afterwards.  A thread's chain is a quarter of that of pack_core.h, whose lanes take 64 symbols, and
// all wavefronts of the chunk share it.
//
// Entries in LDS are the table's turned round: the codeword (up to 24 bits) from the top bit on, its length in the low
// byte; kRunSlow alone for a longer code or none.  Codewords are placed two at a time; one by one in a run that has a pair of
// 32 bits or more together.  A run with a code that its entry does not hold is coded symbol by symbol from the full table
// (run_append_exact); so is a chunk of more words than the window holds, window by window.
#pragma once

#include "co3_internal.h"
#include "wave_ops.h"

namespace co3 {

constexpr int kRun = 16;                      // symbols per thread
constexpr int kRunWindow = 2048;              // words: 16 bits per symbol of a chunk
constexpr int kRunWindowStride = kRunWindow + 4;   // a run without bits behind a full window ORs nothing into the word behind it

constexpr uint32_t kRunSlow = 96;             // with any second length 32 or more, and less than 256

__device__ inline uint32_t run_entry(uint32_t fast)
{
    const uint32_t len = fast >> 24;
    return len == kFastSlow ? kRunSlow : (len ? fast << (32u - len) : 0u) | len;
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
            if (L == kRunSlow) {
                L = book.len[x & 0xffu];
                nocode += L == 0u ? 1u : 0u;
            }
            bits += L;
        }
    }
    return bits;
}

// The two lengths of a pair of entries.
__device__ inline uint32_t pair_bits(uint32_t e0, uint32_t e1) { return (e0 + e1) & 0xffu; }

// Codewords of a run's entries, kStep at a time (together less than 32 bits), from bit pos on; 0 stands for no symbol.  A word is ORed
// in with every step: what it holds so far is in its place already.  Not for a run without bits: all those behind a short chunk's end would OR
// nothing into the same word, one after the other (k_pack_chunk of 24 000 chunks of 1237 symbols 162 us, of whole ones 60; without 52).
template <int kStep, int kN>
__device__ inline void run_append(const uint32_t (&e)[kN], uint32_t pos, uint32_t *win)
{
    static_assert((kStep == 1 || kStep == 2) && kN % kStep == 0, "single codewords or pairs");
    typedef __attribute__((address_space(3))) uint32_t lds_word_t;
    auto or_in = [](uint32_t at, uint32_t x) {
        __hip_atomic_fetch_or((lds_word_t *)at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // counted from the start of LDS, so that a word's address is in the bit's
    uint32_t bit = pos + 8u * (uint32_t)(uintptr_t)(const lds_word_t *)win;
    uint32_t at = (bit >> 3) & ~3u, cur = 0u;   // cur: the run's bits in that word
#pragma unroll
    for (int j = 0; j < kN; j += kStep) {
        uint32_t c = e[j] & 0xffffff00u;
        if constexpr (kStep == 2) c |= (e[j + 1] & 0xffffff00u) >> (e[j] & 31u);
        cur |= c >> (bit & 31u);
        or_in(at, cur);
        const uint32_t rest = __builtin_amdgcn_alignbit(c, 0u, bit);
        bit += kStep == 2 ? pair_bits(e[j], e[j + kStep - 1]) : e[j] & 0xffu;
        const uint32_t next = (bit >> 3) & ~3u;
        cur = next != at ? rest : cur;
        at = next;
    }
    or_in(at, cur);
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
            if (L == kRunSlow) {
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

// ---- a team: four wavefronts a chunk ----

// What a thread keeps of its run between the sweep and the coding.
struct TeamRun {
    uint32_t w[4];        // symbols
    uint32_t e[kRun];     // their entries; 0 where there is none, or where the chunk's last ones stand in the first run
    uint32_t tail[4];     // those
    uint32_t from, to;    // its symbols in w
    uint32_t excl, bits;  // bits before it in the wavefront's share of the chunk, its own
    uint32_t total;       // that share
    uint32_t in_order;    // bits of the wavefront's run of the lane's number
    uint32_t tail_bits;
    bool slow;            // an entry is not enough
    bool wide;            // that, or a pair is too long to be placed at once
};

// Where the lanes' runs come from a transposition within quads (kQuads), lane 4 q + i has run 16 i + q; else they come in the lanes' order.
__device__ inline uint32_t run_of_lane(uint32_t lane) { return 16u * (lane & 3u) + (lane >> 2); }
__device__ inline uint32_t lane_of_run(uint32_t r) { return 4u * (r & 15u) + (r >> 4); }

// The wavefront's share is the chunk's elements base .. end - 1, all of its runs whole where `whole`.
// A run's entries, its bits and its place among the wavefront's; head: the bits of its first `shift` symbols, which belong to
// the sub-chunk before.
template <bool kQuads>
__device__ inline void team_lengths(TeamRun &run, uint32_t base, uint32_t end, bool whole, uint32_t shift, const uint32_t *entry,
                                    const BookDev &book, uint32_t &head, uint64_t *__restrict__ status)
{
    const uint32_t lane = threadIdx.x & 63u, first = base + (uint32_t)kRun * (kQuads ? run_of_lane(lane) : lane);
    const bool opens = shift && first == 0;   // the chunk's first run
    run.from = opens ? shift : 0u;
    run.to = end > first ? (end - first < (uint32_t)kRun ? end - first : (uint32_t)kRun) : 0u;
    uint32_t over = 0;   // 32 or more: a pair is too long; 64 or more: an entry is not enough (up to 48 without such, or in the tail it does no harm)
    run.bits = run.tail_bits = head = 0;
#pragma unroll
    for (int j = 0; j < kRun; ++j) run.e[j] = entry[run_symbol(run.w, j)];
    if (!whole) {
#pragma unroll
        for (int j = 0; j < kRun; ++j) run.e[j] = (uint32_t)j < run.to ? run.e[j] : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) run.tail[j] = 0;
    if (shift) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const bool ahead = (uint32_t)j < shift;
            run.tail[j] = ahead && opens ? run.e[j] : 0u;
            run.e[j] = ahead && opens ? 0u : run.e[j];
            head += ahead ? run.e[j] & 0xffu : 0u;
        }
        run.tail_bits = (run.tail[0] & 0xffu) + (run.tail[1] & 0xffu) + (run.tail[2] & 0xffu);
        over = run.tail_bits;
    }
#pragma unroll
    for (int j = 0; j < kRun; j += 2) {
        const uint32_t both = pair_bits(run.e[j], run.e[j + 1]);
        run.bits += both;
        over |= both;
    }
    // A pair of 32 bits and more is two of the rarest symbols side by side, one or a few in a launch, but a small launch waits for
    // its slowest thread: symbol by symbol from the full table such a run took 3 us (encode of four users of 66 000 elements
    // 10.7 -> 13 us, of twelve of 30 000 11 -> 13.5).
    run.wide = over > 31u;
    run.slow = over > 63u;
    if (__any(run.slow)) {
        if (run.slow) {
            uint32_t nocode = 0;
            run.bits = run_bits_exact(run.w, (int)run.from, (int)run.to, entry, book, nocode);
            run.tail_bits = opens ? run_bits_exact(run.w, 0, (int)shift, entry, book, nocode) : 0u;
            if (nocode) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_NOCODE), (unsigned long long)nocode);
            uint32_t counted = 0;
            head = opens ? 0u : run_bits_exact(run.w, 0, (int)shift, entry, book, counted);
        }
    }
    // in the runs' order and back
    run.in_order = kQuads ? (uint32_t)__shfl((int)run.bits, (int)lane_of_run(lane), 64) : run.bits;
    const uint32_t incl = wave_inclusive_scan_dpp(run.in_order);
    run.total = __builtin_amdgcn_readlane((int)incl, 63);
    run.excl = incl - run.in_order;
    if constexpr (kQuads) run.excl = (uint32_t)__shfl((int)run.excl, (int)run_of_lane(lane), 64);
}

// The run's codewords, any length, with those that stand ahead of the chunk's first run at its end: words wbase .. wbase + wn - 1.
__device__ inline void team_append_exact(const TeamRun &run, const uint32_t *entry, const BookDev &book, uint32_t pos, uint32_t chunk_bits,
                                         uint32_t *win, uint32_t wbase, uint32_t wn)
{
    run_append_exact(run.w, (int)run.from, (int)run.to, entry, book, pos, win, wbase, wn);
    if (run.from) run_append_exact(run.w, 0, (int)run.from, entry, book, chunk_bits - run.tail_bits, win, wbase, wn);
}

}  // namespace co3
