// The whole user side in one sweep for a code that is held fixed (Algorithm 1 lines 8-10 with
// the Huffman code designed beforehand, Sec. IV-A (ii)): error correction, fp conversion, memory
// update and Huffman coding without the symbols ever reaching HBM.
//
// HBM traffic per element: read g (4) + read m (4) + write m' (4) + write b (r/d bits).
//
// A workgroup takes four consecutive chunks of one user (small inputs: one).  Two forms of the sweep and the coding share the
// rest.  Streaming, a wavefront a chunk, for large inputs and for layers of few elements:
//   1. wavefront w quantizes chunk w (16 KB of g and of m, requested a quarter at a time with the
//      next quarter in flight while the current one is computed) and leaves the symbols in LDS,
//      in the rows of 16 + 1 words the pack step reads without bank conflicts; the code's tables go
//      to LDS while the first vectors are under way and the code length of every symbol is summed as
//      it is produced, so the chunk's size is known when the sweep ends.  A chunk that starts
//      at an element off the 16-byte grid (layers begin anywhere) takes the same vectors from the
//      boundary below it; only the ragged last chunk of a layer goes element by element;
//   2. the workgroup's 32-bit-rounded size is published and the sizes of all earlier workgroups of
//      the user are collected by a decoupled look-back: every workgroup first publishes its own
//      size, then reads its predecessors' until it meets one that already knows its running total.
//      Workgroups take their position from a ticket counter, so every predecessor is already
//      running and publishes without waiting for anyone: the wait always ends.  It is bounded all
//      the same; a workgroup whose bound runs out marks its entry as stalled, which its successors
//      inherit instead of waiting, writes no stream words and is counted in the status block.
//      An entry is one 64-bit word (flag and size together) and carries everything a successor
//      needs, so it is written and read with relaxed device-scope atomics: ordering fences would
//      make every workgroup write back and invalidate its L2;
//   3. while the look-back's answers travel, lane j of every wavefront codes sub-chunk j: the
//      wavefront-level coder of pack_core.h concatenates the lane's codewords in a private LDS row
//      (which also yields the sub-chunk sizes) and moves the rows to their bit offsets within the
//      chunk (this needs no stream offset: chunks are word-aligned);
//   4. the chunk's words are copied out coalesced at the offset the look-back gave.
// Teams, four wavefronts a chunk (run_coder.h): a thread takes sixteen elements, all requested at once, and codes their run of
// symbols from registers to its place among the chunk's words in LDS; the look-back's answers travel meanwhile.  What such a
// launch takes is a workgroup's way, at 2 M elements of sixteen users: ticket 3.6 us, sweep 6.4, the slowest
// wavefront of sixteen 4.3, lengths and coding 2.5, the predecessors' sizes 5.8, out 1.6.
#include <atomic>

#include "co3_internal.h"
#include "lookback.h"
#include "pack_core.h"
#include "quantize_math.h"
#include "run_coder.h"
#include "wave_ops.h"

namespace co3 {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef f4 f4_any __attribute__((aligned(4)));   // at any element

constexpr int kFuCpb = 4;                            // chunks per workgroup ...
constexpr int kFuCpbSmall = 1;                       // ... and for small inputs
constexpr int kFuTeam = 4;                           // wavefronts that share a chunk where they do
constexpr int kFuRow = kPcSymRow;                    // 16 words of symbols + 1 pad
constexpr int kFuStage = kPcSymWords;                // 1088 words hold a chunk's symbols
constexpr int kFuBatch = 4;                          // 16-byte vectors of g (and of m) a lane requests at a time
constexpr int kFuBatches = kChunk / 4 / 64 / kFuBatch; // batches per chunk
constexpr int kFuScalar = 8;                         // element rounds a lane requests together on the element path
static std::atomic<uint32_t> g_spin_limit{CO3_LOOKBACK_POLLS_DEFAULT};  // polls of one predecessor entry before giving up
uint32_t lookback_polls() { return g_spin_limit.load(); }

static_assert(kChunk % (4 * 64 * kFuBatch) == 0, "whole batches per chunk");
static_assert(kChunk % (64 * kFuScalar) == 0, "whole element rounds per chunk");

__device__ inline uint32_t fu_find_chunk_segment(const SegDev *segs, uint32_t nseg, uint64_t chunk)
{
    uint32_t lo = 0, hi = nseg;  // segs[nseg].chunk_start = nchunks > chunk
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (segs[mid].chunk_start <= chunk) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ inline void fu_wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup barrier that orders LDS accesses only: unlike __syncthreads() it does not wait for the
// wavefront's outstanding global stores (the m' vectors just written), which nobody in the
// workgroup reads.
__device__ inline void fu_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- a team: four wavefronts a chunk, a run of 16 symbols a thread (run_coder.h) ----

// The team's wavefront `part` quantizes vectors 256 part .. 256 part + 255 of the chunk, 64 side by side with every request.  A
// transposition within the quads of lanes then gives lane 4 q + i the symbols of vectors 64 i + 4 q .. + 3: run 16 i + q of the
// wavefront's (run_of_lane).
// A chunk that starts `shift` elements behind the 16-byte grid takes the vectors from the boundary below it, and vector 0, of
// which the first `shift` elements lie before the chunk, has the chunk's last ones in their place: every vector is whole, and the
// runs are those `shift` elements ahead, with the last few symbols of the chunk in front of the first run.
// odd: non-finite and clamped elements of the workgroup, which has one addition to each of the status words: all wavefronts of a
// launch add to the same two words, some 11 ns each, one after the other (sixteen a workgroup: twenty users of 4.4 M elements
// in [1,3,0] with 2 of 1000 beyond the largest 920 us, four, in the streaming form, 340).
// The ragged end of a layer has `vecs` vectors a lane, as few as hold it, so that all four wavefronts share it; the runs behind it
// are empty.  (Sixteen elements a lane whatever its length, one by one: encode of eight users of fifty layers of 1000 elements 15.4 us,
// of four of 3000 layers of 5333 elements 239, of 6000 of 1237 214; so 14, 209 and 177.  Stochastic, forty users of thirty layers of 100
// elements 38 and 28.)
template <bool kSR, bool kHist>
__device__ inline void team_sweep(TeamRun &run, const Layout &lay, uint32_t u, uint32_t part, uint64_t e0, uint32_t nk, uint32_t vecs, uint32_t shift,
                                  int32_t bias, float gain, float inv_gain, const float *__restrict__ gu, const float *mu,
                                  float *mo, float gamma, uint64_t seed, uint32_t *hist, uint32_t *odd)
{
    const uint32_t lane = threadIdx.x & 63u, sign_shift = lay.E + lay.M;
    const uint32_t v0 = 256u * part + lane;   // vectors v0, v0 + 64, + 128, + 192
    const QConst qc = make_qconst(lay.E, lay.M, bias);
    uint32_t n_nonfinite = 0, n_clamped = 0;
    auto element = [&](float gj, float mj, uint32_t rnd, uint32_t in, float &eo) {
        const float v = __fadd_rn(gj, __fmul_rn(gamma, mj));
        const float y = __fmul_rn(v, gain);
        uint32_t s, flags;
        float q;
        if constexpr (kSR) quantize_stochastic(y, qc, lay.E, lay.M, bias, sign_shift, rnd, s, q, flags);
        else quantize(y, qc, sign_shift, s, q, flags);
        q = __fmul_rn(q, inv_gain);
        eo = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
        n_nonfinite += flags & in;
        n_clamped += (flags >> 1) & in;
        if constexpr (kHist) {
            if (in) atomicAdd(&hist[s], 1u);
        }
        return s;
    };
    if (nk == (uint32_t)kChunk) {
        const float *ga = gu - shift, *ma = mu - shift;
        float *moa = mo - shift;
        const bool turned = shift && v0 == 0;    // this lane's first vector
        f4 gv[4], mv[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            if (r == 0 && turned) {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) {
                    const uint32_t i = j < shift ? (uint32_t)kChunk + j : j;
                    gv[0][j] = ga[i];
                    mv[0][j] = ma[i];
                }
                continue;
            }
            gv[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(ga + 4u * (v0 + 64u * r)));
            mv[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(ma + 4u * (v0 + 64u * r)));
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = 4u * (v0 + 64u * r);
            Philox4 rw;
            if constexpr (kSR) {
                rw = element_random_words(e0 - shift + i, u, seed);
                if (r == 0 && turned) {
                    const Philox4 last = element_random_words(e0 - shift + kChunk, u, seed);
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j) rw.w[j] = j < shift ? last.w[j] : rw.w[j];
                }
            }
            f4 eo;
            uint32_t packed = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float e;
                packed |= element(gv[r][j], mv[r][j], kSR ? rw.w[j] : 0u, 1u, e) << (8 * j);
                eo[j] = e;
            }
            if (r == 0 && turned) {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) moa[j < shift ? (uint32_t)kChunk + j : j] = eo[j];
            } else {
                __builtin_nontemporal_store(eo, reinterpret_cast<f4 *>(moa + i));
            }
            run.w[r] = packed;
        }
    } else if constexpr (kSR) {
        // the ragged end of a layer, element by element
        const uint32_t i0 = 4u * (64u * vecs * part + lane);
        float gs[16], ms[16];
#pragma unroll
        for (uint32_t k = 0; k < 16; ++k) {
            const uint32_t i = i0 + 256u * (k >> 2) + (k & 3u);
            const bool in = (k >> 2) < vecs && i < nk;
            gs[k] = in ? gu[i] : 0.0f;
            ms[k] = in ? mu[i] : 0.0f;
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            uint32_t packed = 0;
            run.w[r] = 0u;
            if (r >= vecs) continue;   // the same in all lanes
            uint32_t rnd[8] = {};   // the words from the vector's first element on
            const uint64_t first = e0 + i0 + 256u * r;
            const Philox4 rw = element_random_words(first, u, seed);
#pragma unroll
            for (int k = 0; k < 4; ++k) rnd[k] = rw.w[k];
            if (e0 & 3u) {   // the same in all lanes
                const Philox4 more = element_random_words(first + 4u, u, seed);
#pragma unroll
                for (int k = 0; k < 4; ++k) rnd[4 + k] = more.w[k];
#pragma unroll
                for (int k = 0; k < 7; ++k) rnd[k] = e0 & 1u ? rnd[k + 1] : rnd[k];
#pragma unroll
                for (int k = 0; k < 5; ++k) rnd[k] = e0 & 2u ? rnd[k + 2] : rnd[k];
            }
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t i = i0 + 256u * r + j;
                float e;
                const uint32_t in = i < nk ? 1u : 0u;
                const uint32_t s = element(gs[4 * r + j], ms[4 * r + j], rnd[j], in, e);
                if (in) mo[i] = e;
                packed |= (in ? s : 0u) << (8 * j);
            }
            run.w[r] = packed;
        }
    } else {
        // the ragged end of a layer, at any element: vectors, and its last few elements one by one; all one by one where the
        // registers are for counts
        constexpr bool kVectors = !kHist;
        const uint32_t i0 = 4u * (64u * vecs * part + lane);
        float gs[16], ms[16];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = i0 + 256u * r;
            if (kVectors && r < vecs && i + 4u <= nk) {
                const f4 gv = *reinterpret_cast<const f4_any *>(gu + i), mv = *reinterpret_cast<const f4_any *>(mu + i);
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) {
                    gs[4 * r + j] = gv[j];
                    ms[4 * r + j] = mv[j];
                }
            } else {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) {
                    const bool in = r < vecs && i + j < nk;
                    gs[4 * r + j] = in ? gu[i + j] : 0.0f;
                    ms[4 * r + j] = in ? mu[i + j] : 0.0f;
                }
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            run.w[r] = 0u;
            if (r >= vecs) continue;   // the same in all lanes
            uint32_t packed = 0;
            f4 eo;
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t i = i0 + 256u * r + j;
                float e;
                const uint32_t in = i < nk ? 1u : 0u;
                const uint32_t s = element(gs[4 * r + j], ms[4 * r + j], 0u, in, e);
                if constexpr (kVectors) eo[j] = e;
                else if (in) mo[i] = e;
                packed |= (in ? s : 0u) << (8 * j);
            }
            if constexpr (kVectors) {
                const uint32_t i = i0 + 256u * r;
                if (i + 4u <= nk) {
                    *reinterpret_cast<f4_any *>(mo + i) = eo;
                } else {
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j)
                        if (i + j < nk) mo[i + j] = eo[j];
                }
            }
            run.w[r] = packed;
        }
    }
    quad_transpose(run.w, lane);
    if (n_nonfinite) atomicAdd(&odd[0], n_nonfinite);
    if (n_clamped) atomicAdd(&odd[1], n_clamped);
}

// kSR: the stochastic conversion (dither from Philox words of (element, user, seed)) instead of
// the closest representative.
// kWaves: wavefronts per SIMD the register budget is cut for.  Five (a few values spill) is what the streaming of
// whole 16-byte-aligned chunks wants; layers that start at arbitrary elements take the shifted path, which holds
// more state and runs faster at four without spills, and so does the stochastic conversion (1.05 against 1.29 ms).
// kHist: also count the symbols per code table (hist_rep: kHistGlobalRep partial tables, folded afterwards), for
// callers that hold a code but want this round's histogram, e.g. to design the next round's code from it.
// kTeam: wavefronts per chunk: 1, the streaming form, or kFuTeam.  (A former team of four quantized together, then one of them
// packed: one user of 300 000 elements 23.3 -> 14.4 us, eight of 100 000 21.4 -> 13.7, of 300 000 30.5 -> 18.4.  Teams that take two or
// four of the workgroup's chunks one after the other: sixteen users of 25.6 M elements 966 -> 1100 and 1070 us.)
template <bool kSR, int kCpb, int kTeam, int kWaves, bool kHist>
__global__ __launch_bounds__(64 * kCpb * kTeam, kWaves) void k_encode_fused(
    Layout lay, const float *__restrict__ g, const float *m, float *m_out, uint64_t row_stride, float gamma,
    uint64_t seed, const BookDev *__restrict__ books, uint32_t *__restrict__ tickets, uint64_t *lb_state, uint32_t nblk,
    uint32_t spin_limit, uint64_t *__restrict__ chunk_offset, uint16_t *__restrict__ sub_bits,
    uint64_t *__restrict__ payload_bits, uint32_t *__restrict__ words, uint64_t words_stride,
    uint64_t *__restrict__ status, uint64_t *__restrict__ hist_rep)
{
    constexpr bool kIsTeam = kTeam > 1;
    // a wavefront's symbols, then its lanes' rows, then its chunk's words; a team's: the words
    __shared__ __align__(16) uint32_t s_stage[kCpb][kIsTeam ? kRunWindowStride : kPcRegion];
    __shared__ uint32_t s_fast[kCpb][kMaxA];
    __shared__ uint8_t s_len[kIsTeam ? 1 : kCpb][kIsTeam ? 4 : kMaxA];   // code lengths (0: no code), for the chunk's size
    __shared__ uint32_t s_hist[kHist ? kCpb : 1][kHist ? kMaxA : 1];   // symbol counts of a chunk
    __shared__ uint64_t s_e0[kCpb];
    __shared__ uint32_t s_n[kCpb], s_book[kCpb], s_cbits[kCpb];
    __shared__ int32_t s_bias[kCpb];
    __shared__ float s_gain[kCpb][2];
    __shared__ uint64_t s_prefix;
    __shared__ uint32_t s_ticket, s_stalled;
    __shared__ uint32_t s_odd[2];                     // (a team's) non-finite and clamped elements of the workgroup
    __shared__ uint32_t s_part[kCpb][kTeam];          // a team's wavefronts' shares of their chunk's size
    __shared__ uint32_t s_head[kIsTeam ? kCpb : 1][kIsTeam ? kSubsPerChunk + 1 : 1];   // bits of a sub-chunk that the run before its first whole one has not
    static_assert(kTeam == 1 || kTeam * 64 * kRun == kChunk, "a run for every thread of a team");
    constexpr uint32_t kLbWave = kTeam > 1 ? 1 : 0;   // wavefront that looks back

    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = kIsTeam ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(t / (64u * kTeam))) : t >> 6;      // chunk of the workgroup
    const uint32_t part = kIsTeam ? (uint32_t)__builtin_amdgcn_readfirstlane((int)((t >> 6) % kTeam)) : 0u;   // wavefront of the chunk's team
    const uint32_t wv = t >> 6;
    const uint32_t u = blockIdx.y;

    if (t == 0) s_ticket = atomicAdd(&tickets[kCpb == 1 ? 2 * (uint64_t)u * (nblk + 1ull) : u], 1u);
    // While a team's ticket is on its way: the first layer's entry and table (often there is no other), the window cleared.
    SegDev sd;
    uint32_t seg = 0, bk = 0, tab = 0;
    if constexpr (kIsTeam) {
        if (t < 2) s_odd[t] = 0u;
        sd = load_segment(lay.segs);
        bk = (lay.per_user_books ? u * lay.books_per_user : 0u) + (uint32_t)sd.book;
        tab = books[bk].fast[t % kMaxA];
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        for (uint32_t i = 4u * (t % (64u * kTeam)); i < (uint32_t)kRunWindowStride; i += 256u * kTeam)
            *reinterpret_cast<u4 *>(&s_stage[wave][i]) = u4{0u, 0u, 0u, 0u};
        if constexpr (kHist) s_hist[wave][t % kMaxA] = 0u;
    }
    fu_lds_barrier();
    const uint32_t b = kIsTeam ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_ticket) : s_ticket;  // position among the user's workgroups, < nblk = gridDim.x
    const uint64_t c0 = (uint64_t)b * kCpb;
    const uint32_t nck = lay.nchunks - c0 < (uint64_t)kCpb ? (uint32_t)(lay.nchunks - c0) : (uint32_t)kCpb;
    const bool active = wave < nck;

    TeamRun run;
    uint32_t nk = 0, shift = 0, head = 0, vecs = 4;
    uint32_t len_sum = 0;   // code lengths of the elements this lane quantizes
    if constexpr (kIsTeam) {
        // ---- 1. a team quantizes its chunk; runs of symbols and their places in the wavefront's share of its bits --------
        static_assert(!kIsTeam || 64 * kTeam == kMaxA, "a thread for every entry");
        run.total = run.tail_bits = 0;
        if (active) {
            const uint64_t c = c0 + wave;
            if (lay.nseg > 1) {
                seg = wave_find_chunk_segment(lay.segs, lay.nseg, c);
                sd = load_segment(lay.segs + seg);
                bk = (lay.per_user_books ? u * lay.books_per_user : 0u) + (uint32_t)sd.book;
                tab = books[bk].fast[t % kMaxA];
            }
            const uint64_t e0 = sd.offset + (c - sd.chunk_start) * kChunk, left = sd.offset + sd.length - e0;
            nk = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
            shift = nk == (uint32_t)kChunk ? (uint32_t)(e0 & 3u) : 0u;
            vecs = (nk + 1023u) >> 10;
            const uint64_t pair = (uint64_t)u * lay.nseg + seg, at = (uint64_t)u * row_stride + e0;
            team_sweep<kSR, kHist>(run, lay, u, part, e0, nk, vecs, shift, lay.bias[pair], lay.gain[2 * pair], lay.gain[2 * pair + 1],
                                          g + at, m + at, m_out + at, gamma, seed, s_hist[kHist ? wave : 0], s_odd);
            s_fast[wave][t % kMaxA] = run_entry(tab);
        }
        fu_lds_barrier();   // tables, counts
        if (t < 2 && s_odd[t]) atomicAdd(reinterpret_cast<unsigned long long *>(status + (t ? CO3_STAT_CLAMPED : CO3_STAT_NONFINITE)), (unsigned long long)s_odd[t]);
        if (active) {
            const bool whole = nk == (uint32_t)kChunk;
            const uint32_t from = 256u * vecs * part;
            const uint32_t end = from + 256u * vecs > nk ? nk : from + 256u * vecs;
            team_lengths<true>(run, from, end, whole, shift, s_fast[wave], books[bk], head, status);
            if ((lane & 15u) < 4u) s_head[wave][16u * part + (run_of_lane(lane) >> 2)] = head;
            if (part == 0 && lane == 0) s_head[wave][kSubsPerChunk] = run.tail_bits;
            if constexpr (kHist) {
                // the chunk's counts go to one of the partial tables of its code table
                uint64_t *dst = hist_rep + ((uint64_t)(blockIdx.x % kHistGlobalRep) * lay.nbooks + bk) * lay.A;
                const uint32_t cnt = s_hist[wave][t % kMaxA];
                if (cnt && t % kMaxA < lay.A) atomicAdd(reinterpret_cast<unsigned long long *>(dst + t % kMaxA), (unsigned long long)cnt);
            }
        } else if (part == 0 && lane == 0) {
            s_head[wave][kSubsPerChunk] = 0u;
        }
        if (lane == 0) s_part[wave][part] = run.total;
    } else {
        if (t < (uint32_t)kCpb) {
            uint64_t e0 = 0;
            uint32_t n = 0, bk = 0;
            int32_t bias = 0;
            float gn = 1.0f, gi = 1.0f;
            if (t < nck) {
                const uint64_t c = c0 + t;
                const uint32_t seg = fu_find_chunk_segment(lay.segs, lay.nseg, c);
                const SegDev sd = lay.segs[seg];
                e0 = sd.offset + (c - sd.chunk_start) * kChunk;
                const uint64_t left = sd.offset + sd.length - e0;
                n = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
                bk = (lay.per_user_books ? u * lay.books_per_user : 0u) + (uint32_t)sd.book;
                bias = lay.bias[(uint64_t)u * lay.nseg + seg];
                gn = lay.gain[2 * ((uint64_t)u * lay.nseg + seg)];
                gi = lay.gain[2 * ((uint64_t)u * lay.nseg + seg) + 1];
            }
            s_e0[t] = e0; s_n[t] = n; s_book[t] = bk; s_bias[t] = bias; s_gain[t][0] = gn; s_gain[t][1] = gi;
        }
        fu_lds_barrier();

        // ---- 1. wavefront w quantizes chunk w, symbols to LDS ---------------------------------------
        const uint32_t sign_shift = lay.E + lay.M;
        if (active) {
            const uint64_t e0 = s_e0[wave];
            const uint32_t nk = s_n[wave];
            const int bias = s_bias[wave];
            const QConst qc = make_qconst(lay.E, lay.M, bias);
            const float gain = s_gain[wave][0], inv_gain = s_gain[wave][1];   // real-valued scale: (1, 1) unless the plan carries one
            const float *gu = g + (uint64_t)u * row_stride + e0;
            const float *mu = m + (uint64_t)u * row_stride + e0;
            float *mo = m_out + (uint64_t)u * row_stride + e0;
            uint32_t n_nonfinite = 0, n_clamped = 0;
            // The code's tables are requested first and stored to LDS once the first vectors of g and m are under
            // way: the chunk's size is summed while it is quantized, so that it can be published right after.
            uint32_t tab_fast[kMaxA / 64];
#pragma unroll
            for (int r = 0; r < kMaxA / 64; ++r) tab_fast[r] = books[s_book[wave]].fast[lane + 64 * r];
            const uint32_t tab_len = reinterpret_cast<const uint32_t *>(books[s_book[wave]].len)[lane];
            auto tables_to_lds = [&]() {
#pragma unroll
                for (int r = 0; r < kMaxA / 64; ++r) s_fast[wave][lane + 64 * r] = tab_fast[r];
                reinterpret_cast<uint32_t *>(s_len[wave])[lane] = tab_len;
                if constexpr (kHist) {
#pragma unroll
                    for (int r = 0; r < kMaxA / 64; ++r) s_hist[wave][lane + 64 * r] = 0u;
                }
                fu_wave_sync_lds();
            };
            const uint8_t *len_tab = s_len[wave];
            // Four elements of a 16-byte vector: symbols packed into a word, new memory, counters and code
            // lengths for the elements `valid` marks (bit j: element j belongs to this chunk).
            auto quant4 = [&](const f4 &gv, const f4 &mv, uint64_t elem, uint32_t valid, f4 &eo, uint32_t &packed) {
                packed = 0;
                Philox4 rw;
                if constexpr (kSR) rw = element_random_words(elem, u, seed);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = __fadd_rn(gv[j], __fmul_rn(gamma, mv[j]));
                    const float y = __fmul_rn(v, gain);
                    uint32_t s, flags;
                    float q;
                    if constexpr (kSR) quantize_stochastic(y, qc, lay.E, lay.M, bias, sign_shift, rw.w[j], s, q, flags);
                    else quantize(y, qc, sign_shift, s, q, flags);
                    q = __fmul_rn(q, inv_gain);
                    eo[j] = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
                    const uint32_t ok = (valid >> j) & 1u;
                    n_nonfinite += flags & ok;
                    n_clamped += (flags >> 1) & ok;
                    len_sum += ok ? (uint32_t)len_tab[s] : 0u;
                    if constexpr (kHist) {
                        if (ok) atomicAdd(&s_hist[wave][s], 1u);
                    }
                    packed |= s << (8 * j);
                }
            };
            // A whole chunk takes a vector path: kFuBatch 16-byte vectors of g and of m per lane at a time,
            // the next batch requested before the current one is computed.
            const uint32_t shift = (uint32_t)(e0 & 3u);
            if (nk == (uint32_t)kChunk && shift == 0) {
                f4 gn[kFuBatch], mn[kFuBatch];
#pragma unroll
                for (int r = 0; r < kFuBatch; ++r) {
                    const uint32_t i = 4u * (lane + 64u * (uint32_t)r);
                    gn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(gu + i));
                    mn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(mu + i));
                }
                tables_to_lds();
#pragma unroll 1
                for (int bt = 0; bt < kFuBatches; ++bt) {
                    f4 gc[kFuBatch], mc[kFuBatch];
#pragma unroll
                    for (int r = 0; r < kFuBatch; ++r) { gc[r] = gn[r]; mc[r] = mn[r]; }
                    if (bt + 1 < kFuBatches) {
#pragma unroll
                        for (int r = 0; r < kFuBatch; ++r) {
                            const uint32_t i = 4u * (lane + 64u * (uint32_t)((bt + 1) * kFuBatch + r));
                            gn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(gu + i));
                            mn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(mu + i));
                        }
                    }
#pragma unroll
                    for (int r = 0; r < kFuBatch; ++r) {
                        const uint32_t dw = lane + 64u * (uint32_t)(bt * kFuBatch + r);  // word of the chunk's symbols
                        f4 eo;
                        uint32_t packed;
                        quant4(gc[r], mc[r], e0 + 4u * dw, 0xfu, eo, packed);
                        __builtin_nontemporal_store(eo, reinterpret_cast<f4 *>(mo + 4u * dw));
                        s_stage[wave][dw + (dw >> 4)] = packed;
                    }
                }
            } else if (nk == (uint32_t)kChunk) {
                // A layer may start at any element.  (Never in the cut for five wavefronts, which only plans on the grid take; but without
                // this path its registers come out worse, sixteen users of 25.6 M elements 942 -> 969 to 998 us.)  The same vectors, taken from the 16-byte boundary
                // below the chunk: vector k holds the chunk's elements 4k - shift .. 4k - shift + 3, so
                // its symbols fall into words k - 1 and k of the stage (OR-ed in; the stage is cleared
                // first) and the vectors at both ends are partial.
                const float *ga = gu - shift, *ma = mu - shift;
                float *moa = mo - shift;
                f4 gn[kFuBatch], mn[kFuBatch];
#pragma unroll
                for (int r = 0; r < kFuBatch; ++r) {
                    const uint32_t i = 4u * (lane + 64u * (uint32_t)r);
                    gn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(ga + i));
                    mn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(ma + i));
                }
                for (uint32_t i = lane; i < (uint32_t)(kFuStage + 1); i += 64) s_stage[wave][i] = 0;
                tables_to_lds();
#pragma unroll 1
                for (int bt = 0; bt < kFuBatches; ++bt) {
                    f4 gc[kFuBatch], mc[kFuBatch];
#pragma unroll
                    for (int r = 0; r < kFuBatch; ++r) { gc[r] = gn[r]; mc[r] = mn[r]; }
                    if (bt + 1 < kFuBatches) {
#pragma unroll
                        for (int r = 0; r < kFuBatch; ++r) {
                            const uint32_t i = 4u * (lane + 64u * (uint32_t)((bt + 1) * kFuBatch + r));
                            gn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(ga + i));
                            mn[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(ma + i));
                        }
                    }
#pragma unroll
                    for (int r = 0; r < kFuBatch; ++r) {
                        const uint32_t k = lane + 64u * (uint32_t)(bt * kFuBatch + r);  // vector, 0 .. 1023
                        const uint32_t valid = k ? 0xfu : (0xfu << shift) & 0xfu;      // vector 0 starts before the chunk
                        f4 eo;
                        uint32_t packed;
                        quant4(gc[r], mc[r], e0 - shift + 4u * k, valid, eo, packed);
                        if (k) {
                            __builtin_nontemporal_store(eo, reinterpret_cast<f4 *>(moa + 4u * k));
                            atomicOr(&s_stage[wave][(k - 1u) + ((k - 1u) >> 4)], packed << (8u * (4u - shift)));
                        } else {
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                if ((valid >> j) & 1u) moa[j] = eo[j];
                        }
                        atomicOr(&s_stage[wave][k + (k >> 4)], packed >> (8u * shift));
                    }
                }
                if (lane == 0) {
                    // vector 1024: the chunk's last `shift` elements
                    f4 gv = {0.0f, 0.0f, 0.0f, 0.0f}, mv = {0.0f, 0.0f, 0.0f, 0.0f}, eo;
                    for (uint32_t j = 0; j < shift; ++j) { gv[j] = ga[kChunk + j]; mv[j] = ma[kChunk + j]; }
                    uint32_t packed;
                    quant4(gv, mv, e0 - shift + kChunk, (1u << shift) - 1u, eo, packed);
                    for (uint32_t j = 0; j < shift; ++j) moa[kChunk + j] = eo[j];
                    const uint32_t last = kChunk / 4 - 1;
                    atomicOr(&s_stage[wave][last + (last >> 4)], (packed & ((1u << (8u * shift)) - 1u)) << (8u * (4u - shift)));
                }
            } else {
                // ragged chunk (the end of a layer): a lane takes one element of every 64, kFuScalar rounds requested together; four neighbouring lanes then gather
                // their symbols into one word of the stage
                tables_to_lds();
                for (uint32_t base = 0; base < nk; base += 64u * kFuScalar) {
                    float gs[kFuScalar], ms[kFuScalar];
#pragma unroll
                    for (int r = 0; r < kFuScalar; ++r) {
                        const uint32_t j = base + lane + 64u * r;
                        gs[r] = j < nk ? gu[j] : 0.0f;
                        ms[r] = j < nk ? mu[j] : 0.0f;
                    }
#pragma unroll
                    for (int r = 0; r < kFuScalar; ++r) {
                        const uint32_t j = base + lane + 64u * r;  // < kChunk: base is a multiple of 64 kFuScalar
                        const bool in = j < nk;
                        const float v = __fadd_rn(gs[r], __fmul_rn(gamma, ms[r]));
                        const float y = __fmul_rn(v, gain);
                        uint32_t s, flags;
                        float q;
                        if constexpr (kSR)
                            quantize_stochastic(y, qc, lay.E, lay.M, bias, sign_shift,
                                                element_random_words(e0 + j, u, seed).w[(e0 + j) & 3u], s, q, flags);
                        else quantize(y, qc, sign_shift, s, q, flags);
                        q = __fmul_rn(q, inv_gain);
                        if (in) {
                            mo[j] = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
                            n_nonfinite += flags & 1u;
                            n_clamped += (flags >> 1) & 1u;
                            len_sum += (uint32_t)len_tab[s];
                            if constexpr (kHist) atomicAdd(&s_hist[wave][s], 1u);
                        }
                        s = in ? s : 0u;
                        const uint32_t s4 = s | (__shfl_down(s, 1, 64) << 8) | (__shfl_down(s, 2, 64) << 16) |
                                            (__shfl_down(s, 3, 64) << 24);
                        const uint32_t dw = j >> 2;
                        if ((lane & 3u) == 0 && in) s_stage[wave][dw + (dw >> 4)] = s4;
                    }
                }
            }
            if (n_nonfinite)
                atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_NONFINITE),
                          (unsigned long long)n_nonfinite);
            if (n_clamped)
                atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CLAMPED), (unsigned long long)n_clamped);
            if constexpr (kHist) {
                // the chunk's counts go to one of the partial tables of its code table
                fu_wave_sync_lds();
                uint64_t *dst = hist_rep + ((uint64_t)(blockIdx.x % kHistGlobalRep) * lay.nbooks + s_book[wave]) * lay.A;
#pragma unroll
                for (int r = 0; r < kMaxA / 64; ++r) {
                    const uint32_t bin = lane + 64u * (uint32_t)r;
                    const uint32_t cnt = s_hist[wave][bin];
                    if (cnt && bin < lay.A) atomicAdd(reinterpret_cast<unsigned long long *>(dst + bin), (unsigned long long)cnt);
                }
            }
        }
        // the chunk's size: every lane summed the code lengths of the elements it quantized
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) len_sum += __shfl_xor(len_sum, o, 64);
        if (lane == 0) s_cbits[wave] = len_sum;  // 0 for a wavefront without a chunk
    }
    fu_lds_barrier();                        // also: every wavefront's symbols are staged

    // ---- 2. publish the workgroup's size; request the predecessors' ------------------------------
    uint32_t before = 0;  // 32-bit-rounded sizes of the workgroup's chunks ahead of this wavefront's
    uint32_t own = 0, pay = 0;
    uint32_t chunk_bits = 0, windows = 0;   // (a team's) of its chunk; that the longest chunk of the workgroup takes
#pragma unroll
    for (int k = 0; k < kCpb; ++k) {
        uint32_t cbits;
        if constexpr (kIsTeam) {
            cbits = s_head[k][kSubsPerChunk];
#pragma unroll
            for (int i = 0; i < kTeam; ++i) cbits += s_part[k][i];
            const uint32_t nw = (cbits + 31u) >> 5, wins = (nw + kRunWindow - 1) / kRunWindow;
            windows = windows > wins ? windows : wins;
            if ((uint32_t)k == wave) chunk_bits = cbits;
        } else {
            cbits = s_cbits[k];
        }
        const uint32_t a = (cbits + 31u) & ~31u;
        if ((uint32_t)k < wave) before += a;
        own += a;
        pay += cbits;
    }
    uint64_t *state = lb_state + (uint64_t)u * (kCpb == 1 ? nblk + 1ull : nblk);
    // By the lane that replaces the entry with the running total (or the stalled mark) below: the two stores are
    // relaxed, only one lane's program order keeps the size from landing last.
    if (t == 64u * kLbWave)
        __hip_atomic_store(&state[b], (b == 0 ? kLbPrefix : kLbAgg) | own, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    // the nearest 64 predecessor entries, requested now and looked at after the coding below
    uint64_t lb_first = kLbPrefix;  // before the first workgroup: running total 0
    if (wv == kLbWave && (int64_t)b - 1 - (int64_t)lane >= 0)
        lb_first = __hip_atomic_load(&state[b - 1 - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- 3. wavefront = chunk, lane = sub-chunk: the chunk's words, built in LDS ---------------------
    // A chunk starts on a word boundary, so its words do not depend on where it lands in the stream.
    const uint64_t c = c0 + wave;
    uint32_t *region = s_stage[wave];
    uint32_t nwords = 0;
    uint32_t excl = 0;
    const uint32_t *fast = s_fast[wave];
    int cnt = 0;
    bool fast_ok = true;
    if constexpr (kIsTeam) {
        // every thread codes its run at its place among the chunk's words
        uint32_t base = 0;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)kTeam; ++i) base += i < part ? s_part[wave][i] : 0u;
        excl = base + run.excl;
        nwords = (chunk_bits + 31u) >> 5;
        if (active) {
            if (windows == 1u) {
                if (run.slow) team_append_exact(run, fast, books[bk], excl, chunk_bits, region, 0, kRunWindow);
                else if (run.wide) run_append<1>(run.e, excl, region);
                else if (run.bits) run_append<2>(run.e, excl, region);
                if (shift && run.from && !run.slow) run_append<1>(run.tail, chunk_bits - run.tail_bits, region);
            }
            // a sub-chunk has what its four runs hold, but for the symbols ahead of the first, and with those ahead of the next
            // (behind those of the chunk's elements the empty ones, as many from every wavefront)
            const uint32_t j = lane >> 2, subs = 4u * vecs;
            const uint32_t sub = j < subs ? subs * part + j : 4u * subs + (16u - subs) * part + (j - subs);
            const uint32_t bits = quad_sum(run.in_order) + (shift ? s_head[wave][sub + 1] - s_head[wave][sub] : 0u);
            if ((lane & 3u) == 0) sub_bits[((uint64_t)u * lay.nchunks + c) * kSubsPerChunk + sub] = (uint16_t)bits;
        }
    } else {
        const uint32_t n = active ? s_n[wave] : 0u;
        const int first = (int)lane * kSub;
        cnt = (int)n - first < 0 ? 0 : ((int)n - first > kSub ? kSub : (int)n - first);
        uint32_t symw[kSub / 4];
        uint32_t my_bits = 0;
        if (active) {
            const uint32_t *row = region + kFuRow * lane;
#pragma unroll
            for (int jj = 0; jj < kSub / 4; ++jj) symw[jj] = row[jj];
            fu_wave_sync_lds();  // every lane has its symbols: the region is free
            fast_ok = n == (uint32_t)kChunk ? pc_pack_rows<true>(symw, cnt, fast, region, lane, my_bits)
                                            : pc_pack_rows<false>(symw, cnt, fast, region, lane, my_bits);
            if (!fast_ok) {
                uint32_t nocode = 0;
                my_bits = pc_general_count(symw, cnt, fast, books[s_book[wave]], region, lane, nocode);
                if (nocode)
                    atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_NOCODE), (unsigned long long)nocode);
            }
            sub_bits[((uint64_t)u * lay.nchunks + c) * kSubsPerChunk + lane] = (uint16_t)my_bits;
        }
        const uint32_t incl = pc_wave_inclusive_scan(my_bits, lane);
        excl = incl - my_bits;
        const uint32_t chunk_total = __shfl(incl, 63, 64);   // equals s_cbits[wave]: the same lengths, summed in another order
        nwords = (chunk_total + 31u) >> 5;
        if (active && fast_ok) pc_rows_to_window(region, lane, my_bits, excl, nwords);
    }

    if (wv == kLbWave) {
        uint64_t prefix = 0;
        int64_t pos = (int64_t)b - 1;
        bool stalled = false;
        while (pos >= 0) {
            const int64_t idx = pos - (int64_t)lane;
            uint64_t v = kLbPrefix;  // before the first workgroup: running total 0
            if (idx >= 0) {
                uint32_t spins = 0;
                v = pos == (int64_t)b - 1 ? lb_first
                                          : __hip_atomic_load(&state[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                while ((v >> 62) == 0 && spins < spin_limit) {
                    __builtin_amdgcn_s_sleep(1);
                    v = __hip_atomic_load(&state[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ++spins;
                }
            }
            // lane 0 holds the nearest predecessor; sum up to and including the first running total
            const uint64_t has_prefix = __ballot((v >> 62) == 2);
            const int stop = has_prefix ? (int)__builtin_ctzll(has_prefix) : 63;
            const bool bad = (int)lane <= stop && ((v >> 62) == 0 || (v >> 62) == 3);
            if (__any(bad)) { stalled = true; break; }
            uint64_t val = ((int)lane <= stop) ? (v & kLbValue) : 0ull;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) val += __shfl_xor(val, o, 64);
            prefix += val;
            if (has_prefix) break;
            pos -= 64;
        }
        if (lane == 0) {
            if (stalled) {
                __hip_atomic_store(&state[b], kLbStalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_STALLED), 1ull);
            } else if (b != 0) {
                __hip_atomic_store(&state[b], kLbPrefix | (prefix + own), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            s_prefix = prefix;
            s_stalled = stalled ? 1u : 0u;
            atomicAdd(reinterpret_cast<unsigned long long *>(payload_bits + u), (unsigned long long)pay);
        }
    }
    fu_lds_barrier();
    if (s_stalled) return;
    if constexpr (!kIsTeam) {
        if (!active) return;  // whole wavefronts; no workgroup barrier below but a team's
    }

    // ---- 4. the chunk's words go to their place in the stream -----------------------------------
    const uint64_t off = s_prefix + before;
    if (active && lane == 0 && part == 0) {
        uint64_t *co = chunk_offset + (uint64_t)u * (lay.nchunks + 1);
        co[c] = off;
        if (c + 1 == lay.nchunks) co[lay.nchunks] = off + ((uint64_t)nwords << 5);
    }
    const uint64_t off_words = off >> 5;
    bool fits = active;
    if (off_words + nwords > words_stride) {
        if (active && lane == 0 && part == 0) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CAPACITY), 1ull);
        fits = false;
        if constexpr (!kIsTeam) return;
    }
    uint32_t *dst = words + (uint64_t)u * words_stride + off_words;
    if constexpr (kIsTeam) {
        const uint32_t th = lane + 64u * part;
        if (windows == 1u) {
            for (uint32_t i = th; fits && i < nwords; i += 64 * kTeam) __builtin_nontemporal_store(region[i], dst + i);
        } else {
            // a chunk of the workgroup does not fit its window: window by window, in step
            for (uint32_t k = 0; k < windows; ++k) {
                const uint32_t wbase = k * kRunWindow, wn = nwords <= wbase ? 0u : (nwords - wbase < (uint32_t)kRunWindow ? nwords - wbase : (uint32_t)kRunWindow);
                fu_lds_barrier();
                for (uint32_t i = th; i < (uint32_t)kRunWindow; i += 64 * kTeam) region[i] = 0u;
                fu_lds_barrier();
                if (active) team_append_exact(run, fast, books[bk], excl, chunk_bits, region, wbase, wn);
                fu_lds_barrier();
                for (uint32_t i = th; fits && i < wn; i += 64 * kTeam) __builtin_nontemporal_store(region[i], dst + wbase + i);
            }
        }
    } else if (fast_ok) {
        for (uint32_t i = lane; i < nwords; i += 64) __builtin_nontemporal_store(region[i], dst + i);
    } else {
        // the general coder: the symbols are back in LDS, the words pass through a small window
        const uint32_t *win = region + kPcSymWords;
        for (uint32_t wbase = 0; wbase < nwords; wbase += kPcWin) {
            const uint32_t wn = nwords - wbase < (uint32_t)kPcWin ? nwords - wbase : (uint32_t)kPcWin;
            pc_general_window(cnt, fast, books[s_book[wave]], region, lane, excl, wbase, wn);
            for (uint32_t i = lane; i < wn; i += 64) __builtin_nontemporal_store(win[i], dst + wbase + i);
            fu_wave_sync_lds();
        }
    }
}

// Fill kernel for the look-back state and the payload counters (no memset node, so that callers
// may capture the sequence in a graph).
__global__ void k_zero_fused(uint64_t *p, uint64_t n, uint64_t *q, uint64_t nq)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
    if (i < nq) q[i] = 0;
}

// Which form.  Small: a chunk and one team a workgroup.  A user has one ticket counter, whose atomics take turns (some 15 ns
// each), and one chain of look-back entries, here one a chunk, so it is for launches that are one workgroup's way.  The next form is
// best while no CU has two of its workgroups.  Encode in this form and in that, us, by groups of four chunks:
//   groups          96         150        200        256        280        320        350
//   4 users      14.9 14.6  19 16      23 18      28 20      31 24      33 26      36 26
//   8            14.3 14.2  18 16      22 17      26 19      28 24      32 25      33 26
//   16           13.6 14.2  16.1 15.6  18 17      22 19      23.6 24.4  26.2 25.3  28 26
//   24           13.8 14.0  15.6 14.8  17 16      20 18      22 23      23.3 23.2  25.6 24.2
//   off the grid of 16 bytes
//   8            14.8 16.0  18.6 17.8  22 18      26 21      29 26      32 27      34 29
//   16           13.6 16.6  16.8 16.9  18.8 18.9  23 21      24 28      27.0 27.4  28.5 29.3
//   stochastic conversion
//   8            15.6 18.4  18.4 20.5  22 21      26 22      28.6 28.3  31 30      34 30
//   16           15.4 19.8  17.3 20.4  19 20      23.4 22.5  24.6 28.5  27 30      29 30
//   24           15.6 18.5  17.8 20.1  19 20      20.6 20.5  22.5 27.4  24 28      26 29
// (one user of 56 groups 13.4 and 13.6, of 80 16.6 and 14.6, of 190 31 and 18.)
// Teams: four chunks a workgroup, a team each.  All of a chunk's vectors are requested at once, so a launch of
// few workgroups is short and chunks off the 16-byte grid cost nothing more: eight users of 10^6 elements, in this form and in the
// streaming form, 30 and 49 us; one of 8 M 32 and 48; sixteen of 2 M 89 and 107; eight of 6 M 132 and 143; sixteen of
// 6.4 M 260 and 260; of 12 M 466 and 462; of 25.6 M 966 and 942; with a third of the chunks off the grid, of 8 M 333 and 382, of 12 M
// 483 and 560.  The stochastic conversion, teams and streaming: sixteen users of 2 M elements 99 and 106 us, of 6.4 M 289 and 271.
enum class FusedForm { kSmall, kTeams, kStream };
// In groups of kFuCpb chunks and groups per user.  Small: 2 groups + 3 of a user's up to a workgroup of teams for every CU, groups + 5
// of a user's beyond, where a user's counter is what the small form waits for; later off the grid.  Streaming: from a number of
// groups, and sooner where chunks are short on average (layers of few elements), for which a wavefront each is enough.
// us, small, teams, streaming:
//   with symbol counts, which take turns in LDS: [1,2,0], 24 users of 72 groups 17.5 22.3 24.9, of 288 29.8 36.6 38.2, of 2400
//   162 145 138; [1,4,3], eight users of 256 groups 32.5 26.1 29.1, 24 of 2400 163 116 122; [1,3,2], eight of 6980 - 342 316; [1,5,2],
//   four of 2168 - 113 133
//   stochastic, eight users of 296 groups 31.5 30.5 32.8, of 3200 298 163 157, five of 3225 - 187 253
//   layers of one chunk each, off the grid where their length is odd: of 20 elements, 40 users of 600 groups 27 23 20, of 9000 413 205 141;
//   of 301 27 24 19, 427 200 147; of 701, of 600 27 24 21; of 1001 28 24 23, 474 222 200; of 3101, of 9000 - 356 372
//   with counts, of 701, 40 users of 600 groups 34 29 26; of 3101, of 1520 105 79 77
//   stochastic, twelve users, of 701, of 156 groups 25 23 22, of 600 51 39 35, of 1500 105 66 65; of 1500, of 1500 112 75 76; with counts,
//   of 701, of 600 56 44 47, of 301, 40 users of 600 43 42 39.  (From 400 groups on: of layers that differ, a launch waits for the longest's
//   wavefront, fourteen users of sixty layers of 974 elements on average 43 and 52 streaming.)
// Off the grid, where streaming has shifted vectors, layers of many chunks, teams and streaming:
//   six users of 2730, 5010 and 8010 groups 135 159, 228 260, 348 381; 40 of 14 000 601 595: the teams at every size; but layers of 13 333
//   elements, of which a quarter of the chunks are ragged, 40 users of 9000 groups 341 324
//   with counts, of 5010 groups in [1,5,2] 240 269; in [1,2,0] 285 287, 40 users of 3680 209 195, of 8080 436 383
//   stochastic, 40 users of 2720 groups 138 183, of 5040 245 298, of 8080 388 376, of 14 080 668 635; six of 8010 398 457
// Users of up to eight chunks, whose counters are not waited for, small, teams, streaming: of one chunk, 500 users 10 11 19, 2500 31 42 46; of two 18
//   18 24, 54 57 69; of eight 47 48 52, 193 202 202; of one of 300 elements 9 10 13, 16 31 26, of four of 300 16 15 15, 51 54 38; with counts, of
//   eight 52 86 91, 201 349 346, of four of 300 28 56 59, 86 229 232; stochastic, of eight 49 53 52, 194 212 205, of one of 300 23 24 15, 32 50 36
// short_chunk, short_off: the average of a chunk's elements, where all layers are on the grid, and else.
struct FormLines { uint64_t small, small_beyond, stream, short_chunk, short_off, short_stream; };
constexpr FormLines kFuNearest = {280, 400, 7000, 350, 1050, 400};
constexpr FormLines kFuCounts = {400, 550, 7000, 3150, 3150, 400};
constexpr FormLines kFuStochastic = {520, 550, 4000, 1050, 1050, 400};
constexpr FormLines kFuStochasticCounts = {520, 550, 4000, 350, 350, 600};
constexpr uint64_t kFuFewSymbols = 2000, kFuMoreSymbols = 4000;   // counts, alphabets of up to 16 and up to 64
constexpr uint64_t kFuFewGroups = 2;   // of a user's
constexpr uint64_t kFuSmallOff = 60, kFuFewOff = 3500, kFuStreamOff = 7000, kFuWhole = 3500;
static FusedForm fused_form(const Layout &lay, bool stochastic, bool counts)
{
    const FormLines &line = stochastic ? (counts ? kFuStochasticCounts : kFuStochastic) : (counts ? kFuCounts : kFuNearest);
    const uint64_t per_user = (lay.nchunks + kFuCpb - 1) / kFuCpb, groups = (uint64_t)lay.U * per_user, off = lay.vec_aligned ? 0 : kFuSmallOff;
    const bool shorts = groups >= line.short_stream && lay.d <= (lay.vec_aligned ? line.short_chunk : line.short_off) * lay.nchunks;
    if (per_user <= kFuFewGroups && groups < line.stream && (counts || !shorts || (!stochastic && lay.nchunks < 4))) return FusedForm::kSmall;
    if (shorts) return FusedForm::kStream;
    const bool small = groups <= 256 ? 2 * groups + 3 * per_user < line.small + off : groups + 5 * per_user < line.small_beyond + off;
    if (small) return FusedForm::kSmall;
    const uint64_t stream = counts && !stochastic && lay.A <= 64 ? (lay.A <= 16 ? kFuFewSymbols : kFuMoreSymbols) : line.stream;
    if (lay.vec_aligned) return groups < stream ? FusedForm::kTeams : FusedForm::kStream;
    if (counts && !stochastic && lay.A <= 16) return groups < kFuFewOff ? FusedForm::kTeams : FusedForm::kStream;
    return groups >= kFuStreamOff && (stochastic || lay.d <= kFuWhole * lay.nchunks) ? FusedForm::kStream : FusedForm::kTeams;
}

size_t fused_workspace_bytes(const Layout &lay)
{
    // a plan's workspace serves both conversions, with and without counts: the small form, a workgroup a chunk, takes the most
    const bool small = fused_form(lay, false, false) == FusedForm::kSmall || fused_form(lay, false, true) == FusedForm::kSmall ||
                       fused_form(lay, true, false) == FusedForm::kSmall || fused_form(lay, true, true) == FusedForm::kSmall;
    const uint64_t cpb = small ? kFuCpbSmall : kFuCpb;
    const uint64_t nblk = (lay.nchunks + cpb - 1) / cpb;
    // the look-back entries and a ticket counter (one 64-bit slot per user), the partial symbol-count tables of the
    // histogram option, plus alignment slack
    return (size_t)(((uint64_t)lay.U + (uint64_t)lay.U * nblk + (uint64_t)kHistGlobalRep * lay.nbooks * lay.A) *
                        sizeof(uint64_t) + 512);
}

template <bool kSR, int kCpb, int kTeam, int kWaves, bool kHist>
static void launch_fused_waves(const Layout &lay, const co3_encode_args &a, const BookDev *books, uint32_t *tickets,
                               uint64_t *lb_state, uint32_t nblk, uint64_t *hist_rep, hipStream_t s)
{
    hipLaunchKernelGGL((k_encode_fused<kSR, kCpb, kTeam, kWaves, kHist>), dim3(nblk, lay.U), dim3(64 * kCpb * kTeam), 0, s, lay, a.g, a.m,
                       a.m_out, a.row_stride, a.gamma, a.seed, books, tickets, lb_state, nblk, lookback_polls(),
                       a.chunk_offset, a.sub_bits, a.payload_bits, a.words, a.words_stride, a.status, hist_rep);
}

// Wavefronts per SIMD the kernel is cut for.  A team's threads hold sixteen elements: two workgroups of 1024 threads fit a CU up
// to 64 registers (the stochastic conversion spills fifteen for that: sixteen users of 2 M elements 110 -> 99 us).  The
// streaming form: five only for the conversion to the nearest representative without symbol counts, on the grid (k_encode_fused's comment).
template <bool kSR, bool kHist>
static void launch_fused_variant(FusedForm form, const Layout &lay, const co3_encode_args &a, const BookDev *books,
                                 uint32_t *tickets, uint64_t *lb_state, uint32_t nblk, uint64_t *hist_rep, hipStream_t s)
{
    if (form == FusedForm::kSmall) launch_fused_waves<kSR, kFuCpbSmall, kFuTeam, kSR ? 6 : 8, kHist>(lay, a, books, tickets, lb_state, nblk, hist_rep, s);
    else if (form == FusedForm::kTeams) launch_fused_waves<kSR, kFuCpb, kFuTeam, 8, kHist>(lay, a, books, tickets, lb_state, nblk, hist_rep, s);
    else if (kSR || kHist || !lay.vec_aligned) launch_fused_waves<kSR, kFuCpb, 1, 4, kHist>(lay, a, books, tickets, lb_state, nblk, hist_rep, s);
    else if constexpr (!kSR && !kHist) launch_fused_waves<kSR, kFuCpb, 1, 5, kHist>(lay, a, books, tickets, lb_state, nblk, hist_rep, s);
}

hipError_t launch_encode_fused(const Layout &lay, const co3_encode_args &a, const BookDev *books, hipStream_t s)
{
    if (lay.U == 0) return hipSuccess;
    const bool sr = a.rounding == CO3_ROUND_STOCHASTIC;
    const FusedForm form = fused_form(lay, sr, a.hist != nullptr);
    const uint64_t cpb = form == FusedForm::kSmall ? kFuCpbSmall : kFuCpb;
    const uint64_t nblk = (lay.nchunks + cpb - 1) / cpb;
    uint64_t *base = reinterpret_cast<uint64_t *>((reinterpret_cast<uintptr_t>(a.workspace) + 255u) & ~(uintptr_t)255u);
    // A ticket counter per user and the look-back entries.  Atomics on one cache line take turns whichever word they
    // add to.  In the small form all users' workgroups start together, so a user's counter lies in front of its own
    // entries: on a line of its own from fifteen chunks a user on, beside few others below that (eight users of 10^6
    // elements, a round: 87 -> 68 us).  In the large form they lie side by side in front of all entries; where a
    // user's workgroups are fewer than fit the device, the users that run together share the line.
    uint64_t *lb_state = base + (cpb == kFuCpbSmall ? 1 : lay.U);
    uint64_t *hist_rep = base + (uint64_t)lay.U * (nblk + 1);   // [kHistGlobalRep][nbooks][A], with a.hist only
    const uint64_t hist_n = (uint64_t)lay.nbooks * lay.A;
    const uint64_t nz = (uint64_t)lay.U + (uint64_t)lay.U * nblk + (a.hist ? (uint64_t)kHistGlobalRep * hist_n : 0);
    {
        ProfScope prof(K_ZERO, s);
        const uint64_t nmax = nz > lay.U ? nz : lay.U;
        hipLaunchKernelGGL(k_zero_fused, dim3((uint32_t)((nmax + 255) / 256)), dim3(256), 0, s, base, nz,
                           a.payload_bits, (uint64_t)lay.U);
    }
    if (lay.nchunks == 0) {
        // nothing to encode: every user's stream is empty; chunk_offset[u][0] = 0
        {
            ProfScope prof(K_ZERO, s);
            hipLaunchKernelGGL(k_zero_fused, dim3((lay.U + 255) / 256), dim3(256), 0, s, a.chunk_offset,
                               (uint64_t)lay.U, a.chunk_offset, (uint64_t)0);
        }
        if (a.hist) return launch_reduce_hist(hist_rep, a.hist, hist_n, s);   // all-zero counts
        return hipGetLastError();
    }
    {
        ProfScope prof(K_FUSED, s);
        uint32_t *tickets = reinterpret_cast<uint32_t *>(base);
        if (a.hist) {
            if (sr) launch_fused_variant<true, true>(form, lay, a, books, tickets, lb_state, (uint32_t)nblk, hist_rep, s);
            else launch_fused_variant<false, true>(form, lay, a, books, tickets, lb_state, (uint32_t)nblk, hist_rep, s);
        } else {
            if (sr) launch_fused_variant<true, false>(form, lay, a, books, tickets, lb_state, (uint32_t)nblk, hist_rep, s);
            else launch_fused_variant<false, false>(form, lay, a, books, tickets, lb_state, (uint32_t)nblk, hist_rep, s);
        }
    }
    if (a.hist) return launch_reduce_hist(hist_rep, a.hist, hist_n, s);
    return hipGetLastError();
}

}  // namespace co3

extern "C" void co3_set_lookback_polls(uint32_t polls) { co3::g_spin_limit.store(polls); }
