// Alphabets wider than one byte: formats with 9 to 12 symbol bits (1 + exp + mant), e.g. [1,5,6].
//
// The steps are those of the byte path (Algorithm 1 lines 8-10 and 13-14; Sec. IV-A (i)-(iii), Sec. II-B (iv))
// and the container is the same; symbols are 16-bit words and a code table has up to 4096 entries, too many
// for the per-wavefront LDS tables the byte kernels are built around: here a workgroup shares one copy of the
// table in use.  The coder's workgroups end where the table changes, the quantizer's go on with the next one.
//
//   k_quantize_wide      v = g + gamma m, Q_fp, m' = v - ghat, symbol; symbol counts in an LDS table per workgroup
//                        (and, for a held code on layers that start on its tile grid, the chunks' coded sizes)
//   k_build_books_wide   Huffman code of a table on the device (same tie rule and canonical form as the host's):
//                        bitonic sort, two-queue merge, depths, canonical ranks from ballots
//   k_chunk_bits_wide    code lengths summed per chunk, lengths in LDS
//   (k_scan_chunks of k_pack.hip gives the chunk offsets)
//   k_pack_wide          wavefront per chunk, lane per sub-chunk with its 64 symbols in registers: lengths, wave
//                        prefix sum, codewords ORed into an LDS window at their bit offsets, window copied out
//   k_encode_wide        the three steps in one sweep, for a held code whose symbols and counts nobody asks for
// (the PS side is in k_decode_wide.hip)
#include "co3_internal.h"
#include "lookback.h"
#include "quantize_math.h"

namespace co3 {

constexpr int kWqThreads = 256;
constexpr int kWqPer = 8;                        // elements per thread and tile
constexpr int kWqTile = kWqThreads * kWqPer;
constexpr int kWWaves = 4;                       // wavefronts per workgroup of the chunk kernels
constexpr int kWThreads = 64 * kWWaves;
constexpr int kWSymRow = kSub + 2;               // a sub-chunk's 64 staged symbols + pad (16-bit units)
constexpr int kWbThreads = 1024;                 // threads of the table builder

__device__ inline uint32_t w_find_segment(const SegDev *segs, uint32_t nseg, uint64_t elem)
{
    uint32_t lo = 0, hi = nseg;  // segs[nseg].offset = d > elem
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (segs[mid].offset <= elem) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ inline void w_wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline uint32_t w_wave_sum(uint32_t x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ inline uint32_t w_wave_inclusive_scan(uint32_t x, uint32_t lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if ((int)lane >= o) x += y;
    }
    return x;
}

// ---- user side, step 1 ------------------------------------------------------------------------------------

// A workgroup takes `tiles` consecutive tiles of one user and counts their symbols in an LDS table of the code
// table in use (A entries), which it adds to one of the global partial tables when the code table changes (a layer
// with another table begins) and at its end; the few elements of a tile that belong to another table than the
// tile's first element are counted in global memory directly.
// The table's atomics into device memory at a workgroup's end are the price of many workgroups, the memory latency
// that nothing covers the price of few: up to kWqTiles tiles per workgroup, fewer while there would be less than
// kWqGrid workgroups (three users of 2 M elements: 93 workgroups 66 us, 1466 workgroups 25 us; sixteen users of
// 25.6 M elements keep 32 tiles, 1.14 ms).
constexpr uint32_t kWqTiles = 32;
constexpr uint64_t kWqGrid = 1024;
typedef float wf4 __attribute__((ext_vector_type(4)));
typedef uint32_t wu2 __attribute__((ext_vector_type(2)));
// kSR: the stochastic conversion (dither from Philox words of (element, user, seed)) instead of the closest
// representative.
// kBits: the code is known beforehand and every layer starts at a multiple of the tile (lay.tile_aligned), so
// that a tile lies in one chunk: the chunks' coded sizes are summed here (chunk_bits, zero on entry) and the
// sweep over the symbols that would count them is not needed.
template <bool kSR, bool kBits>
__global__ __launch_bounds__(kWqThreads) void k_quantize_wide(Layout lay, const float *__restrict__ g, const float *m,
                                                              float *m_out, uint16_t *__restrict__ sym,
                                                              uint64_t sym_stride, uint64_t row_stride, float gamma,
                                                              uint64_t seed, uint64_t *__restrict__ hist_rep,
                                                              const BookWide *__restrict__ books,
                                                              uint32_t *__restrict__ chunk_bits,
                                                              uint64_t *__restrict__ status, uint32_t tiles)
{
    __shared__ uint32_t s_hist[kWideMaxA];
    __shared__ uint32_t s_len4[kBits ? kWideMaxA / 4 : 1];   // the code lengths of the table in use, four per word
    const uint8_t *s_len8 = reinterpret_cast<const uint8_t *>(s_len4);
    const uint32_t u = blockIdx.y;
    const float *gu = g + (uint64_t)u * row_stride;
    const float *mu = m + (uint64_t)u * row_stride;
    float *mo = m_out + (uint64_t)u * row_stride;
    uint16_t *su = sym + (uint64_t)u * sym_stride;
    const uint32_t book_base = lay.per_user_books ? u * lay.books_per_user : 0u;
    uint64_t *hist = hist_rep + (uint64_t)(blockIdx.x % kHistGlobalRep) * lay.nbooks * lay.A;
    const uint32_t sign_shift = lay.E + lay.M;
    uint32_t n_nonfinite = 0, n_clamped = 0;
    for (uint32_t i = threadIdx.x; i < lay.A; i += kWqThreads) s_hist[i] = 0u;
    __syncthreads();
    auto flush = [&](uint32_t book) {   // between two workgroup barriers
        for (uint32_t i = threadIdx.x; i < lay.A; i += kWqThreads) {
            const uint32_t c = s_hist[i];
            if (c) atomicAdd(reinterpret_cast<unsigned long long *>(hist + (uint64_t)book * lay.A + i), (unsigned long long)c);
            s_hist[i] = 0u;
        }
    };
    uint32_t cur_book = 0xffffffffu;   // workgroup-uniform, like the layer of the tile's first element:
    uint32_t seg0 = 0, tile_book = 0;
    uint64_t seg_end = 0;              // where that layer ends (0: none looked up yet)
    uint64_t seg_off = 0, seg_chunk0 = 0;   // where it starts, and its first chunk
    int bias0 = 0;
    QConst qc0 = make_qconst(lay.E, lay.M, 0);
    float gain0 = 1.0f, inv_gain0 = 1.0f;
    for (uint32_t tile = 0; tile < tiles; ++tile) {
        const uint64_t base = ((uint64_t)blockIdx.x * tiles + tile) * kWqTile;
        if (base >= lay.d) break;      // workgroup-uniform
        if (base >= seg_end) {         // the tile starts in another layer than the last one did: look it up
            seg0 = w_find_segment(lay.segs, lay.nseg, base);
            seg_end = lay.segs[seg0 + 1].offset;
            seg_off = lay.segs[seg0].offset;
            seg_chunk0 = lay.segs[seg0].chunk_start;
            tile_book = book_base + (uint32_t)lay.segs[seg0].book;
            const uint64_t pair0 = (uint64_t)u * lay.nseg + seg0;
            bias0 = lay.bias[pair0];
            qc0 = make_qconst(lay.E, lay.M, bias0);
            gain0 = lay.gain[2 * pair0];
            inv_gain0 = lay.gain[2 * pair0 + 1];
        }
        if (tile_book != cur_book) {
            __syncthreads();
            if (cur_book != 0xffffffffu) flush(cur_book);
            if constexpr (kBits) {
                const uint32_t *len4 = reinterpret_cast<const uint32_t *>(books[tile_book].len);
                for (uint32_t i = threadIdx.x; i < (uint32_t)kWideMaxA / 4; i += kWqThreads) s_len4[i] = len4[i];
            }
            __syncthreads();
            cur_book = tile_book;
        }
        uint32_t tile_bits = 0;        // code lengths of this thread's elements of the tile
        auto add_tile_bits = [&]() {   // by every wavefront, once per tile
            if constexpr (kBits) {
                const uint32_t sum = w_wave_sum(tile_bits);
                if ((threadIdx.x & 63u) == 0u && sum)
                    atomicAdd(&chunk_bits[(uint64_t)u * lay.nchunks + seg_chunk0 + ((base - seg_off) >> 12)], sum);
            }
        };
        // the scale and the quantizer's constants of the tile's first layer serve the whole tile unless it
        // crosses into the next layer
        const uint64_t tile_end = base + kWqTile < lay.d ? base + kWqTile : lay.d;
        const bool one_layer = tile_end <= seg_end;
        if (one_layer && base + kWqTile <= lay.d) {
            // a whole tile of one layer (rows and tiles start on 16-byte boundaries): thread t takes elements
            // 4 t .. 4 t + 3 of each half, 16-byte loads and stores, four symbols per 8-byte store
            wf4 gq[kWqPer / 4], mq[kWqPer / 4];
#pragma unroll
            for (int k = 0; k < kWqPer / 4; ++k) {
                const uint64_t i = base + (uint64_t)k * (kWqThreads * 4) + threadIdx.x * 4;
                gq[k] = __builtin_nontemporal_load(reinterpret_cast<const wf4 *>(gu + i));
                mq[k] = __builtin_nontemporal_load(reinterpret_cast<const wf4 *>(mu + i));
            }
#pragma unroll
            for (int k = 0; k < kWqPer / 4; ++k) {
                const uint64_t i = base + (uint64_t)k * (kWqThreads * 4) + threadIdx.x * 4;
                wf4 eo;
                uint32_t sp[4];
                Philox4 rw;
                if constexpr (kSR) rw = element_random_words(i, u, seed);   // i is a multiple of 4
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = __fadd_rn(gq[k][j], __fmul_rn(gamma, mq[k][j]));
                    const float y = __fmul_rn(v, gain0);
                    uint32_t s, flags;
                    float q;
                    if constexpr (kSR) quantize_stochastic(y, qc0, lay.E, lay.M, bias0, sign_shift, rw.w[j], s, q, flags);
                    else quantize(y, qc0, sign_shift, s, q, flags);
                    q = __fmul_rn(q, inv_gain0);
                    eo[j] = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
                    n_nonfinite += flags & 1u;
                    n_clamped += (flags >> 1) & 1u;
                    sp[j] = s;
                    atomicAdd(&s_hist[s & (kWideMaxA - 1)], 1u);
                    if constexpr (kBits) tile_bits += s_len8[s & (kWideMaxA - 1)];
                }
                __builtin_nontemporal_store(eo, reinterpret_cast<wf4 *>(mo + i));
                wu2 packed;
                packed[0] = sp[0] | (sp[1] << 16);
                packed[1] = sp[2] | (sp[3] << 16);
                __builtin_nontemporal_store(packed, reinterpret_cast<wu2 *>(su + i));
            }
            add_tile_bits();
            continue;   // workgroup-uniform
        }
        float gv[kWqPer], mv[kWqPer];   // the tile's loads are issued together
#pragma unroll
        for (int k = 0; k < kWqPer; ++k) {
            const uint64_t i = base + (uint64_t)k * kWqThreads + threadIdx.x;
            gv[k] = i < lay.d ? __builtin_nontemporal_load(gu + i) : 0.0f;
            mv[k] = i < lay.d ? mu[i] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < kWqPer; ++k) {
            const uint64_t i = base + (uint64_t)k * kWqThreads + threadIdx.x;
            if (i >= lay.d) break;
            uint32_t book = tile_book;
            QConst qc = qc0;
            int bias = bias0;
            float gain = gain0, inv_gain = inv_gain0;
            if (!one_layer) {   // workgroup-uniform: the tile crosses into another layer
                uint32_t s_i = seg0;
                while (i >= lay.segs[s_i + 1].offset) ++s_i;   // ends: segs[nseg].offset = d > i
                const uint64_t pair = (uint64_t)u * lay.nseg + s_i;
                bias = lay.bias[pair];
                qc = make_qconst(lay.E, lay.M, bias);
                gain = lay.gain[2 * pair];
                inv_gain = lay.gain[2 * pair + 1];
                book = book_base + (uint32_t)lay.segs[s_i].book;
            }
            const float v = __fadd_rn(gv[k], __fmul_rn(gamma, mv[k]));
            const float y = __fmul_rn(v, gain);
            uint32_t s, flags;
            float q;
            if constexpr (kSR)
                quantize_stochastic(y, qc, lay.E, lay.M, bias, sign_shift, element_random_words(i, u, seed).w[i & 3u], s, q,
                                    flags);
            else quantize(y, qc, sign_shift, s, q, flags);
            q = __fmul_rn(q, inv_gain);
            mo[i] = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
            n_nonfinite += flags & 1u;
            n_clamped += (flags >> 1) & 1u;
            su[i] = (uint16_t)s;
            if (book == cur_book) atomicAdd(&s_hist[s & (kWideMaxA - 1)], 1u);
            else atomicAdd(reinterpret_cast<unsigned long long *>(hist + (uint64_t)book * lay.A + s), 1ull);
            if constexpr (kBits) tile_bits += s_len8[s & (kWideMaxA - 1)];   // (aligned layers: the tile's own table)
        }
        add_tile_bits();
    }
    __syncthreads();
    if (cur_book != 0xffffffffu) flush(cur_book);
    if (n_nonfinite)
        atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_NONFINITE), (unsigned long long)n_nonfinite);
    if (n_clamped)
        atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CLAMPED), (unsigned long long)n_clamped);
}

__global__ __launch_bounds__(256) void k_reduce_hist_wide(const uint64_t *__restrict__ hist_rep,
                                                         uint64_t *__restrict__ hist, uint64_t n)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint64_t s = 0;
    for (int r = 0; r < kHistGlobalRep; ++r) s += hist_rep[(uint64_t)r * n + i];
    hist[i] = s;
}

__global__ void k_zero_wide(uint64_t *p, uint64_t n, uint64_t *q, uint32_t nq)   // nq <= n
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
    if (i < nq) q[i] = 0;
}

// ---- code tables ------------------------------------------------------------------------------------------

// One workgroup per table.  A is a power of two (512 .. 4096).  Dynamic LDS: node weights (2 A x 8 bytes),
// parents (2 A x 4 bytes), the leaves' symbols and the symbols by rank (A x 2 bytes each).  Steps: bitonic
// sort of the symbols by (weight, symbol) with the unused ones last; the two-queue merge in rounds of many pairs;
// depth of every leaf; canonical order, the rank of a symbol among those of its length from wavefront ballots
// (wavefront w owns symbols w A/16 .. (w + 1) A/16 - 1, in order).
constexpr int kWbWaves = kWbThreads / 64;
__global__ __launch_bounds__(kWbThreads) void k_build_books_wide(BookWide *__restrict__ books, uint32_t A,
                                                                const uint64_t *__restrict__ weights,
                                                                uint64_t *__restrict__ status)
{
    extern __shared__ uint64_t wb_smem[];
    uint64_t *nw = wb_smem;                                        // [2 A] sorted leaves, then internal nodes
    int *parent = reinterpret_cast<int *>(nw + 2 * (size_t)A);      // [2 A]
    uint16_t *leaf_sym = reinterpret_cast<uint16_t *>(parent + 2 * (size_t)A);   // [A] sorted leaf -> symbol
    uint16_t *by_rank = leaf_sym + A;                                            // [A] symbols in canonical order
    __shared__ uint32_t cnt[65], off[65];
    __shared__ uint64_t first[65];
    __shared__ uint32_t wcnt[kWbWaves][65];   // symbols of each length in a wavefront's range; then running ranks
    __shared__ int err, s_n;
    __shared__ int s_wrapped[2];   // a sum of a round wrapped, by the round's parity
    __shared__ uint32_t s_maxlen, s_bits;
    __shared__ unsigned long long s_missing;
    __shared__ uint64_t end32[33];   // codes of up to l bits lie below end32[l], left-aligned in 32 bits

    BookWide &B = books[blockIdx.x];
    const uint64_t *w = weights + (uint64_t)blockIdx.x * A;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t kNone = ~0ull;    // an unused symbol in the sort, an exhausted queue in the merge: refused as a weight

    if (t < 65) { cnt[t] = 0; off[t] = 0; first[t] = 0; }
    for (uint32_t i = t; i < (uint32_t)kWbWaves * 65u; i += kWbThreads) wcnt[i / 65u][i % 65u] = 0;
    if (t == 0) { err = s_wrapped[0] = s_wrapped[1] = 0; s_maxlen = 0; s_n = 0; s_bits = 2; s_missing = 0; end32[0] = 0; }
    for (uint32_t i = t; i < 2 * A; i += kWbThreads) parent[i] = -1;
    __syncthreads();
    int active = 0;
    for (uint32_t s = t; s < A; s += kWbThreads) {
        const uint64_t ws = w[s];
        if (ws == kNone) err = 1;
        active += ws > 0 ? 1 : 0;
        nw[s] = ws ? ws : kNone;
        leaf_sym[s] = (uint16_t)s;
        B.len[s] = 0;
        B.code[s] = 0;
        B.fast[s] = kWFastSlow << kWFastCodeBits;
    }
    if (active) atomicAdd(&s_n, active);
    __syncthreads();
    const int nact = s_n;            // number of symbols with a weight

    // ascending (weight, symbol); the keys are distinct, so the order does not depend on the network.  A step over
    // fewer than 64 entries stays inside a wavefront's own entries: the workgroup meets only where a step or the one
    // after it reaches further (after 15 of the 55 steps of 1024 symbols).
    for (uint32_t k = 2; k <= A; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t i = t; i < A; i += kWbThreads) {
                const uint32_t p = i ^ j;
                if (p > i) {
                    const uint64_t wi = nw[i], wp = nw[p];
                    const uint16_t si = leaf_sym[i], sp = leaf_sym[p];
                    const bool gt = wi > wp || (wi == wp && si > sp);
                    if (gt == ((i & k) == 0)) { nw[i] = wp; nw[p] = wi; leaf_sym[i] = sp; leaf_sym[p] = si; }
                }
            }
            const uint32_t next = j > 1 ? j >> 1 : k;
            if (j >= 64u || next >= 64u || (j == 1 && k == A)) __syncthreads();
            else w_wave_sync_lds();
        }
    }

    // The two-queue merge in rounds.  With T the sum of the two lightest nodes alive, every internal node alive and
    // every leaf of weight <= T is taken before any node created from now on (their weights are >= T; on equal
    // weights a leaf goes before an internal node and an older internal node before a newer one).  So the merged
    // order of those nodes pairs off two by two exactly as the serial merge would; an odd one out stays at the head of
    // its queue.  Every thread keeps the queue positions itself and finds its pair as the byte builder's lanes do
    // (k_codebook.hip): one meeting of the workgroup a round.  A wrapped sum is marked in the round's own word of two, as
    // a thread may be a round ahead of one that has yet to look.
    // With every node's rank looked up and the merged order kept in LDS, two meetings a round: 61 us for 1024 symbols and
    // 126 for 4096, so 50 and 114.
    {
        int li = 0, ii = nact, made = nact;   // next leaf, next internal node, next node to create
        bool over = err != 0;
        for (int round = 0; nact >= 2 && !over && (nact - li) + (made - ii) > 1; round ^= 1) {   // the same in every thread
            const uint64_t c0 = li < nact ? nw[li] : kNone, c1 = li + 1 < nact ? nw[li + 1] : kNone;
            const uint64_t c2 = ii < made ? nw[ii] : kNone, c3 = ii + 1 < made ? nw[ii + 1] : kNone;
            // leaves of weight <= T, every wavefront by itself: of the 64 at equal distances, then of those between two
            const int apart = (nact - li + 63) >> 6;
            const int far = li + (int)lane * apart;
            const uint64_t wide = far < nact ? nw[far] : kNone;
            // the two lightest of two sorted pairs
            const uint64_t m1 = c0 < c2 ? c0 : c2;
            const uint64_t r1 = c0 < c2 ? c1 : c0, r2 = c0 < c2 ? c2 : c3;
            const uint64_t m2 = r1 < r2 ? r1 : r2;
            const uint64_t T = m1 + m2;
            if (T < m2 || T == kNone) {   // the table's weights sum to 2^64 - 1 or more
                if (t == 0) err = 1;
                break;
            }
            int lj = li;
            if (const int c = __popcll(__ballot(wide <= T))) {   // leaf (c - 1) apart is among them, leaf c apart is not
                lj += (c - 1) * apart;
                const int near = lj + (int)lane;
                lj += __popcll(__ballot((int)lane < apart && near < nact && nw[near] <= T));
            }
            const int bL = lj - li, bI = made - ii, nb = bL + bI;   // nb >= 2: the two lightest are among them
            const int npair = nb >> 1;
            for (int k = (int)t; k < npair; k += kWbThreads) {
                // of the first d nodes of the merged order, i are leaves
                const int d = 2 * k;
                int i = d > bI ? d - bI : 0, hi = d < bL ? d : bL;
                while (i < hi) {
                    const int mid = (i + hi) >> 1;
                    if (nw[li + mid] <= nw[ii + (d - 1 - mid)]) i = mid + 1; else hi = mid;
                }
                const int j = d - i;
                const uint64_t l0 = i < bL ? nw[li + i] : kNone, l1 = i + 1 < bL ? nw[li + i + 1] : kNone;
                const uint64_t i0 = j < bI ? nw[ii + j] : kNone, i1 = j + 1 < bI ? nw[ii + j + 1] : kNone;
                const bool leaf1 = l0 <= i0;
                const uint64_t wa = leaf1 ? l0 : i0;
                const uint64_t ln = leaf1 ? l1 : l0, in = leaf1 ? i0 : i1;
                const bool leaf2 = ln <= in;
                const uint64_t wb = leaf2 ? ln : in;
                const uint64_t sum = wa + wb;
                if (sum < wb || sum == kNone) s_wrapped[round] = 1;
                nw[made + k] = sum;
                parent[leaf1 ? li + i : ii + j] = made + k;
                parent[leaf2 ? li + i + leaf1 : ii + j + !leaf1] = made + k;
            }
            __syncthreads();
            over = s_wrapped[round] != 0;
            int next_li = lj, next_ii = made;
            if (nb & 1) {   // the heaviest of the batch stays: the last internal node unless a leaf is heavier
                if (bI > 0 && (bL == 0 || nw[made - 1] >= nw[lj - 1])) next_ii = made - 1;
                else next_li = lj - 1;
            }
            li = next_li;
            ii = next_ii;
            made += npair;
        }
        if (over && t == 0) err = 1;
    }
    __syncthreads();

    // depths of the leaves = code lengths
    for (int i = (int)t; i < nact; i += kWbThreads) {
        int depth = nact == 1 ? 1 : 0;
        for (int p = parent[i]; p >= 0 && depth <= CO3_MAX_CODE_LEN; p = parent[p]) ++depth;
        if (depth > CO3_MAX_CODE_LEN) err = 1;
        else B.len[leaf_sym[i]] = (uint8_t)depth;
    }
    __syncthreads();
    const bool bad = err != 0;
    if (bad) {
        for (uint32_t s = t; s < A; s += kWbThreads) B.len[s] = 0;
        if (t == 0) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CODELEN), 1ull);
    }
    __syncthreads();

    // lengths present in each wavefront's range of symbols, sub-block of 64 by sub-block
    const uint32_t per_wave = A / kWbWaves;   // 32 .. 256
    auto for_each_length_group = [&](uint32_t myL, auto &&body) {   // body(length, lanes with it), once per length
        uint64_t todo = __ballot(myL != 0u);
        while (todo) {
            const int leader = __ffsll((long long)todo) - 1;
            const uint32_t L0 = (uint32_t)__shfl((int)myL, leader, 64);
            const uint64_t mask = __ballot(myL == L0);
            body(L0, mask);
            todo &= ~mask;
        }
    };
    for (uint32_t sb = 0; sb < per_wave; sb += 64) {
        const uint32_t i = sb + lane;
        const uint32_t myL = i < per_wave ? (uint32_t)B.len[wave * per_wave + i] : 0u;
        for_each_length_group(myL, [&](uint32_t L0, uint64_t mask) {
            if (lane == 0) wcnt[wave][L0] += (uint32_t)__popcll(mask);
        });
    }
    __syncthreads();
    if (t < 65) {   // counts per length; a wavefront's entry becomes the rank of its first symbol of that length
        uint32_t run = 0;
        for (int wv = 0; wv < kWbWaves; ++wv) { const uint32_t c = wcnt[wv][t]; wcnt[wv][t] = run; run += c; }
        cnt[t] = run;
        if (run && t) atomicMax(&s_maxlen, t);
    }
    __syncthreads();
    if (t < 64) {
        // lane l - 1 takes length l: first[l] = 2 (first[l - 1] + cnt[l - 1]) as a scan whose step over k lengths
        // shifts by k
        uint64_t sum = t ? cnt[t] : 0u;
        uint32_t o = t ? cnt[t] : 0u;
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const uint64_t s_up = __shfl_up(sum, k, 64);
            const uint32_t o_up = __shfl_up(o, k, 64);
            if ((int)t >= k) {
                sum += s_up << k;
                o += o_up;
            }
        }
        first[t + 1] = sum << 1;
        off[t + 1] = o;
        if (t < 32) end32[t + 1] = ((sum << 1) + cnt[t + 1]) << (31u - t);
    }
    __syncthreads();
    // canonical order: rank among the symbols of the same length, ascending symbol (and, in by_rank, for the table below)
    uint32_t bits = 0;
    for (uint32_t sb = 0; sb < per_wave; sb += 64) {
        const uint32_t i = sb + lane;
        const uint32_t s_i = wave * per_wave + i;
        const uint32_t myL = i < per_wave ? (uint32_t)B.len[s_i] : 0u;
        for_each_length_group(myL, [&](uint32_t L0, uint64_t mask) {
            const uint32_t base = wcnt[wave][L0];
            if (myL == L0) {
                const uint32_t rank = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                const uint64_t code = first[L0] + rank;
                B.code[s_i] = code;
                if (L0 <= kWFastCodeBits) B.fast[s_i] = (L0 << kWFastCodeBits) | (uint32_t)code;
                B.sorted[off[L0] + rank] = (uint16_t)s_i;
                by_rank[off[L0] + rank] = (uint16_t)s_i;
                // mantissa bits that a code with up to ten leading ones asks of the decode table
                const uint32_t ones = (uint32_t)__clzll((long long)~(code << (64u - L0)));   // (a 64-bit code: code itself)
                if (ones <= 10u && ones < L0 && L0 - ones - 1u > bits) bits = L0 - ones - 1u;
            }
            w_wave_sync_lds();   // every lane has read the base
            if (lane == 0) wcnt[wave][L0] = base + (uint32_t)__popcll(mask);
            w_wave_sync_lds();
        });
    }
    for (uint32_t i = (bad ? 0u : (uint32_t)nact) + t; i < A; i += kWbThreads) B.sorted[i] = 0;
    if (bits > 2u) atomicMax(&s_bits, bits);
    if (t < 65) { B.first[t] = first[t]; B.count[t] = cnt[t]; B.offset[t] = off[t]; }
    if (t == 0) { B.maxlen = s_maxlen; B.nactive = bad ? 0u : (uint32_t)nact; }
    __syncthreads();
    // the decode table (decode_core.h): an entry's window by its low end, the length by a binary search of the ends (they
    // grow with it), the symbol by its rank
    const uint32_t nm = s_bits < wide_tab_bits_max(A) ? s_bits : wide_tab_bits_max(A);
    if (t < 32) B.limit[t] = end32[t] >> 32 ? 0u : 0xffffffffu - (uint32_t)end32[t];
    auto entry = [&](uint32_t x, uint32_t longest) {   // window, longest code that covers the entry
        uint32_t l = 0;   // the largest l with x >= end32[l]: the code has l + 1 bits
#pragma unroll
        for (uint32_t k = 16; k; k >>= 1) l = (uint64_t)x >= end32[l + k] ? l + k : l;
        const uint32_t L = l + 1u;
        uint32_t e = kLenSlow;
        if (L < 32u && L <= longest)
            e = ((uint32_t)by_rank[(off[L] + ((x >> (32u - L)) - (uint32_t)first[L])) & (A - 1u)] << 8) | L;
        return e;
    };
    uint64_t missing = 0;   // share of the code space the table leaves to the search, in 2^-32
#pragma unroll 2
    for (uint32_t i = t; i < wide_tab_entries(nm); i += kWbThreads) {
        const uint32_t ex = kWideTabLow + (i >> nm) + 1u;
        const uint32_t e = i >> nm ? entry(~(uint32_t)((uint64_t)((1u << nm) | (i & ((1u << nm) - 1u))) << (ex - nm)), 32u - ex + nm) : kLenSlow;
        if (e == kLenSlow && i >> nm) missing += 1ull << (ex - nm);
        B.tab[i] = e;
    }
    bool prefixes = false;
    // Fewer bits than the most resolve every code with up to ten leading ones, and what they leave of the others (eleven ones and
    // more than nm bits behind the next) has more than twelve bits: a table by the first twelve would resolve no more.
    if (nm == wide_tab_bits_max(A)) {
        if (missing) atomicAdd(&s_missing, (unsigned long long)missing);
        __syncthreads();
        prefixes = s_missing > (1ull << 32) - end32[kWidePrefixBits];
        if (prefixes)
            for (uint32_t i = t; i < wide_tab_entries(0); i += kWbThreads) B.tab[i] = entry(~(i << (32u - kWidePrefixBits)), kWidePrefixBits);
    }
    if (t == 0) B.tab_bits = prefixes ? 0u : nm;
}

// ---- user side, steps 2 and 3 -------------------------------------------------------------------------------

// Both chunk kernels give a workgroup up to kWWaves * cpw consecutive chunks of one user, wavefront w chunks w,
// w + kWWaves, ..., with their code table in LDS; where the next chunk has another table a workgroup ends early.
// (Workgroups that went on kept the first table only and coded the other chunks by rolled loops from device memory:
// three users of 2 M elements in five layers with a table each, k_pack_wide 370 us, this way 16 us.  Workgroups that
// end with every layer read up to 36 KB of table for each and leave wavefronts without a chunk: sixteen users of
// 1000 layers of 1000 elements under one table in [1,4,5], both kernels 226 and 48 us, this way 79 and 23.)
// A wavefront takes four chunks where that still leaves every CU several workgroups, and one otherwise.
static_assert(kWgChunksSmall == kWWaves && kWgChunks == 4 * kWWaves, "the plan's workgroup counts");
constexpr uint64_t kWSmallGrid = 1024;   // workgroups of kWgChunks chunks below which they take kWgChunksSmall
inline uint32_t w_chunks_per_wave(const Layout &lay, const WideCut &cut)
{
    return (uint64_t)cut.nwg * lay.U < kWSmallGrid ? kWgChunksSmall / kWWaves : kWgChunks / kWWaves;
}
// First chunk of workgroup b, the number of its chunks, their code table, the layers [seg, seg_end) they lie in.  Where
// that is one layer, as in any large one, a chunk's place follows from the first's: no search per chunk.  i is the same
// in the whole wavefront and said to be (readfirstlane), so that places are kept in scalar registers: sixteen users of
// 25.6 M elements, k_pack_wide 530 us without that, 488 us with it.
struct WRange {
    uint64_t first, e0, left;   // left: elements of the first chunk's layer from e0 on
    uint32_t nck, book, seg, seg_end;
    __device__ inline void place(const SegDev *segs, uint32_t i, uint64_t &e, uint32_t &n) const   // of the workgroup's chunk i
    {
        e = e0 + i * (uint32_t)kChunk;
        uint64_t rest = left - i * (uint32_t)kChunk;
        if (seg_end - seg > 1) {
            uint32_t lo = seg, hi = seg_end;   // last layer that starts at or before the chunk
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (segs[mid].chunk_start <= first + i) lo = mid; else hi = mid;
            }
            const SegDev sd = segs[lo];
            e = sd.offset + (first + i - sd.chunk_start) * kChunk;
            rest = sd.offset + sd.length - e;
        }
        n = rest < (uint64_t)kChunk ? (uint32_t)rest : (uint32_t)kChunk;
    }
};
__device__ inline WRange w_range(const Layout &lay, const RunDev *runs, uint32_t nrun, uint32_t u, uint32_t b, uint32_t cpw)
{
    const bool small = cpw * kWWaves == kWgChunksSmall;
    uint32_t lo = 0, hi = nrun;   // last run whose first workgroup is <= b: every run has one
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((small ? runs[mid].wg_small_start : runs[mid].wg_start) <= b) lo = mid; else hi = mid;
    }
    const RunDev rd = runs[lo];
    WRange r;
    r.first = rd.chunk_start + (uint64_t)(b - (small ? rd.wg_small_start : rd.wg_start)) * (kWWaves * cpw);
    const uint64_t chunks = runs[lo + 1].chunk_start - r.first;   // > 0: run lo has this workgroup
    r.nck = chunks < (uint64_t)(kWWaves * cpw) ? (uint32_t)chunks : kWWaves * cpw;
    r.book = (lay.per_user_books ? u * lay.books_per_user : 0u) + (uint32_t)rd.book;
    r.seg = rd.seg;
    r.seg_end = runs[lo + 1].seg;
    uint32_t top = r.seg_end;     // last layer that starts at or before the first chunk
    while (top - r.seg > 1) {
        const uint32_t mid = (r.seg + top) >> 1;
        if (lay.segs[mid].chunk_start <= r.first) r.seg = mid; else top = mid;
    }
    const SegDev sd = lay.segs[r.seg];
    if (r.first + r.nck <= lay.segs[r.seg + 1].chunk_start) r.seg_end = r.seg + 1;
    r.e0 = sd.offset + (r.first - sd.chunk_start) * kChunk;
    r.left = sd.offset + sd.length - r.e0;
    return r;
}
constexpr int kWSymLoads = (kChunk / 2 + 1 + 63) / 64;    // dword loads per lane to cover a chunk at any 2-byte offset (33)
constexpr uint32_t kWSymMask2 = (uint32_t)(kWideMaxA - 1) * 0x10001u;
// A wavefront's LDS words in the coder: 64 rows of 32 + 1 words and one word more.  They hold the staged symbols,
// then (symbols in registers) every lane's own codewords, then the chunk's words; the plain loops for long codes
// keep the symbols in the rows and use a small window behind them.
constexpr int kWRowWords = kWSymRow / 2 - 1;                      // 32
constexpr int kWRowStride = kWRowWords + 1;                       // odd: no bank conflicts
constexpr int kWRegion = kSubsPerChunk * kWRowStride + 1;         // 2113
constexpr int kWWinSlow = 128;
constexpr int kWWinMedium = 2048;                                // the rows' storage as a window
constexpr int kWPackWaveWords = kWRegion + kWWinSlow + 1;
constexpr size_t kWPackLds = sizeof(uint32_t) * (kWideMaxA + kWWaves * kWPackWaveWords);   // 52 KB: three workgroups per CU

// Step 1 of the coder: every lane concatenates the codewords of its 64 symbols (two per word of sym) from bit 0
// of its row, without knowing where they will land in the chunk; its bit count falls out at the end.  A
// codeword enters a 64-bit shift register; it completes at most one 32-bit word, which is stored without a
// branch (a store of the word still being filled is harmless: the slot is written again; stores beyond the row
// go to the row's spare slot).  A lane that met a kWFastSlow entry (a code of more than kWFastCodeBits bits, or
// a symbol without one: a handful of elements in a round of a large vector) codes its row again by itself in a
// rolled loop, its symbols parked in `scratch` (32 words), those entries taken from the table in device memory
// and appended in pieces; nocode counts its symbols without a code.  Returns, for the whole wavefront: kRowsOk;
// kRowsOverflow if a lane's codewords do not fit its row (bits is still every lane's bit count, and no lane met
// a kWFastSlow entry); kRowsSlow if more than kWRedoLanes lanes met one, or one did and a row overflowed.
enum { kRowsOk = 0, kRowsOverflow = 1, kRowsSlow = 2 };
constexpr int kWRedoLanes = 4;
template <bool kFull>
__device__ inline int w_pack_rows(const uint32_t (&sym)[kSub / 2], int cnt, const uint32_t *fast, const BookWide &book,
                                  uint32_t *region, uint32_t *scratch, uint32_t lane, uint32_t &bits, uint32_t &nocode)
{
    uint64_t acc = 0;
    uint32_t np = 0;                                     // bits of acc not yet stored: < 32 between symbols
    const uint32_t row0 = lane * kWRowStride;
    uint32_t waddr = row0;
    const uint32_t wend = row0 + kWRowWords;
    bool left = false;
#pragma unroll
    for (int j = 0; j < kSub; ++j) {
        uint32_t e = fast[(j & 1) ? sym[j >> 1] >> 16 : sym[j >> 1] & 0xffffu];
        if (!kFull) e = (j < cnt) ? e : 0u;              // nothing to append beyond the chunk's end
        const uint32_t L = e >> kWFastCodeBits;          // <= kWFastCodeBits, or kWFastSlow
        np += L;
        left = left || np > 63u;                         // exactly the kWFastSlow entries
        acc = (acc << (L & 63u)) | (e & ((1u << kWFastCodeBits) - 1u));
        const uint32_t rest = np & 31u;
        region[waddr < wend ? waddr : wend] = (uint32_t)(acc >> rest);
        waddr += (np >> 5) & 1u;
        np = rest;
    }
    nocode = 0;
    const uint64_t slow_lanes = __ballot(left);
    if (slow_lanes) {
        if (__popcll(slow_lanes) > kWRedoLanes) return kRowsSlow;
        for (uint64_t todo = slow_lanes; todo; todo &= todo - 1) {   // the same in every lane
            const uint32_t l = (uint32_t)__ffsll((long long)todo) - 1u;
            w_wave_sync_lds();                                       // the scratch words are free
            if (lane == l) {
#pragma unroll
                for (int jj = 0; jj < kSub / 2; ++jj) scratch[jj] = sym[jj];
            }
            w_wave_sync_lds();
            if (lane == l) {
                const uint16_t *mine = reinterpret_cast<const uint16_t *>(scratch);
                acc = 0; np = 0; waddr = row0;
                for (int j = 0; j < (kFull ? kSub : cnt); ++j) {
                    const uint32_t sj = mine[j];
                    const uint32_t e = fast[sj];
                    uint32_t L = e >> kWFastCodeBits;
                    uint64_t code = e & ((1u << kWFastCodeBits) - 1u);
                    if (L == kWFastSlow) {
                        L = book.len[sj];
                        code = book.code[sj];
                        nocode += L == 0u ? 1u : 0u;
                    }
                    while (L) {   // the codeword's leading bits first, at most kWFastCodeBits at a time
                        const uint32_t piece = L < kWFastCodeBits ? L : kWFastCodeBits;
                        L -= piece;
                        np += piece;
                        acc = (acc << piece) | ((code >> L) & ((1ull << piece) - 1ull));
                        const uint32_t rest = np & 31u;
                        region[waddr < wend ? waddr : wend] = (uint32_t)(acc >> rest);
                        waddr += (np >> 5) & 1u;
                        np = rest;
                    }
                }
            }
        }
    }
    const uint32_t whole = waddr - row0;                 // complete words, counted also beyond the row
    if (np) region[waddr < wend ? waddr : wend] = (uint32_t)(acc << (32u - np));
    bits = whole * 32u + np;
    if (__any(whole + (np ? 1u : 0u) > (uint32_t)kWRowWords)) return slow_lanes ? kRowsSlow : kRowsOverflow;
    return kRowsOk;
}

// Step 2: every lane's row holds its `bits` bits; excl: bits of the lanes before it.  The rows go to registers,
// their storage is cleared and becomes the chunk's words: every lane ORs its words in, shifted by its offset.
// On return region[0 .. nwords) holds them, nwords = ceil(sum of bits / 32) <= 64 x 32.
__device__ inline void w_rows_to_window(uint32_t *region, uint32_t lane, uint32_t bits, uint32_t excl, uint32_t nwords)
{
    const uint32_t nw = (bits + 31u) >> 5;               // <= kWRowWords
    uint32_t maxnw = nw;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { const uint32_t y = (uint32_t)__shfl_xor((int)maxnw, o, 64); maxnw = maxnw > y ? maxnw : y; }
    uint32_t r[kWRowWords];
    const uint32_t *row = region + lane * kWRowStride;
#pragma unroll
    for (int i = 0; i < kWRowWords; ++i) {
        r[i] = 0u;
        if ((uint32_t)i < maxnw) r[i] = (uint32_t)i < nw ? row[i] : 0u;
    }
    w_wave_sync_lds();                                   // all rows are in registers
    for (uint32_t i = lane; i <= nwords; i += 64) region[i] = 0u;
    w_wave_sync_lds();
    const uint32_t sh = excl & 31u, w0 = excl >> 5;
    uint32_t prev = 0u;
#pragma unroll
    for (int i = 0; i < kWRowWords; ++i) {
        if ((uint32_t)i < maxnw) {
            const uint32_t out = __builtin_amdgcn_alignbit(prev, r[i], sh);   // ({prev, r[i]} >> sh), low word
            if (out) atomicOr(&region[w0 + (uint32_t)i], out);
            prev = r[i];
        }
    }
    const uint32_t tail = __builtin_amdgcn_alignbit(prev, 0u, sh);   // what the shift pushed out of the last word
    if (sh && tail && nw) atomicOr(&region[w0 + nw], tail);
    w_wave_sync_lds();
}

__global__ __launch_bounds__(kWThreads) void k_chunk_bits_wide(Layout lay, const uint16_t *__restrict__ sym,
                                                              uint64_t sym_stride, const BookWide *__restrict__ books,
                                                              uint32_t *__restrict__ chunk_bits, const RunDev *__restrict__ runs,
                                                              uint32_t nrun, uint32_t cpw)
{
    __shared__ uint8_t s_len[kWideMaxA];
    const uint32_t lane = threadIdx.x & 63, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t u = blockIdx.y;
    const WRange wg = w_range(lay, runs, nrun, u, blockIdx.x, cpw);
    for (uint32_t i = threadIdx.x; i < (uint32_t)kWideMaxA; i += kWThreads)
        s_len[i] = i < lay.A ? books[wg.book].len[i] : (uint8_t)0;
    __syncthreads();
    for (uint32_t i_ck = wave; i_ck < wg.nck; i_ck += kWWaves) {   // whole wavefronts; no workgroup barriers below
        const uint64_t c = wg.first + i_ck;
        uint64_t e0;
        uint32_t n;
        wg.place(lay.segs, i_ck, e0, n);
        const uint16_t *src = sym + (uint64_t)u * sym_stride + e0;
        uint32_t total = 0;
        if ((reinterpret_cast<uintptr_t>(src) & 15u) == 0) {   // eight symbols per load
            const uint4 *src8 = reinterpret_cast<const uint4 *>(src);
            uint4 v[kChunk / 8 / 64];   // a whole chunk is eight loads per lane, all requested before the first is used
#pragma unroll
            for (int r = 0; r < kChunk / 8 / 64; ++r) {
                const uint32_t i = lane + 64u * r;
                v[r] = i < (n >> 3) ? src8[i] : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int r = 0; r < kChunk / 8 / 64; ++r) {
                if (lane + 64u * r >= (n >> 3)) continue;
                const uint32_t w[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    total += (uint32_t)s_len[w[q] & (kWideMaxA - 1)] + (uint32_t)s_len[(w[q] >> 16) & (kWideMaxA - 1)];
            }
            for (uint32_t e = (n & ~7u) + lane; e < n; e += 64) total += s_len[src[e] & (kWideMaxA - 1)];
        } else {   // any element offset: dwords from the 4-byte boundary below the chunk, requested together
            const uint32_t shift = (uint32_t)(reinterpret_cast<uintptr_t>(src) >> 1) & 1u;
            const uint32_t *src32 = reinterpret_cast<const uint32_t *>(src - shift);
            const uint32_t end = shift + n;          // symbols from the boundary
            uint32_t v[kWSymLoads];
#pragma unroll
            for (int r = 0; r < kWSymLoads; ++r) {
                const uint32_t i = lane + 64u * r;
                v[r] = i < ((end + 1u) >> 1) ? src32[i] : 0u;
            }
#pragma unroll
            for (int r = 0; r < kWSymLoads; ++r) {
                const uint32_t p = 2u * (lane + 64u * r);   // position of the low half
                const uint32_t l0 = s_len[v[r] & (kWideMaxA - 1)], l1 = s_len[(v[r] >> 16) & (kWideMaxA - 1)];
                total += (p >= shift && p < end ? l0 : 0u) + (p + 1u < end ? l1 : 0u);
            }
        }
        total = w_wave_sum(total);
        if (lane == 0) chunk_bits[(uint64_t)u * lay.nchunks + c] = total;
    }
}

// A chunk's coded sub-chunks: `rows` says where the codewords are (w_pack_rows), bits and excl are the lane's own and
// those of the lanes before it, nwords the words of the whole chunk.
struct WCoded {
    uint32_t bits, excl, nwords;
    int rows;
};

// What the plain loops know of a symbol: from the table in LDS where that holds the symbol's code, else from device memory.
__device__ inline void w_lookup(const uint32_t *fast, const BookWide &book, uint32_t s, uint32_t &L, uint64_t &code)
{
    const uint32_t e = fast[s];
    L = e >> kWFastCodeBits;
    code = e & ((1u << kWFastCodeBits) - 1u);
    if (L == kWFastSlow) { L = book.len[s]; code = book.code[s]; }
}

// Codes a wavefront's chunk, lane l its sub-chunk of cnt symbols in sym (two per word); whole: every lane has kSub.
// Where rows says kRowsOk, w_rows_to_window makes the chunk's words of the rows.
__device__ inline WCoded w_code_chunk(const uint32_t (&sym)[kSub / 2], int cnt, bool whole, const uint32_t *fast,
                                      const BookWide &book, uint32_t *region, uint32_t lane, uint64_t *status)
{
    WCoded r;
    r.bits = 0;
    uint32_t nocode = 0;
    r.rows = whole ? w_pack_rows<true>(sym, cnt, fast, book, region, region + kWRegion, lane, r.bits, nocode)
                   : w_pack_rows<false>(sym, cnt, fast, book, region, region + kWRegion, lane, r.bits, nocode);
    if (r.rows == kRowsSlow) {
        // long codes or symbols without one in more than a few lanes: the symbols go back to the rows, plain loops
        uint32_t *row32 = region + lane * kWRowStride;
        w_wave_sync_lds();
#pragma unroll
        for (int jj = 0; jj < kSub / 2; ++jj) row32[jj] = sym[jj];
        w_wave_sync_lds();
        const uint16_t *row = reinterpret_cast<const uint16_t *>(row32);
        nocode = 0;      // (the rows' redone lanes are counted here again)
        r.bits = 0;
        for (int j = 0; j < cnt; ++j) {
            uint32_t L;
            uint64_t code;
            w_lookup(fast, book, row[j], L, code);
            nocode += L == 0u ? 1u : 0u;
            r.bits += L;
        }
    }
    if (nocode)
        atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_NOCODE), (unsigned long long)nocode);
    const uint32_t incl = w_wave_inclusive_scan(r.bits, lane);
    r.excl = incl - r.bits;
    r.nwords = ((uint32_t)__shfl(incl, 63, 64) + 31u) >> 5;
    return r;
}

// Writes the words of a coded chunk to dst: the window, where there is one.
__device__ inline void w_store_chunk(const WCoded &r, const uint32_t (&sym)[kSub / 2], int cnt, const uint32_t *fast,
                                     const BookWide &book, uint32_t *region, uint32_t lane, uint32_t *dst)
{
    if (r.rows == kRowsOk) {
        for (uint32_t i = lane; i < r.nwords; i += 64) __builtin_nontemporal_store(region[i], dst + i);
        return;
    }
    // Rows too short for some lane (more than 16 bits per symbol on average): the codewords are appended at
    // their final bit offsets instead, entries from the table in LDS, the rows' storage as the window.  After
    // the plain loops above: the same from the rows' symbols, a small window behind them.
    const bool medium = r.rows == kRowsOverflow;
    const uint16_t *row = reinterpret_cast<const uint16_t *>(region + lane * kWRowStride);
    uint32_t *win = medium ? region : region + kWRegion;
    const uint32_t wcap = medium ? (uint32_t)kWWinMedium : (uint32_t)kWWinSlow;
    for (uint32_t wbase = 0; wbase < r.nwords; wbase += wcap) {
        const uint32_t wn = r.nwords - wbase < wcap ? r.nwords - wbase : wcap;
        w_wave_sync_lds();
        for (uint32_t i = lane; i <= wn; i += 64) win[i] = 0u;
        w_wave_sync_lds();
        uint32_t wi = (r.excl >> 5) - wbase;  // window word receiving the next completed 32 bits (may start below the window)
        uint32_t np = r.excl & 31u;           // bits pending in acc (the leading np bits belong to earlier lanes)
        uint64_t acc = 0;
        auto append = [&](uint64_t code, uint32_t L) {  // L <= 32, np < 32
            acc = (acc << L) | code;
            np += L;
            if (np >= 32u) {
                np -= 32u;
                if (wi < wn) atomicOr(&win[wi], (uint32_t)(acc >> np));  // unsigned: false below the window
                ++wi;
            }
        };
        // a lane whose bits all lie outside this window has nothing to add
        const bool overlaps = r.excl + r.bits > wbase * 32u && r.excl < (wbase + wn) * 32u;
        if (medium) {   // whole wavefront; every existing symbol has a code of at most kWFastCodeBits bits
#pragma unroll
            for (int j = 0; j < kSub; ++j) {
                const uint32_t e = fast[(j & 1) ? sym[j >> 1] >> 16 : sym[j >> 1] & 0xffffu];
                if (overlaps && j < cnt) append(e & ((1u << kWFastCodeBits) - 1u), e >> kWFastCodeBits);
            }
        }
        for (int j = 0; !medium && overlaps && j < cnt; ++j) {
            uint32_t L;
            uint64_t code;
            w_lookup(fast, book, row[j], L, code);
            if (!L) continue;
            if (L > 32u) {
                append(code >> 32, L - 32u);
                code &= 0xffffffffull;
                L = 32u;
            }
            append(code, L);
        }
        if (overlaps && np && wi < wn) atomicOr(&win[wi], (uint32_t)(acc << (32u - np)));
        w_wave_sync_lds();
        for (uint32_t i = lane; i < wn; i += 64) dst[wbase + i] = win[i];
        w_wave_sync_lds();
    }
}

__global__ __launch_bounds__(kWThreads, 3) void k_pack_wide(Layout lay, const uint16_t *__restrict__ sym, uint64_t sym_stride,
                                                        const BookWide *__restrict__ books,
                                                        const uint64_t *__restrict__ chunk_offset,
                                                        uint16_t *__restrict__ sub_bits, uint32_t *__restrict__ words,
                                                        uint64_t words_stride, uint64_t *__restrict__ status,
                                                        const RunDev *__restrict__ runs, uint32_t nrun, uint32_t cpw)
{
    extern __shared__ uint32_t wp_smem[];   // kWPackLds bytes
    uint32_t *s_fast = wp_smem;                      // [kWideMaxA]
    uint32_t *s_wave_all = s_fast + kWideMaxA;       // [kWWaves][kWPackWaveWords]
    const uint32_t lane = threadIdx.x & 63, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t u = blockIdx.y;
    const WRange wg = w_range(lay, runs, nrun, u, blockIdx.x, cpw);
    {
        const BookWide &tb = books[wg.book];
        uint32_t tab[kWideMaxA / kWThreads];   // the loads are issued together
#pragma unroll
        for (int r = 0; r < kWideMaxA / kWThreads; ++r) tab[r] = tb.fast[threadIdx.x + (uint32_t)r * kWThreads];
#pragma unroll
        for (int r = 0; r < kWideMaxA / kWThreads; ++r) s_fast[threadIdx.x + (uint32_t)r * kWThreads] = tab[r];
    }
    __syncthreads();
    const BookWide &book = books[wg.book];
    uint32_t *region = s_wave_all + wave * kWPackWaveWords;
    for (uint32_t i_ck = wave; i_ck < wg.nck; i_ck += kWWaves) {   // whole wavefronts; wavefront-level synchronisation only below
        const uint64_t c = wg.first + i_ck;
        uint64_t e0;
        uint32_t n;
        wg.place(lay.segs, i_ck, e0, n);
        const uint16_t *src = sym + (uint64_t)u * sym_stride + e0;
        // The chunk's symbols, at any 2-byte offset and of any length: coalesced dwords from the 4-byte boundary
        // below the chunk go to LDS rows of 32 + 1 words (word i of the chunk at i + i / 32), from which lane l
        // funnels its 64 symbols (words 32 l .. 32 l + 32) into registers, two per word.
        const uint32_t shift = (uint32_t)(reinterpret_cast<uintptr_t>(src) >> 1) & 1u;
        const uint32_t *src32 = reinterpret_cast<const uint32_t *>(src - shift);
        const uint32_t ndw = (shift + n + 1u) >> 1;      // <= kChunk / 2 + 1
        uint32_t tmp[kWSymLoads];
#pragma unroll
        for (int r = 0; r < kWSymLoads; ++r) {
            const uint32_t i = lane + 64u * r;
            tmp[r] = i < ndw ? __builtin_nontemporal_load(src32 + i) : 0u;   // all requested before the first is used
        }
        const uint64_t off = chunk_offset[(uint64_t)u * (lay.nchunks + 1) + c];
        w_wave_sync_lds();   // the previous chunk's words have been copied out
#pragma unroll
        for (int r = 0; r < kWSymLoads; ++r) {
            const uint32_t i = lane + 64u * r;
            if (i < (uint32_t)kChunk / 2 + 1) region[i + (i >> 5)] = tmp[r];   // word 2048 lands at 2112
        }
        w_wave_sync_lds();
        const int first = (int)lane * kSub;
        const int cnt = (int)n - first < 0 ? 0 : ((int)n - first > kSub ? kSub : (int)n - first);
        uint32_t *row32 = region + lane * kWRowStride;
        uint32_t symw[kSub / 2];
        {
            uint32_t cur = row32[0];
#pragma unroll
            for (int jj = 0; jj < kSub / 2; ++jj) {
                const uint32_t nxt = row32[jj + 1 + (jj == kSub / 2 - 1 ? 1 : 0)];   // row32[32] is the row's spare slot
                symw[jj] = (shift ? __builtin_amdgcn_alignbit(nxt, cur, 16u) : cur) & kWSymMask2;   // table indices stay below kWideMaxA
                cur = nxt;
            }
        }
        w_wave_sync_lds();   // every lane holds its symbols: the rows are free

        const WCoded coded = w_code_chunk(symw, cnt, n == (uint32_t)kChunk, s_fast, book, region, lane, status);
        sub_bits[((uint64_t)u * lay.nchunks + c) * kSubsPerChunk + lane] = (uint16_t)coded.bits;
        const uint64_t off_words = off >> 5;
        if (off_words + coded.nwords > words_stride) {   // whole wavefront
            if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CAPACITY), 1ull);
            continue;
        }
        uint32_t *dst = words + (uint64_t)u * words_stride + off_words;
        if (coded.rows == kRowsOk) {
            w_rows_to_window(region, lane, coded.bits, coded.excl, coded.nwords);
            for (uint32_t i = lane; i < coded.nwords; i += 64) __builtin_nontemporal_store(region[i], dst + i);
            continue;
        }
        w_store_chunk(coded, symw, cnt, s_fast, book, region, lane, dst);
    }
}

// ---- user side for a held code, in one sweep ------------------------------------------------------------------

// The same steps without the symbols ever reaching memory, as the byte path's k_encode_fused does it: a workgroup takes
// the next four chunks under one code table (its place from a ticket counter), a wavefront quantizes a chunk into LDS
// rows while it sums the code lengths, the size is published, and while the predecessors' sizes are looked up every
// wavefront codes its chunk.  The look-back and its bound are k_encode_fused's.
// Bound by the streams of g, m and m' (12 bytes an element; the three steps move 4 more for the symbols, and wait for
// one another): sixteen users of 25.6 M elements in [1,5,6], 1.64 ms in three steps, 1.04 in this, 5.2 TB/s.
// 52 KB of LDS (the table 16, a wavefront's rows 9) let three workgroups share a CU, so the registers are cut for that.
// A chunk starts at any element: its vectors are read and written at 4-byte alignment, which a vector access to device
// memory may have, so there is one path for whole chunks and one, element by element, for a layer's ragged last one.
// kSR: the stochastic conversion.  A vector's four random words are one Philox block, so layers have to start at
// multiples of four elements (lay.vec_aligned).
typedef float wf4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kWfBatch = 4;                                   // vectors of g (and of m) a lane requests at a time
constexpr int kWfBatches = kChunk / 4 / 64 / kWfBatch;
constexpr int kWfScalar = 8;                                  // element rounds a lane requests together
static_assert(kChunk % (4 * 64 * kWfBatch) == 0 && kChunk % (64 * kWfScalar) == 0, "whole batches per chunk");

__device__ inline void w_lds_barrier()   // orders LDS accesses only: nobody here reads the stores to memory that are under way
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <bool kSR>
__global__ __launch_bounds__(kWThreads, 3) void k_encode_wide(
    Layout lay, const float *__restrict__ g, const float *m, float *m_out, uint64_t row_stride, float gamma, uint64_t seed,
    const BookWide *__restrict__ books, uint64_t *lookback, uint32_t nwg, uint32_t spin_limit,
    uint64_t *__restrict__ chunk_offset, uint16_t *__restrict__ sub_bits, uint64_t *__restrict__ payload_bits,
    uint32_t *__restrict__ words, uint64_t words_stride, uint64_t *__restrict__ status, const RunDev *__restrict__ runs,
    uint32_t nrun)
{
    __shared__ uint32_t s_fast[kWideMaxA];
    __shared__ uint32_t s_wave_all[kWWaves * kWPackWaveWords];
    __shared__ uint32_t s_cbits[kWWaves];
    __shared__ uint64_t s_prefix;
    __shared__ uint32_t s_ticket, s_stalled;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t u = blockIdx.y;
    uint64_t *state = lookback + (uint64_t)u * (nwg + 1ull) + 1;   // a user's ticket counter lies in front of its entries

    if (t == 0) s_ticket = atomicAdd(reinterpret_cast<uint32_t *>(state - 1), 1u);
    w_lds_barrier();
    const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_ticket);   // < nwg = gridDim.x
    const WRange wg = w_range(lay, runs, nrun, u, b, 1u);
    const bool active = wave < wg.nck;
    const BookWide &book = books[wg.book];
    uint32_t *region = s_wave_all + wave * kWPackWaveWords;
    uint64_t e0 = 0;
    uint32_t n = 0;
    if (active) wg.place(lay.segs, wave, e0, n);
    const float *gu = g + (uint64_t)u * row_stride + e0;
    const float *mu = m + (uint64_t)u * row_stride + e0;
    float *mo = m_out + (uint64_t)u * row_stride + e0;
    const bool whole = n == (uint32_t)kChunk;

    // The code's table is requested first and stored to LDS when the first vectors are under way.
    uint32_t tab[kWideMaxA / kWThreads];
#pragma unroll
    for (int r = 0; r < kWideMaxA / kWThreads; ++r) tab[r] = book.fast[t + (uint32_t)r * kWThreads];
    wf4u gn[kWfBatch], mn[kWfBatch];
    if (whole) {
#pragma unroll
        for (int r = 0; r < kWfBatch; ++r) {
            const uint32_t i = 4u * (lane + 64u * (uint32_t)r);
            gn[r] = __builtin_nontemporal_load(reinterpret_cast<const wf4u *>(gu + i));
            mn[r] = __builtin_nontemporal_load(reinterpret_cast<const wf4u *>(mu + i));
        }
    }
#pragma unroll
    for (int r = 0; r < kWideMaxA / kWThreads; ++r) s_fast[t + (uint32_t)r * kWThreads] = tab[r];
    w_lds_barrier();

    // ---- 1. wavefront w quantizes chunk w: two symbols a word, word i at i + i / 32 of its rows ---------------------
    const uint32_t sign_shift = lay.E + lay.M;
    uint32_t len_sum = 0, n_nonfinite = 0, n_clamped = 0;
    if (active) {
        // the chunk's layer: last one that starts at or before the chunk
        uint32_t seg = wg.seg, seg_end = wg.seg_end;
        while (seg_end - seg > 1) {
            const uint32_t mid = (seg + seg_end) >> 1;
            if (lay.segs[mid].chunk_start <= wg.first + wave) seg = mid; else seg_end = mid;
        }
        const uint64_t pair = (uint64_t)u * lay.nseg + seg;
        const int bias = lay.bias[pair];
        const QConst qc = make_qconst(lay.E, lay.M, bias);
        const float gain = lay.gain[2 * pair], inv_gain = lay.gain[2 * pair + 1];
        // an entry of the table holds the length of a code of up to kWFastCodeBits bits
        auto code_len = [&](uint32_t s, uint32_t e) { return e >> kWFastCodeBits == kWFastSlow ? (uint32_t)book.len[s] : e >> kWFastCodeBits; };
        if (whole) {
#pragma unroll 1
            for (int bt = 0; bt < kWfBatches; ++bt) {
                wf4u gc[kWfBatch], mc[kWfBatch];
#pragma unroll
                for (int r = 0; r < kWfBatch; ++r) { gc[r] = gn[r]; mc[r] = mn[r]; }
                if (bt + 1 < kWfBatches) {
#pragma unroll
                    for (int r = 0; r < kWfBatch; ++r) {
                        const uint32_t i = 4u * (lane + 64u * (uint32_t)((bt + 1) * kWfBatch + r));
                        gn[r] = __builtin_nontemporal_load(reinterpret_cast<const wf4u *>(gu + i));
                        mn[r] = __builtin_nontemporal_load(reinterpret_cast<const wf4u *>(mu + i));
                    }
                }
#pragma unroll
                for (int r = 0; r < kWfBatch; ++r) {
                    const uint32_t k = lane + 64u * (uint32_t)(bt * kWfBatch + r);   // vector of the chunk
                    wf4u eo;
                    uint32_t sp[4], en[4];
                    Philox4 rw;
                    if constexpr (kSR) rw = element_random_words(e0 + 4u * k, u, seed);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float v = __fadd_rn(gc[r][j], __fmul_rn(gamma, mc[r][j]));
                        const float y = __fmul_rn(v, gain);
                        uint32_t s, flags;
                        float q;
                        if constexpr (kSR) quantize_stochastic(y, qc, lay.E, lay.M, bias, sign_shift, rw.w[j], s, q, flags);
                        else quantize(y, qc, sign_shift, s, q, flags);
                        q = __fmul_rn(q, inv_gain);
                        eo[j] = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
                        n_nonfinite += flags & 1u;
                        n_clamped += (flags >> 1) & 1u;
                        sp[j] = s & (uint32_t)(kWideMaxA - 1);
                        en[j] = s_fast[sp[j]];
                    }
                    __builtin_nontemporal_store(eo, reinterpret_cast<wf4u *>(mo + 4u * k));
                    const uint32_t at = 2u * k + ((2u * k) >> 5);   // both words lie in one row
                    region[at] = sp[0] | (sp[1] << 16);
                    region[at + 1u] = sp[2] | (sp[3] << 16);
                    const uint32_t top = max(max(en[0], en[1]), max(en[2], en[3]));
                    if (__any(top >= (kWFastSlow << kWFastCodeBits))) {   // a long code, or a symbol without one
#pragma unroll
                        for (int j = 0; j < 4; ++j) len_sum += code_len(sp[j], en[j]);
                    } else {
                        len_sum += (en[0] >> kWFastCodeBits) + (en[1] >> kWFastCodeBits) + (en[2] >> kWFastCodeBits) +
                                   (en[3] >> kWFastCodeBits);
                    }
                }
            }
        } else {
            uint16_t *half = reinterpret_cast<uint16_t *>(region);
            for (uint32_t base = 0; base < n; base += 64u * kWfScalar) {
                float gs[kWfScalar], ms[kWfScalar];
#pragma unroll
                for (int r = 0; r < kWfScalar; ++r) {
                    const uint32_t j = base + lane + 64u * (uint32_t)r;
                    gs[r] = j < n ? gu[j] : 0.0f;
                    ms[r] = j < n ? mu[j] : 0.0f;
                }
#pragma unroll
                for (int r = 0; r < kWfScalar; ++r) {
                    const uint32_t j = base + lane + 64u * (uint32_t)r;   // < kChunk: base is a multiple of 64 kWfScalar
                    if (j < n) {
                        const float v = __fadd_rn(gs[r], __fmul_rn(gamma, ms[r]));
                        const float y = __fmul_rn(v, gain);
                        uint32_t s, flags;
                        float q;
                        if constexpr (kSR)
                            quantize_stochastic(y, qc, lay.E, lay.M, bias, sign_shift,
                                                element_random_words(e0 + j, u, seed).w[(e0 + j) & 3u], s, q, flags);
                        else quantize(y, qc, sign_shift, s, q, flags);
                        q = __fmul_rn(q, inv_gain);
                        mo[j] = (flags & 1u) ? 0.0f : __fsub_rn(v, q);
                        n_nonfinite += flags & 1u;
                        n_clamped += (flags >> 1) & 1u;
                        s &= (uint32_t)(kWideMaxA - 1);
                        len_sum += code_len(s, s_fast[s]);
                        half[j + 2u * (j >> 6)] = (uint16_t)s;
                    }
                }
            }
        }
        if (n_nonfinite)
            atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_NONFINITE), (unsigned long long)n_nonfinite);
        if (n_clamped)
            atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CLAMPED), (unsigned long long)n_clamped);
    }
    len_sum = w_wave_sum(len_sum);
    if (lane == 0) s_cbits[wave] = len_sum;      // 0 for a wavefront without a chunk
    w_lds_barrier();

    // ---- 2. the workgroup's size is published, its predecessors' are requested ---------------------------------------
    uint32_t before = 0, own = 0, pay = 0;       // 32-bit-rounded sizes of the chunks ahead of this one, of all; exact size
#pragma unroll
    for (int k = 0; k < kWWaves; ++k) {
        const uint32_t cbits = s_cbits[k], a = (cbits + 31u) & ~31u;
        if ((uint32_t)k < wave) before += a;
        own += a;
        pay += cbits;
    }
    if (t == 0) lookback_publish(state, b, own);   // by the lane that looks back: an entry has one writer
    const uint64_t lb_first = wave == 0 ? lookback_first(state, b, lane) : 0ull;

    // ---- 3. wavefront = chunk, lane = sub-chunk: the chunk's words, from a word boundary on ----------------------
    const int first = (int)lane * kSub;
    const int cnt = (int)n - first < 0 ? 0 : ((int)n - first > kSub ? kSub : (int)n - first);
    uint32_t symw[kSub / 2];
    WCoded coded = {0u, 0u, 0u, kRowsOk};
    if (active) {
        const uint32_t *row32 = region + lane * kWRowStride;
#pragma unroll
        for (int jj = 0; jj < kSub / 2; ++jj) symw[jj] = row32[jj] & kWSymMask2;   // (beyond a ragged chunk's end: stale words)
        w_wave_sync_lds();   // every lane holds its symbols: the rows are free
        coded = w_code_chunk(symw, cnt, whole, s_fast, book, region, lane, status);
        sub_bits[((uint64_t)u * lay.nchunks + wg.first + wave) * kSubsPerChunk + lane] = (uint16_t)coded.bits;
        if (coded.rows == kRowsOk) w_rows_to_window(region, lane, coded.bits, coded.excl, coded.nwords);
    }
    if (wave == 0) {
        uint64_t prefix;
        const bool ok = lookback_collect(state, b, lb_first, lane, spin_limit, prefix);
        if (lane == 0) {
            lookback_finish(state, b, ok, prefix, own, status);
            s_prefix = prefix;
            s_stalled = ok ? 0u : 1u;
            atomicAdd(reinterpret_cast<unsigned long long *>(payload_bits + u), (unsigned long long)pay);
        }
    }
    w_lds_barrier();
    if (!active || s_stalled) return;   // whole wavefronts; no workgroup barrier below

    // ---- 4. the chunk's words go to their place in the stream -------------------------------------------------------
    const uint64_t off = s_prefix + before, c = wg.first + wave;
    if (lane == 0) {
        uint64_t *co = chunk_offset + (uint64_t)u * (lay.nchunks + 1);
        co[c] = off;
        if (c + 1 == lay.nchunks) co[lay.nchunks] = off + ((uint64_t)coded.nwords << 5);
    }
    const uint64_t off_words = off >> 5;
    if (off_words + coded.nwords > words_stride) {
        if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CAPACITY), 1ull);
        return;
    }
    w_store_chunk(coded, symw, cnt, s_fast, book, region, lane, words + (uint64_t)u * words_stride + off_words);
}

// ---- launchers ----------------------------------------------------------------------------------------------

static inline size_t w_up256(size_t x) { return (x + 255) & ~(size_t)255; }

// partial symbol counts, chunk sizes, and (for a fixed code without a symbol buffer) the symbols and their counts
size_t wide_workspace_bytes(const Layout &lay)
{
    const size_t sym_stride = (size_t)symbol_row_stride(lay.d);
    return w_up256((size_t)kHistGlobalRep * lay.nbooks * lay.A * sizeof(uint64_t)) +
           w_up256((size_t)lay.U * lay.nchunks * sizeof(uint32_t)) + w_up256((size_t)lay.nbooks * lay.A * sizeof(uint64_t)) +
           w_up256(sym_stride * lay.U * sizeof(uint16_t) + 32) + 512;
}

hipError_t launch_build_books_wide(BookWide *books, uint32_t nbooks, uint32_t A, const uint64_t *weights,
                                   uint64_t *status, hipStream_t s)
{
    if (nbooks == 0) return hipSuccess;
    const size_t lds = (size_t)2 * A * (sizeof(uint64_t) + sizeof(int)) + (size_t)A * 2 * sizeof(uint16_t);   // 112 KB at A = 4096
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_build_books_wide),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(K_BUILD_BOOKS, s);
    hipLaunchKernelGGL(k_build_books_wide, dim3(nbooks), dim3(kWbThreads), lds, s, books, A, weights, status);
    return hipGetLastError();
}

// The single sweep's look-back entries, a ticket counter in front of every user's.
static uint64_t sweep_entries(const Layout &lay, const WideCut &cut) { return (uint64_t)lay.U * (cut.nwg_small + 1ull); }

// A held code whose symbols and counts nobody asks for is coded in one sweep: it moves 12 bytes an element beside the
// streams, the three steps 16.  They keep the stochastic conversion of layers off the four-element grid (a vector's four
// random words are one block of the generator), and a plan whose workgroups are so many, with tables that change every
// few elements, that their entries do not fit the workspace laid out for the three steps.
static bool sweep_fits(const Layout &lay, const WideCut &cut, const co3_encode_args &a)
{
    return a.mode == CO3_BOOK_FIXED && !a.symbols && !a.hist && lay.nchunks &&
           (a.rounding != CO3_ROUND_STOCHASTIC || lay.vec_aligned) &&
           sweep_entries(lay, cut) * sizeof(uint64_t) + 256 <= wide_workspace_bytes(lay);
}

hipError_t launch_encode_wide(const Layout &lay, const WideCut &cut, const co3_encode_args &a, BookWide *books, void *workspace,
                              hipStream_t s)
{
    if (lay.U == 0) return hipSuccess;
    if (sweep_fits(lay, cut, a)) {
        uint64_t *lookback = reinterpret_cast<uint64_t *>((reinterpret_cast<uintptr_t>(workspace) + 255u) & ~(uintptr_t)255u);
        const uint64_t nlb = sweep_entries(lay, cut);
        {
            ProfScope prof(K_ZERO, s);
            hipLaunchKernelGGL(k_zero_wide, dim3((uint32_t)((nlb + 255) / 256)), dim3(256), 0, s, lookback, nlb, a.payload_bits,
                               lay.U);
        }
        ProfScope prof(K_FUSED, s);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(cut.nwg_small, lay.U), dim3(kWThreads), 0, s, lay, a.g, a.m, a.m_out, a.row_stride,
                               a.gamma, a.seed, static_cast<const BookWide *>(books), lookback, cut.nwg_small,
                               lookback_polls(), a.chunk_offset, a.sub_bits, a.payload_bits, a.words, a.words_stride,
                               a.status, cut.runs, cut.nrun);
        };
        if (a.rounding == CO3_ROUND_STOCHASTIC) launch(k_encode_wide<true>);
        else launch(k_encode_wide<false>);
        return hipGetLastError();
    }
    const uint64_t sym_stride = symbol_row_stride(lay.d);
    const uint64_t hist_n = (uint64_t)lay.nbooks * lay.A, hist_rep_n = (uint64_t)kHistGlobalRep * hist_n;
    uintptr_t p = (reinterpret_cast<uintptr_t>(workspace) + 255u) & ~(uintptr_t)255u;
    uint64_t *hist_rep = reinterpret_cast<uint64_t *>(p);
    p += w_up256(hist_rep_n * sizeof(uint64_t));
    uint32_t *chunk_bits = reinterpret_cast<uint32_t *>(p);
    p += w_up256((size_t)lay.U * lay.nchunks * sizeof(uint32_t));
    uint64_t *ws_hist = reinterpret_cast<uint64_t *>(p);
    p += w_up256(hist_n * sizeof(uint64_t));
    uint16_t *ws_sym = reinterpret_cast<uint16_t *>(p);
    // a fixed code without a symbol buffer: the symbols (and their counts, unused) stay in the workspace
    uint16_t *sym = a.symbols ? reinterpret_cast<uint16_t *>(a.symbols) : ws_sym;
    uint64_t *hist = a.hist ? a.hist : ws_hist;
    // a code that is held and layers on the quantizer's tile grid: the chunks' sizes come out of the first sweep
    const bool bits_in_sweep = a.mode == CO3_BOOK_FIXED && lay.tile_aligned && lay.nchunks;
    {
        // the partial counts and, behind them in the workspace, the chunk sizes the sweep adds to
        const uint64_t zero_n = bits_in_sweep ? (w_up256(hist_rep_n * sizeof(uint64_t)) + w_up256((size_t)lay.U * lay.nchunks * sizeof(uint32_t))) / sizeof(uint64_t)
                                              : hist_rep_n;
        ProfScope prof(K_ZERO, s);
        hipLaunchKernelGGL(k_zero_wide, dim3((uint32_t)((zero_n + 255) / 256)), dim3(256), 0, s, hist_rep, zero_n, a.payload_bits, 0u);
    }
    if (lay.d) {
        ProfScope prof(K_QUANTIZE, s);
        const uint64_t ntiles = (lay.d + kWqTile - 1) / kWqTile, per = ntiles * lay.U / kWqGrid;
        const uint32_t tiles = per < 1 ? 1u : per < kWqTiles ? (uint32_t)per : kWqTiles;
        const dim3 grid((uint32_t)((ntiles + tiles - 1) / tiles), lay.U);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(kWqThreads), 0, s, lay, a.g, a.m, a.m_out, sym, sym_stride, a.row_stride,
                               a.gamma, a.seed, hist_rep, static_cast<const BookWide *>(books), chunk_bits, a.status, tiles);
        };
        if (a.rounding == CO3_ROUND_STOCHASTIC) {
            if (bits_in_sweep) launch(k_quantize_wide<true, true>);
            else launch(k_quantize_wide<true, false>);
        } else {
            if (bits_in_sweep) launch(k_quantize_wide<false, true>);
            else launch(k_quantize_wide<false, false>);
        }
    }
    {
        ProfScope prof(K_REDUCE_HIST, s);
        hipLaunchKernelGGL(k_reduce_hist_wide, dim3((uint32_t)((hist_n + 255) / 256)), dim3(256), 0, s, hist_rep, hist, hist_n);
    }
    if (a.mode == CO3_BOOK_EMPIRICAL) {
        hipError_t e = launch_build_books_wide(books, lay.nbooks, lay.A, hist, a.status, s);
        if (e != hipSuccess) return e;
    }
    const uint32_t cpw = w_chunks_per_wave(lay, cut);
    const uint32_t gx = cpw * kWWaves == kWgChunksSmall ? cut.nwg_small : cut.nwg;
    if (lay.nchunks && !bits_in_sweep) {
        ProfScope prof(K_CHUNK_BITS, s);
        hipLaunchKernelGGL(k_chunk_bits_wide, dim3(gx, lay.U), dim3(kWThreads), 0, s, lay, sym, sym_stride, books, chunk_bits,
                           cut.runs, cut.nrun, cpw);
    }
    hipError_t e = launch_scan_chunks(lay, chunk_bits, a.chunk_offset, a.payload_bits, s);   // the byte path's scan
    if (e != hipSuccess) return e;
    if (lay.nchunks) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_pack_wide), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kWPackLds);
        if (e != hipSuccess) return e;
        ProfScope prof(K_PACK, s);
        hipLaunchKernelGGL(k_pack_wide, dim3(gx, lay.U), dim3(kWThreads), kWPackLds, s, lay, sym, sym_stride, books,
                           a.chunk_offset, a.sub_bits, a.words, a.words_stride, a.status, cut.runs, cut.nrun, cpw);
    }
    return hipGetLastError();
}

}  // namespace co3
