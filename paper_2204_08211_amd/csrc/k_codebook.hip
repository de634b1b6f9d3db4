// Huffman code tables built on the device from symbol counts (Sec. IV-A (ii)), one workgroup
// per table, so that an encoder using this round's histogram needs no host round trip.
//
// Same tie rule and canonical form as the host builder: leaves sorted by (weight, symbol),
// internal nodes in creation order, merge the two smallest with leaves first on equal weight.
// The merge runs in rounds that each pair off every node the serial merge would take before any
// node it has yet to create; a table of 256 symbols takes some twenty rounds.
//
// What bounds it is the chain of dependent LDS accesses in one workgroup, not the work, so whatever was a loop of one
// thread over the lengths is a scan over the lanes, and the merge runs in one wavefront without barriers (one user of
// 2^20 elements in [1,3,0] with the code rebuilt, the whole round: 64.9 -> 52.2 us; tables of 256 symbols save more).
#include "co3_internal.h"
#include "pack_core.h"
#include "quantize_math.h"

namespace co3 {

constexpr int kCbThreads = 256;

// x of a lane, the same in all of them.
__device__ inline uint64_t lane_value(uint64_t x, int lane)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane) << 32;
}

// counts: `weights` are the sweep's kHistGlobalRep partial tables of symbol counts, one table of all codes after the
// other; their sum is the weight and is left in `counts` (a kernel of its own for it was another 3.4 to 5 us).
__global__ __launch_bounds__(kCbThreads) void k_build_books(BookDev *__restrict__ books, int E, int M,
                                                           const uint64_t *__restrict__ weights,
                                                           uint64_t *__restrict__ counts,
                                                           uint64_t *__restrict__ status)
{
    BookDev &B = books[blockIdx.x];
    const uint32_t A = 1u << (1 + E + M);
    const uint64_t *w = weights + (uint64_t)blockIdx.x * A;
    const int t = threadIdx.x;

    __shared__ uint64_t lw[kMaxA];        // weight of symbol t
    __shared__ uint64_t nw[2 * kMaxA];    // node weights: sorted leaves, then internal nodes
    __shared__ int parent[2 * kMaxA];
    __shared__ uint32_t leaf_sym[kMaxA];  // sorted leaf -> symbol
    __shared__ uint32_t slen[kMaxA];      // symbol -> length
    __shared__ uint32_t cnt[65], off[65];
    __shared__ uint64_t first[65];
    __shared__ uint32_t sorted[kMaxA];
    __shared__ uint32_t wcnt[kCbThreads / 64][65];   // codes of every length per wavefront of symbols
    __shared__ uint32_t limit[32];        // a window's complement <= limit[l] (and not 0): its code has more than l bits
    __shared__ uint32_t base[65];         // a code of l bits has rank base[l] + code
    __shared__ uint32_t entry_sym[kMaxA];   // what a decode table's entry carries, by rank
    __shared__ int err;

    uint64_t myw = 0;
    if (t < (int)A) {
        if (counts) {
            const uint64_t n = (uint64_t)gridDim.x * A;
#pragma unroll 16
            for (int r = 0; r < kHistGlobalRep; ++r) myw += w[(uint64_t)r * n + t];
            counts[(uint64_t)blockIdx.x * A + t] = myw;
        } else {
            myw = w[t];
        }
    }
    slen[t] = 0;
    parent[t] = -1;
    parent[t + kMaxA] = -1;
    for (int i = t; i < (kCbThreads / 64) * 65; i += kCbThreads) (&wcnt[0][0])[i] = 0;
    if (t == 0) { cnt[0] = 0; off[0] = 0; first[0] = 0; }
    if (t == 0) err = 0;
    __syncthreads();
    // 2^64 - 1 marks an exhausted queue in the merge below; as a weight it is refused, like the
    // host builder refuses it (the table's weights would sum to 2^64 - 1 or more)
    if (myw == ~0ull) err = 1;
    const int n = __syncthreads_count(myw > 0);

    // rank of this leaf in (weight, symbol) order among the active symbols; an inactive one counts as heavier than
    // all.  Of equal weights the earlier symbol comes first, so a symbol of an earlier wavefront counts up to this
    // weight and one of a later wavefront below it: only the thread's own wavefront compares the symbols as well.
    lw[t] = myw ? myw : ~0ull;
    __syncthreads();
    {
        const int w0 = t & ~63, a = (int)A;
        int rank = 0;
#pragma unroll 8
        for (int j = 0; j < (w0 < a ? w0 : a); ++j) rank += lw[j] <= myw;
#pragma unroll 8
        for (int j = w0; j < (w0 + 64 < a ? w0 + 64 : a); ++j) rank += lw[j] < myw + (uint64_t)(j < t);
#pragma unroll 8
        for (int j = w0 + 64; j < a; ++j) rank += lw[j] < myw;
        if (myw > 0 && myw != ~0ull) {
            nw[rank] = myw;
            leaf_sym[rank] = t;
        }
    }
    __syncthreads();

    // The two-queue merge in rounds.  With T the sum of the two lightest nodes alive, every internal node alive and
    // every leaf of weight <= T is taken before any node created from now on (their weights are >= T; on equal
    // weights a leaf goes before an internal node and an older internal node before a newer one).  So the merged
    // order of those nodes pairs off two by two exactly as the serial merge would; an odd one out stays at the head of
    // its queue.  One wavefront runs the rounds, a pair a lane: the rounds of a table average n / 10 nodes, and without
    // the other wavefronts a round needs no barrier.
    // A lane finds where its pair begins in the two queues by bisection over the merged order's diagonal, a load from
    // each queue a step, and takes the two lightest of the four nodes there: the merged order is never written down.
    // The whole builder, us, with every node's rank looked up by one of two searches and the order kept in LDS, and so:
    // [1,4,3] 32.2 and 28.0, [1,5,2] 28.7 and 25.4, 16 symbols 12.2 and 10.7.  (The odd one known from its lane instead of
    // two weights read back: 28.5, 26.0, 11.2.)
    if (t < 64) {
        const uint64_t kNone = ~0ull;
        int li = 0, ii = n, made = n;   // next leaf, next internal node, next node to create
        bool over = err != 0;   // the weights of this table sum to 2^64 - 1 or more
        while (n >= 2 && !over && (n - li) + (made - ii) > 1) {   // the same in every lane
            // the leaf li + t and the internal node ii + t; the lightest two of each queue are lanes 0 and 1
            uint64_t leaf = li + t < n ? nw[li + t] : kNone;
            const uint64_t inner = ii + t < made ? nw[ii + t] : kNone;
            const uint64_t c0 = lane_value(leaf, 0), c1 = lane_value(leaf, 1);
            const uint64_t c2 = lane_value(inner, 0), c3 = lane_value(inner, 1);
            // the two lightest of two sorted pairs
            const uint64_t m1 = c0 < c2 ? c0 : c2;
            const uint64_t r1 = c0 < c2 ? c1 : c0, r2 = c0 < c2 ? c2 : c3;
            const uint64_t m2 = r1 < r2 ? r1 : r2;
            const uint64_t T = m1 + m2;
            if (T < m2 || T == kNone) {
                over = true;
                break;
            }
            // leaves of weight <= T: they are sorted, so counting them (lane t looks at leaf lj + t) gives the end; no
            // leaf is as heavy as what stands for none, and T is below it
            int lj = li, c;
            for (;;) {
                c = __popcll(__ballot(leaf <= T));
                lj += c;
                if (c < 64) break;
                leaf = lj + t < n ? nw[lj + t] : kNone;
            }
            const int bL = lj - li;
            const int bI = made - ii, nb = bL + bI;   // 2 <= nb <= 256: the two lightest are among them
            const int npair = nb >> 1;
            bool wrapped = false;
            for (int k = t; k < npair; k += 64) {
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
                wrapped |= sum < wb || sum == kNone;
                nw[made + k] = sum;
                parent[leaf1 ? li + i : ii + j] = made + k;
                parent[leaf2 ? li + i + leaf1 : ii + j + !leaf1] = made + k;
            }
            over = __any(wrapped);
            pc_wave_sync_lds();
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

    if (t < n && !err) {
        int depth = 0;
        if (n == 1) depth = 1;
        for (int p = parent[t]; p >= 0 && depth <= CO3_MAX_CODE_LEN; p = parent[p]) ++depth;
        if (depth > CO3_MAX_CODE_LEN) err = 1;
        else slen[leaf_sym[t]] = (uint32_t)depth;
    }
    __syncthreads();
    const bool bad = err != 0;
    if (bad) {
        slen[t] = 0;
        if (t == 0) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CODELEN), 1ull);
    }
    __syncthreads();

    // rank of the symbol among those of its length: the lanes of its wavefront with the same length by one ballot per
    // bit of it, the wavefronts before by their counts
    const uint32_t L = slen[t];
    const int wave = t >> 6, lane = t & 63;
    uint64_t same = ~0ull;
#pragma unroll
    for (int b = 0; b < 7; ++b) {
        const uint64_t ones = __ballot((L >> b) & 1u);
        same &= ((L >> b) & 1u) ? ones : ~ones;
    }
    const uint64_t before = same & ((1ull << lane) - 1ull);
    uint32_t rank = (uint32_t)__popcll(before);
    if (L && !before) wcnt[wave][L] = (uint32_t)__popcll(same);
    __syncthreads();
    for (int k = 0; k < wave; ++k) rank += wcnt[k][L];
    if (t < 64) {
        // lane l - 1 takes length l; first[l] = 2 (first[l - 1] + cnt[l - 1]) as a scan whose step over k lengths
        // shifts by k
        uint32_t cl = 0, cp = 0;   // codes of length l, of length l - 1
#pragma unroll
        for (int k = 0; k < kCbThreads / 64; ++k) {
            cl += wcnt[k][t + 1];
            cp += t ? wcnt[k][t] : 0u;
        }
        uint64_t sum = cp;
        uint32_t o = cp;
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const uint64_t s_up = __shfl_up(sum, k, 64);
            const uint32_t o_up = __shfl_up(o, k, 64);
            if (t >= k) {
                sum += s_up << k;
                o += o_up;
            }
        }
        const int l = t + 1;
        const uint64_t code = sum << 1;
        cnt[l] = cl;
        first[l] = code;
        off[l] = o;
        const uint64_t used = __ballot(cl != 0);
        base[l] = o - (uint32_t)code;
        const uint64_t end = l < 32 ? (code + cl) << (32 - l) : 0;   // codes of up to l bits lie below, left-aligned in 32 bits
        if (l < 32) limit[l] = end >> 32 ? 0u : ~(uint32_t)end;
        if (t == 0) {
            B.maxlen = used ? 64u - (uint32_t)__clzll((long long)used) : 0u;
            B.nactive = bad ? 0 : (uint32_t)n;
            B.format = dec_format(E, M);
        }
    }
    __syncthreads();

    uint64_t code = 0;
    uint32_t fast = kFastSlow << 24;  // a longer code, or none: the coders' general path
    if (L) {
        code = first[L] + rank;
        sorted[off[L] + rank] = (uint32_t)t;
        entry_sym[off[L] + rank] = ((uint32_t)t << 8) | L;
        if (L <= (uint32_t)kFastLen) fast = (L << 24) | (uint32_t)code;
    }
    B.code[t] = code;
    B.fast[t] = fast;
    B.len[t] = (uint8_t)L;
    if (t < 65) { B.first[t] = first[t]; B.count[t] = cnt[t]; B.offset[t] = off[t]; }
    __syncthreads();
    B.sorted[t] = (t < n && !bad) ? (uint8_t)sorted[t] : 0;

    // decode tables (decode_core.h), two entries at a time: the window's complement at the entry's low end, its code's
    // length by a binary search of the limits (they fall with the length; the first steps' from registers), the rest from
    // the code's rank
    const uint32_t nm = (uint32_t)(E + M);
    const bool values = dec_value_is_int(E);   // only integer sums read them
    const uint32_t l8[4] = {0u, limit[8], limit[16], limit[24]}, l4[4] = {limit[4], limit[12], limit[20], limit[28]};
#pragma unroll 8
    for (uint32_t i2 = t; i2 < dec_table_entries(A) / 2; i2 += kCbThreads) {
        uint32_t es[2];
#pragma unroll
        for (uint32_t b = 0; b < 2; ++b) {
            const uint32_t i = 2 * i2 + b, binade = i >> nm;
            const uint32_t ex = binade == 31u ? 0u : binade + 1u;            // exponent of u
            const uint32_t lead = (1u << nm) | (i & ((1u << nm) - 1u));
            const uint32_t u = ex >= nm ? (uint32_t)((uint64_t)lead << (ex - nm)) : lead >> (nm - ex);
            // the largest l with u <= limit[l]: the code has l + 1 bits
            const uint32_t q = u <= l8[2] ? (u <= l8[3] ? 3u : 2u) : (u <= l8[1] ? 1u : 0u);
            const uint32_t at4 = q > 1u ? (q > 2u ? l4[3] : l4[2]) : (q ? l4[1] : l4[0]);
            uint32_t l = 8u * q + (u <= at4 ? 4u : 0u);
            l += u <= limit[l + 2u] ? 2u : 0u;
            l += u <= limit[l + 1u] ? 1u : 0u;
            es[b] = kLenSlow;
            const uint32_t L = l + 1;
            if (binade != 0 && L < 32u) {   // (below the end of every code of up to 31 bits)
                es[b] = entry_sym[(base[L] + (~u >> (32 - L))) & (kMaxA - 1)];
            }
        }
        reinterpret_cast<uint32_t *>(B.dsym)[i2] = es[0] | (es[1] << 16);
        if (values)
            reinterpret_cast<uint2 *>(B.dval)[i2] = make_uint2(dec_value_bits(es[0] >> 8, E, M) | (es[0] & 0xffu),
                                                              dec_value_bits(es[1] >> 8, E, M) | (es[1] & 0xffu));
    }
}

hipError_t launch_build_books(BookDev *books, uint32_t nbooks, int E, int M, const uint64_t *weights, uint64_t *counts,
                              uint64_t *status, hipStream_t s)
{
    if (nbooks == 0) return hipSuccess;
    ProfScope prof(K_BUILD_BOOKS, s);
    hipLaunchKernelGGL(k_build_books, dim3(nbooks), dim3(kCbThreads), 0, s, books, E, M, weights, counts, status);
    return hipGetLastError();
}

}  // namespace co3
