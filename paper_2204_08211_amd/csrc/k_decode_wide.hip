// PS side for alphabets of 9 to 12 bits (Sec. II-B (iv); Algorithm 1 lines 13-14): the decoder of decode_core.h with a
// table of up to 42 KB, so that the wavefronts of a workgroup share one as far as they can.  Bound by the chain from one
// pair of symbols to the next (two dependent look-ups, an add, the window's read) with the 16 wavefronts that fit a CU.
// Sixteen users of 25.6 M elements in [1,5,6], against a canonical search per symbol: decoded 1063 -> 369 us, averaged
// 907 -> 481 (the copy rate would take 135 and 120), averaged with a table per user 2310 -> 1022.
#include "decode_core.h"

namespace co3 {

typedef AggArgsT<BookWide> WideAggArgs;
constexpr int kWdWaves = 16;                       // wavefronts of a full workgroup: one fits a CU
constexpr uint32_t kWdWindow = kRowsWide * 64;     // words of a wavefront's window
// LDS words: notes (the code tables of the chunks, the lengths' limits), which are also what the reads of a damaged stream
// below the first window meet; windows; the row behind them and tables.
constexpr uint32_t kWdLimits = 64, kWdFront = kFrontWords;
__host__ __device__ constexpr uint32_t wide_table_words(uint32_t A) { return kWideTabBinades << wide_tab_bits_max(A); }

struct WideEntry {
    __device__ inline uint32_t operator()(uint32_t s) const { return s << 8; }
};

// A code's table and limits to LDS; `bits` of it.
__device__ inline uint32_t load_wide_table(uint32_t *table, uint32_t *limits, const BookWide *__restrict__ book, uint32_t t, uint32_t nthreads)
{
    const uint32_t bits = uniform(book->tab_bits);
    for (uint32_t i = t; i < 32u; i += nthreads) limits[i] = book->limit[i];
    load_table(table, book->tab, 4u * wide_tab_entries(bits), t, nthreads);
    return bits;
}

// A started chunk's symbols to `packed`, by the table in LDS.
template <class Packed>
__device__ inline void decode_wide(Stream &st, const ChunkGeom &g, const ChunkIndex &ix, uint32_t A, const uint32_t *table,
                                   uint32_t bits, const uint32_t *limits, const BookWide *__restrict__ book, Packed &packed)
{
    WideDecTable tab;
    tab.init(lds_address(table), bits, lds_address(limits));
    decode_started<false>(st, g, ix, A, tab, book, WideEntry{},
                                 [&](int gr, const uint32_t (&e)[kGroup]) { packed.group(gr, e); });
}

// A sub-chunk's symbols, two to a word: the first 32, the last 32.
struct WidePacked {
    u32x16 h[2];
    __device__ inline void clear() { h[0] = 0u; h[1] = 0u; }
    __device__ inline void group(int gr, const uint32_t (&e)[kGroup])
    {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x06050201u);   // bytes 1 and 2 of two entries
        const int at = 4 * (gr & 3);
        if (gr < 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) h[0][at + i] = w[i];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) h[1][at + i] = w[i];
        }
    }
};

// co3_decode: as k_decode, a wavefront per chunk of one user; a workgroup takes `sets` sets of chunks one after the other
// and loads the table where it changes, so that its wavefronts are not held together.  by_chunk: the users' chunks 0, then
// their chunks 1, ...
constexpr int kWdStageStride = 20;   // words per staged half sub-chunk (16, and 4 that keep 16-byte accesses apart)
static_assert(kSubsPerChunk * kWdStageStride <= (int)kWdWindow, "half a chunk's symbols are staged in the window");
__global__ __launch_bounds__(64 * kWdWaves, 4) void k_decode_wide(Layout lay, const uint32_t *__restrict__ words, uint64_t words_stride,
                                                                const uint64_t *__restrict__ chunk_offset,
                                                                const uint16_t *__restrict__ sub_bits,
                                                                const BookWide *__restrict__ books, uint16_t *__restrict__ sym,
                                                                uint64_t sym_stride, float *__restrict__ q, uint64_t q_stride,
                                                                uint64_t *__restrict__ status, uint32_t sets, uint32_t by_chunk)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const uint32_t t = threadIdx.x, lane = t & 63, waves = blockDim.x >> 6;
    const uint32_t wave = uniform(t >> 6);
    uint32_t *win = smem + kWdFront + wave * kWdWindow, *s_tab = smem + kWdFront + waves * kWdWindow + kBehindWords;
    int32_t *s_book = reinterpret_cast<int32_t *>(smem);
    const SymbolValue val(lay.E, lay.M);
    const uint64_t per_user = (lay.nchunks + waves - 1) / waves;   // sets
    const uint64_t items = lay.nchunks * lay.U, all = by_chunk ? (items + waves - 1) / waves : per_user * lay.U;
    const bool several = lay.books_per_user > 1;
    uint64_t loaded_table = ~0ull;
    uint32_t bits = 0;
#pragma unroll 1
    for (uint32_t i = 0; i < sets; ++i) {
        const uint64_t set = (uint64_t)blockIdx.x * sets + i;
        if (set >= all) break;
        uint32_t u;
        uint64_t c;
        bool active;
        if (by_chunk) {
            uint64_t item = set * waves + wave;
            active = item < items;
            if (!active) item = items - 1;
            c = item / lay.U;
            u = (uint32_t)(item - c * lay.U);
        } else {
            u = (uint32_t)(set / per_user);
            c = (set - u * per_user) * waves + wave;
            active = c < lay.nchunks;
            if (!active) c = lay.nchunks - 1;
        }
        const ChunkGeom g = chunk_geom(lay, c);
        const ChunkIndex ix = read_index(lay, c, u, words, words_stride, chunk_offset, sub_bits);
        WidePacked packed;
        packed.clear();
        if (several) {
            __syncthreads();
            if (lane == 0) s_book[wave] = g.book;
            __syncthreads();
        }
        uint32_t w0 = 0;
        do {   // where the code table changes among the chunks (layers), one stretch after the other
            int32_t b = 0;
            uint32_t w1 = waves;
            if (several) {
                b = __builtin_amdgcn_readfirstlane(s_book[w0]);
                for (w1 = w0 + 1; w1 < waves && __builtin_amdgcn_readfirstlane(s_book[w1]) == b;) ++w1;
            }
            const uint64_t id = (lay.per_user_books ? (uint64_t)u * lay.books_per_user : 0u) + (uint32_t)b;
            if (id != loaded_table) {   // the same in all wavefronts
                __syncthreads();        // the one before is done with
                bits = load_wide_table(s_tab, smem + kWdLimits, books + id, t, 64 * waves);
                __syncthreads();
                loaded_table = id;
            }
            if (active && wave >= w0 && wave < w1) {
                Stream st;
                round_toward_zero();
                start_chunk<kRowsWide>(st, g, ix, lds_address(win), kRowsWide);
                decode_wide(st, g, ix, lay.A, s_tab, bits, smem + kWdLimits, books + id, packed);
                finish_chunk(st, ix, status);
                round_to_nearest();
            }
            w0 = w1;
        } while (w0 < waves);
        if (!active) continue;   // (the wavefront still meets the others at the next table)
        const uint64_t pair = (uint64_t)u * lay.nseg + g.seg;
        const int up = 127 - (int)uniform((uint32_t)lay.bias[pair]);
        const float inv_gain = lay.gain[2 * pair + 1];   // 1 unless the plan carries a scale
        uint16_t *dst = sym + (uint64_t)u * sym_stride + g.e0;
        float *dq = q + (uint64_t)u * q_stride + g.e0;
        const bool full = g.n == (uint32_t)kChunk;
        const uint32_t l = here(lane);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            // 32 symbols of every sub-chunk to rows of 16 words, and out eight symbols a lane
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<u32x4 *>(win + l * kWdStageStride + 4 * j) =
                    u32x4{packed.h[half][4 * j], packed.h[half][4 * j + 1], packed.h[half][4 * j + 2], packed.h[half][4 * j + 3]};
            wave_lds_fence();
#pragma unroll 1
            for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t sub = 16u * k + (l >> 2), piece = l & 3u;
                const u32x4 w = *reinterpret_cast<const u32x4 *>(win + sub * kWdStageStride + 4u * piece);
                const uint32_t e = 64u * sub + 32u * (uint32_t)half + 8u * piece;
                if (sym) {
                    if (full) {   // layers start anywhere
                        *reinterpret_cast<u32x4_u16 *>(dst + e) = w;
                    } else {
#pragma unroll
                        for (uint32_t b = 0; b < 8; ++b)
                            if (e + b < g.n) dst[e + b] = (uint16_t)(w[b >> 1] >> (16u * (b & 1u)));
                    }
                }
                if (q) {
                    f32x4 v[2];
#pragma unroll
                    for (uint32_t b = 0; b < 8; ++b) v[b >> 2][b & 3u] = __fmul_rn(ldexpf(val(w[b >> 1], 16u * (b & 1u)), up), inv_gain);
                    if (full) {
                        *reinterpret_cast<f32x4_any *>(dq + e) = v[0];
                        *reinterpret_cast<f32x4_any *>(dq + e + 4) = v[1];
                    } else {
#pragma unroll
                        for (uint32_t b = 0; b < 8; ++b)
                            if (e + b < g.n) dq[e + b] = v[b >> 2][b & 3u];
                    }
                }
            }
            wave_lds_fence();
        }
    }
}

// fl32(value * inv_gain) of a symbol as fp64 (inv_gain is 1 unless the plan carries a scale).
__device__ inline double wide_value(const SymbolValue &val, uint32_t word, uint32_t bit, int up, float inv_gain)
{
    return (double)__fmul_rn(ldexpf(val(word, bit), up), inv_gain);
}

constexpr int kWaStride = 65;       // sums of a workgroup's 16 rows: element i of sub-chunk s at i * stride + s
constexpr int kWaAloneStride = 68;  // of a wavefront's 8 rows
static_assert(8 * kWaAloneStride * 2 <= (int)kWdWindow && 16 * kWaStride * 2 <= 2 * (int)kWdWindow, "the sums go through the windows");

// co3_ps_aggregate: `split` wavefronts share a chunk and its users (a power of two; the workgroup's wavefronts / split
// chunks in one workgroup, under one table or one stretch after the other), each decodes up to kUsers of them at a time to
// packed symbols and adds their values in fp64.  With a table per user every wavefront has a table (split wavefronts, one
// chunk).  all_at: where the sums are kept when the users come in several turns, else 0.  A workgroup takes `sets` sets of
// chunks one after the other.
// kFew: three or four users over two wavefronts.  Up to four users keep their order: the first wavefront takes the first two, and
// the second adds its own to their sum one by one.
template <int kUsers, bool kFew>
__global__ __launch_bounds__(64 * kWdWaves, 4) void k_aggregate_wide(Layout lay, WideAggArgs a, uint32_t split_log2, uint32_t all_at, uint32_t sets)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const uint32_t t = threadIdx.x, lane = t & 63, waves = blockDim.x >> 6;
    const uint32_t wave = uniform(t >> 6);
    const uint32_t split = 1u << split_log2, slot = wave >> split_log2, part = wave & (split - 1u), slots = waves >> split_log2;
    const bool own = lay.per_user_books != 0;
    const uint32_t tab_words = wide_table_words(lay.A);
    uint32_t *win = smem + kWdFront + wave * kWdWindow;
    uint32_t *s_tab = smem + kWdFront + waves * kWdWindow + kBehindWords + (own ? wave * tab_words : 0u);
    uint32_t *s_limits = smem + kWdLimits + (own ? 32u * wave : 0u);
    int32_t *s_book = reinterpret_cast<int32_t *>(smem);
    double *s_all = all_at ? reinterpret_cast<double *>(smem + all_at) : nullptr;
    const SymbolValue val(lay.E, lay.M);
    const double inv_u = 1.0 / (double)lay.U;
    const bool several = lay.books_per_user > 1;
    int32_t loaded_table = -1;
    uint32_t bits = 0;
    WidePacked pk[kUsers];
    auto user = [&](uint32_t u0, int s) { return u0 + (kFew ? part * kUsers + (uint32_t)s : part + (uint32_t)s * split); };
#pragma unroll 1
    for (uint32_t set = 0; set < sets; ++set) {
        if (((uint64_t)blockIdx.x * sets + set) * slots >= lay.nchunks) break;
        uint64_t c = ((uint64_t)blockIdx.x * sets + set) * slots + slot;
        const bool active = c < lay.nchunks;
        if (!active) c = lay.nchunks - 1;
        const ChunkGeom g = uniform(chunk_geom(lay, c));
        if (several) {
            __syncthreads();
            if (lane == 0) s_book[wave] = g.book;
            __syncthreads();
        }
        for (uint32_t u0 = 0; u0 < lay.U; u0 += split * kUsers) {
#pragma unroll
            for (int s = 0; s < kUsers; ++s) pk[s].clear();
            round_toward_zero();
            uint32_t w0 = 0;
            do {
                int32_t b = 0;
                uint32_t w1 = waves;
                if (several) {
                    b = __builtin_amdgcn_readfirstlane(s_book[w0]);
                    for (w1 = w0 + 1; w1 < waves && __builtin_amdgcn_readfirstlane(s_book[w1]) == b;) ++w1;
                }
                if (!own && b != loaded_table) {   // the same in all wavefronts
                    __syncthreads();               // the one before is done with
                    bits = load_wide_table(s_tab, s_limits, a.books + b, t, 64 * waves);
                    __syncthreads();
                    loaded_table = b;
                }
                if (active && wave >= w0 && wave < w1) {
#pragma unroll
                    for (int s = 0; s < kUsers; ++s) {
                        const uint32_t u = user(u0, s);
                        if (u >= lay.U) continue;
                        const ChunkIndex ix = read_index(lay, c, u, a.words, a.words_stride, a.chunk_offset, a.sub_bits);
                        const BookWide *book = a.books + (own ? (uint64_t)u * lay.books_per_user : 0u) + b;
                        if (own) {
                            bits = load_wide_table(s_tab, s_limits, book, lane, 64);
                            wave_lds_fence();
                        }
                        Stream st;
                        start_chunk<kRowsWide>(st, g, ix, lds_address(win), kRowsWide);
                        decode_wide(st, g, ix, lay.A, s_tab, bits, s_limits, book, pk[s]);
                        finish_chunk(st, ix, a.status);
                    }
                }
                w0 = w1;
            } while (w0 < waves);
            round_to_nearest();
#pragma unroll
            for (int s = 0; s < kUsers; ++s) {   // (the values round: not before the mode is back)
                words_here(pk[s].h[0]);
                words_here(pk[s].h[1]);
            }

            int up[kUsers];
            float inv_gain[kUsers];
#pragma unroll
            for (int s = 0; s < kUsers; ++s) {
                const uint32_t u = user(u0, s);
                const uint64_t pair = (uint64_t)(u < lay.U ? u : 0u) * lay.nseg + g.seg;
                up[s] = 127 - (int)uniform((uint32_t)lay.bias[pair]);
                inv_gain[s] = lay.gain[2 * pair + 1];
            }
            auto sum_of = [&](int j, double sum = 0.0) {   // in the users' order
#pragma unroll
                for (int s = 0; s < kUsers; ++s) sum += wide_value(val, pk[s].h[j >> 5][(j & 31) >> 1], 16u * (uint32_t)(j & 1), up[s], inv_gain[s]);
                return sum;
            };
            const bool first = u0 == 0, last = u0 + split * kUsers >= lay.U, whole = g.n == (uint32_t)kChunk;
            if (split > 1) {
                const uint32_t tt = (part << 6) | lane;
                // up to four users keep their order, more are added as they come (exact for any reasonable spread of biases)
                const uint32_t turns = lay.U <= 4u ? split : 2u;
#pragma unroll
                for (int j = 0; j < kSub; j += 16) {
                    double *s_sum = s_all ? s_all + j * kWaStride : reinterpret_cast<double *>(smem + kWdFront + slot * split * kWdWindow);
                    __syncthreads();
                    if constexpr (kFew) {
                        if (part == 0u) {
#pragma unroll
                            for (int i = 0; i < 16; ++i) s_sum[i * kWaStride + lane] = sum_of(j + i);
                        }
                        __syncthreads();
                        if (part == 1u) {
#pragma unroll
                            for (int i = 0; i < 16; ++i) s_sum[i * kWaStride + lane] = sum_of(j + i, s_sum[i * kWaStride + lane]);
                        }
                        __syncthreads();
                    } else {
                        double v[16];
#pragma unroll
                        for (int i = 0; i < 16; ++i) v[i] = here(sum_of(j + i));
#pragma unroll 1
                        for (uint32_t w = 0; w < turns; ++w) {
                            if (turns == 2u && w ? part > 0u : part == w) {
#pragma unroll
                                for (int i = 0; i < 16; ++i) {
                                    double *at = &s_sum[i * kWaStride + lane];
                                    if (w == 0 && first) *at = v[i];
                                    else __hip_atomic_fetch_add(at, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                                }
                            }
                            __syncthreads();
                        }
                    }
#pragma unroll 1
                    for (uint32_t k = tt; last && active && k < 256u; k += 64u << split_log2) {
                        const uint32_t s = k >> 2, i = 4u * (k & 3u);
                        double avg[4];
#pragma unroll
                        for (int b = 0; b < 4; ++b) avg[b] = s_sum[(i + b) * kWaStride + s] * inv_u;
                        write_four(g, a, s * kSub + (uint32_t)j + i, avg, whole);
                    }
                }
                __syncthreads();   // the sums are read
            } else if (active) {
                double *s_sum = reinterpret_cast<double *>(win);
#pragma unroll
                for (int j = 0; j < kSub; j += 8) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) s_sum[i * kWaAloneStride + lane] = sum_of(j + i);
                    wave_lds_fence();
                    const uint32_t l = here(lane);
#pragma unroll 1
                    for (uint32_t k = l; k < 128u; k += 64u) {
                        const uint32_t s = k >> 1, i = 4u * (k & 1u);
                        double avg[4];
#pragma unroll
                        for (int b = 0; b < 4; ++b) avg[b] = s_sum[(i + b) * kWaAloneStride + s] * inv_u;
                        write_four(g, a, s * kSub + (uint32_t)j + i, avg, whole);
                    }
                    wave_lds_fence();
                }
            }
        }
    }
}

// co3_ps_aggregate with a table per user and many chunks: the wavefronts of a workgroup take a chunk each and share the
// table of one user after the other; fp64 sums of half of every sub-chunk at a time, so the users are decoded twice.
__global__ __launch_bounds__(64 * kWdWaves, 4) void k_aggregate_wide_own(Layout lay, WideAggArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const uint32_t t = threadIdx.x, lane = t & 63, waves = blockDim.x >> 6;
    const uint32_t wave = uniform(t >> 6);
    uint32_t *win = smem + kWdFront + wave * kWdWindow, *s_tab = smem + kWdFront + waves * kWdWindow + kBehindWords;
    int32_t *s_book = reinterpret_cast<int32_t *>(smem);
    uint64_t c = (uint64_t)blockIdx.x * waves + wave;
    const bool active = c < lay.nchunks;
    if (!active) c = lay.nchunks - 1;
    const ChunkGeom g = chunk_geom(lay, c);
    const SymbolValue val(lay.E, lay.M);
    const double inv_u = 1.0 / (double)lay.U;
    if (lane == 0) s_book[wave] = g.book;
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        double sum[kSub / 2];
#pragma unroll
        for (int i = 0; i < kSub / 2; ++i) sum[i] = 0.0;
#pragma unroll 1
        for (uint32_t u = 0; u < lay.U; ++u) {
            const ChunkIndex ix = read_index(lay, c, u, a.words, a.words_stride, a.chunk_offset, a.sub_bits);
            const BookWide *set = a.books + (uint64_t)u * lay.books_per_user;
            uint32_t w0 = 0;
            do {
                __syncthreads();   // the table before is done with (and s_book written)
                const int32_t b = __builtin_amdgcn_readfirstlane(s_book[w0]);
                uint32_t w1 = w0 + 1;
                while (w1 < waves && __builtin_amdgcn_readfirstlane(s_book[w1]) == b) ++w1;
                const uint32_t bits = load_wide_table(s_tab, smem + kWdLimits, set + b, t, 64 * waves);
                __syncthreads();
                if (active && wave >= w0 && wave < w1) {
                    WidePacked pk;
                    pk.clear();
                    Stream st;
                    round_toward_zero();
                    start_chunk<kRowsWide>(st, g, ix, lds_address(win), kRowsWide);
                    decode_wide(st, g, ix, lay.A, s_tab, bits, smem + kWdLimits, set + b, pk);
                    if (half == 0) finish_chunk(st, ix, a.status);
                    else wave_lds_fence();
                    round_to_nearest();
                    const uint64_t pair = (uint64_t)u * lay.nseg + g.seg;
                    const int up = 127 - (int)uniform((uint32_t)lay.bias[pair]);
                    const float inv_gain = lay.gain[2 * pair + 1];
#pragma unroll
                    for (int i = 0; i < kSub / 2; ++i) {
                        const uint32_t w = half ? pk.h[1][i >> 1] : pk.h[0][i >> 1];
                        sum[i] = here(sum[i] + wide_value(val, here(w), 16u * (uint32_t)(i & 1), up, inv_gain));
                    }
                }
                w0 = w1;
            } while (w0 < waves);
        }
        if (active) {
            double *s_sum = reinterpret_cast<double *>(win);
            const bool whole = g.n == (uint32_t)kChunk;
#pragma unroll
            for (int j = 0; j < kSub / 2; j += 8) {
#pragma unroll
                for (int i = 0; i < 8; ++i) s_sum[i * kWaAloneStride + lane] = sum[j + i];
                wave_lds_fence();
                const uint32_t l = here(lane);
#pragma unroll 1
                for (uint32_t k = l; k < 128u; k += 64u) {
                    const uint32_t s = k >> 1, i = 4u * (k & 1u);
                    double avg[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) avg[b] = s_sum[(i + b) * kWaAloneStride + s] * inv_u;
                    write_four(g, a, s * kSub + (uint32_t)(half * (kSub / 2) + j) + i, avg, whole);
                }
                wave_lds_fence();
            }
        }
    }
}

// Chunks from which wavefronts that share the users' tables one after the other and decode twice beat two wavefronts a chunk
// with a table each, of which a CU holds two (ten users in [1,4,5], 977 chunks 258 against 215 us, 3907 chunks 275 against
// 841; two users 61 against 65 and 77 against 246).
constexpr uint64_t kWaOwnChunks = 1200;

static size_t wide_lds(const Layout &lay, uint32_t waves, uint32_t tables)
{
    return 4 * ((size_t)kWdFront + waves * kWdWindow + kBehindWords + tables * wide_table_words(lay.A));
}

// Sets of chunks that a workgroup takes one after the other, for `groups` workgroups: a CU holds one (its table and windows
// take the LDS), so a new one stands still until its table is there, and at the barriers of the last.  Sixteen users of
// 25.6 M elements in [1,5,6], one set each, 1024, 512 and 256 workgroups: decoded 447, 379, 369 and 430 us, averaged (whose
// wavefronts meet with every set anyway) 507, 576, 514 and 481 us.
static uint32_t wide_sets(uint64_t all, uint32_t groups) { return (uint32_t)((all + groups - 1) / groups); }

hipError_t launch_decode_wide(const Layout &lay, const co3_decode_args &a, const BookWide *books, hipStream_t s)
{
    if (lay.U == 0 || lay.nchunks == 0) return hipSuccess;
    uint32_t waves = lay.nchunks < (uint32_t)kWdWaves ? (uint32_t)lay.nchunks : kWdWaves;
    // Layers under tables of their own: by chunk a workgroup meets few of them, and small launches of smaller workgroups have
    // more of them side by side (users of 353 444 elements in twelve layers: 24 in [1,5,6] by user 64, by chunk 37 us; four
    // in [1,4,5] 59 and 17).
    const bool several = lay.books_per_user > 1, by_chunk = several && !lay.per_user_books;
    while (several && waves > 4 && lay.nchunks * lay.U < 256ull * waves) waves = (waves + 1) / 2;
    const size_t lds = wide_lds(lay, waves, 1);
    const uint64_t all = by_chunk ? (lay.nchunks * lay.U + waves - 1) / waves : (lay.nchunks + waves - 1) / waves * lay.U;
    const uint32_t sets = wide_sets(all, 512);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_decode_wide), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(K_DECODE, s);
    hipLaunchKernelGGL(k_decode_wide, dim3((uint32_t)((all + sets - 1) / sets)), dim3(64 * waves), lds, s, lay,
                       a.words, a.words_stride, a.chunk_offset, a.sub_bits, books, reinterpret_cast<uint16_t *>(a.symbols),
                       symbol_row_stride(lay.d), a.q, a.q_stride, a.status, sets, by_chunk ? 1u : 0u);
    return hipGetLastError();
}

template <class Kernel, class... Args>
static hipError_t launch_wide(Kernel k, uint64_t grid, uint32_t waves, size_t lds, hipStream_t s, Args... args)
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(K_AGGREGATE, s);
    hipLaunchKernelGGL(k, dim3((uint32_t)grid), dim3(64 * waves), lds, s, args...);
    return hipGetLastError();
}

hipError_t launch_aggregate_wide(const Layout &lay, const co3_aggregate_args &a, const BookWide *books, hipStream_t s)
{
    if (lay.U == 0 || lay.nchunks == 0) return hipSuccess;
    const WideAggArgs args = {a.words, a.words_stride, a.chunk_offset, a.sub_bits, books, a.out, a.model, (double)a.eta, a.status};
    const size_t sums = (size_t)kSub * kWaStride * sizeof(double);
    if (lay.per_user_books) {
        if (lay.nchunks >= kWaOwnChunks) {
            const uint32_t waves = kWdWaves;
            return launch_wide(k_aggregate_wide_own, (lay.nchunks + waves - 1) / waves, waves, wide_lds(lay, waves, 1), s, lay, args);
        }
        // few chunks: two wavefronts a chunk with a table each
        const uint32_t log2 = lay.U > 1 ? 1 : 0, waves = 1u << log2;
        size_t lds = wide_lds(lay, waves, waves);
        uint32_t all_at = 0;
        if (lay.U > 2 * waves) {
            all_at = (uint32_t)((lds + 15) / 16 * 4);
            lds = 4 * (size_t)all_at + sums;
        }
        return lay.U == 3u || lay.U == 4u
                   ? launch_wide(k_aggregate_wide<2, true>, lay.nchunks, waves, lds, s, lay, args, log2, all_at, 1u)
                   : launch_wide(k_aggregate_wide<2, false>, lay.nchunks, waves, lds, s, lay, args, log2, all_at, 1u);
    }
    // Wavefronts per chunk: two users each, or one where the chip has room (eight users of 1 M elements, 245 chunks, in
    // [1,4,5]: eight wavefronts 19 us, four 25; of 2 M 33 and 28; sixteen users of 1 M, sixteen wavefronts 24, eight 27;
    // two users of 4 M, two wavefronts 20, one 24; of 8 M 35 and 32).
    uint32_t log2 = 0;
    while ((1u << log2) < (uint32_t)kWdWaves && (2u << log2) < lay.U) ++log2;
    while ((1u << log2) < (uint32_t)kWdWaves && (1u << log2) < lay.U &&
           (lay.nchunks <= 256 || (lay.nchunks << (log2 + 1)) <= 2048)) ++log2;
    const uint32_t split = 1u << log2;
    const bool one = lay.U <= split;
    if (lay.U > 2 * split) {   // more users than a turn takes: the sums need a place of their own
        const uint32_t waves = 8;
        const size_t all_at = (wide_lds(lay, waves, 1) + 15) / 16 * 4;
        return launch_wide(k_aggregate_wide<2, false>, lay.nchunks, waves, 4 * all_at + sums, s, lay, args, 3u, (uint32_t)all_at, 1u);
    }
    // a full workgroup where there are enough of them, else one chunk each
    uint32_t waves = lay.nchunks * split >= 16 * 256 ? (uint32_t)kWdWaves : (split > 4 ? split : 4u);
    const uint64_t slots = waves >> log2, all = (lay.nchunks + slots - 1) / slots;
    const uint32_t sets = waves == (uint32_t)kWdWaves ? wide_sets(all, 256) : 1u;
    const uint64_t grid = (all + sets - 1) / sets;
    const size_t lds = wide_lds(lay, waves, 1);
    if (one) return launch_wide(k_aggregate_wide<1, false>, grid, waves, lds, s, lay, args, log2, 0u, sets);
    // (two wavefronts a chunk; in the users' order four users of 25 M elements take 113 us, in any order 112)
    return lay.U == 3u || lay.U == 4u ? launch_wide(k_aggregate_wide<2, true>, grid, waves, lds, s, lay, args, log2, 0u, sets)
                                      : launch_wide(k_aggregate_wide<2, false>, grid, waves, lds, s, lay, args, log2, 0u, sets);
}

}  // namespace co3
