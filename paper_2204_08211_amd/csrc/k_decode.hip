// PS side (Sec. II-B (iv); Algorithm 1 lines 13-14): invert h_Hf for every user's stream and
// form (1/U) sum_u ghat^(u), eq. (aggregate hat) without the learning rate.
//
// A wavefront decodes one chunk of one user at a time (decode_core.h): lane j takes sub-chunk j, whose start is the prefix
// sum of the sub-chunk bit counts.  co3_decode packs the symbols in registers; the average keeps the sums of a lane's 64
// elements over the users in registers.  Both go through LDS once at the end so that the stores are coalesced.
#include <cstddef>

#include "decode_core.h"

namespace co3 {

typedef AggArgsT<BookDev> AggArgs;

// Symbols 8 gr .. 8 gr + 7 of a sub-chunk (or of the part that `packed` has room for): byte 1 of their entries.
template <class Packed>
__device__ inline void pack_group(Packed &packed, int gr, const uint32_t (&e)[kGroup])
{
#pragma unroll
    for (int h = 0; h < 2; ++h)
        packed[2 * gr + h] = __builtin_amdgcn_perm(e[4 * h + 1], e[4 * h], 0x0c0c0501u) |
                             __builtin_amdgcn_perm(e[4 * h + 3], e[4 * h + 2], 0x05010c0cu);
}

// co3_decode: a workgroup takes kDecWaves consecutive chunks of one user, a wavefront per chunk, so that one copy of the
// table serves them; where the code table changes among them (layers) the workgroup takes one stretch after the other.
// by_chunk: the users' chunks 0, then their chunks 1, ...
constexpr int kDecWaves = 8;
constexpr int kStageStride = 20;   // words per staged sub-chunk row (16, and 4 that keep 16-byte accesses apart)
// Words of a wavefront's window where something is staged in it afterwards: a chunk's symbols, pieces of its sums.
constexpr uint32_t kStageWords = kSubsPerChunk * kStageStride;
static_assert(kStageWords % 64 == 0, "windows are whole rows");
__host__ __device__ constexpr uint32_t stage_window_words(uint32_t A) { return window_words(A) > kStageWords ? window_words(A) : kStageWords; }
// kOne: the average of a single user, which is its values: out and model of `one` instead of symbols and q (one of the averages'
// kernels with sums in registers took 12.2 us for 300 000 elements in [1,4,3] and 134 for 10^8; this 10.8 and 96).
template <bool kOne>
__global__ __launch_bounds__(64 * kDecWaves) void k_decode(Layout lay, const uint32_t *__restrict__ words,
                                                           uint64_t words_stride,
                                                           const uint64_t *__restrict__ chunk_offset,
                                                           const uint16_t *__restrict__ sub_bits,
                                                           const BookDev *__restrict__ books, uint8_t *__restrict__ sym,
                                                           uint64_t sym_stride, float *__restrict__ q, uint64_t q_stride,
                                                           uint64_t *__restrict__ status, uint32_t by_chunk, AggArgs one)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const uint32_t tab_words = dec_table_entries(lay.A) / 2;
    const uint32_t win_words = stage_window_words(lay.A);
    uint32_t *s_tab = smem;                                                    // [tab_words]
    uint32_t *s_win = s_tab + front_words(tab_words);                          // [kDecWaves][win_words]
    int32_t *s_book = reinterpret_cast<int32_t *>(s_win + kDecWaves * win_words);   // [kDecWaves], part of the row behind
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    uint64_t c = (uint64_t)blockIdx.x * kDecWaves + wave;
    uint32_t u = blockIdx.y;
    if (by_chunk) {
        const uint64_t item = c;
        c = item / lay.U;
        u = (uint32_t)(item - c * lay.U);
    }
    const bool active = c < lay.nchunks;
    const bool several = lay.books_per_user > 1;
    const ChunkGeom g = chunk_geom(lay, active ? c : lay.nchunks - 1);
    const ChunkIndex ix = read_index(lay, active ? c : lay.nchunks - 1, u, words, words_stride, chunk_offset, sub_bits);
    uint32_t *win = s_win + wave * win_words;
    const BookDev *set = books + (lay.per_user_books ? (uint64_t)u * lay.books_per_user : 0u);
    u32x16 packed = 0u;
    DecTable<2> tab;
    tab.init(lds_address(s_tab), lay.A);
    round_toward_zero();
    bool todo = true;
    if (several) {
        if (lane == 0) s_book[wave] = g.book;
        __syncthreads();
    }
    uint32_t w0 = 0;
    do {
        int32_t b = g.book;
        uint32_t w1 = kDecWaves;
        if (several) {
            b = __builtin_amdgcn_readfirstlane(s_book[w0]);
            for (w1 = w0 + 1; w1 < kDecWaves && __builtin_amdgcn_readfirstlane(s_book[w1]) == b;) ++w1;
            if (w0) __syncthreads();   // the stretch before is decoded
        }
        const BookDev *book = set + b;
        load_table(s_tab, book->dsym, 4u * tab_words, t, 64 * kDecWaves);
        __syncthreads();
        if (active && todo && wave >= w0 && wave < w1) {
            todo = false;
            Stream st;
            start_chunk<kRowsByte>(st, g, ix, lds_address(win), window_rows(lay.A));
            decode_started<false>(st, g, ix, lay.A, tab, book, [](uint32_t s) { return s << 8; },
                                  [&](int gr, const uint32_t (&e)[kGroup]) { pack_group(packed, gr, e); });
            finish_chunk(st, ix, status);
        }
        w0 = w1;
    } while (w0 < kDecWaves);
    round_to_nearest();
    if (!active) return;  // whole wavefront; wavefront-level synchronisation only from here on
    // the symbols to rows of 16 words and out in 1 KB pieces of 16 bytes a lane
    uint32_t *s_stage = win;
#pragma unroll
    for (int i = 0; i < kSub / 16; ++i)
        *reinterpret_cast<u32x4 *>(s_stage + lane * kStageStride + 4 * i) =
            u32x4{packed[4 * i], packed[4 * i + 1], packed[4 * i + 2], packed[4 * i + 3]};
    wave_lds_fence();
    const uint8_t *stage_b = reinterpret_cast<const uint8_t *>(s_stage);
    const bool full = g.n == (uint32_t)kChunk;
    if constexpr (kOne) {
        const SymbolValue val(lay.E, lay.M);
        const int up = 127 - (int)uniform((uint32_t)lay.bias[g.seg]);
        const float inv_gain = lay.gain[2 * g.seg + 1];   // 1 unless the plan carries a scale
        auto four = [&](uint32_t e, bool whole) {
            const uint32_t w = s_stage[(e >> 6) * kStageStride + ((e & 63u) >> 2)];
            double avg[4];
#pragma unroll
            for (uint32_t b = 0; b < 4; ++b) avg[b] = 0.0 + (double)__fmul_rn(ldexpf(val(w, 8u * b), up), inv_gain);
            write_four(g, one, e, avg, whole);
        };
        if (full) {
#pragma unroll 4
            for (uint32_t e = 4 * lane; e < (uint32_t)kChunk; e += 256) four(e, true);
        } else {
            for (uint32_t e = 4 * lane; e < g.n; e += 256) four(e, false);
        }
        return;
    }
    if (sym) {
        uint8_t *dst = sym + (uint64_t)u * sym_stride + g.e0;
        if (full) {   // layers start anywhere
#pragma unroll
            for (int k = 0; k < kChunk / 1024; ++k)
                *reinterpret_cast<u32x4_u8 *>(dst + 1024 * k + 16 * lane) =
                    *reinterpret_cast<const u32x4 *>(s_stage + (16 * k + (lane >> 2)) * kStageStride + 4 * (lane & 3u));
        } else {
            for (uint32_t e = lane; e < g.n; e += 64)
                dst[e] = stage_b[(e >> 6) * (kStageStride * 4) + (e & 63u)];
        }
    }
    if (q) {
        const uint64_t pair = (uint64_t)u * lay.nseg + g.seg;
        const SymbolValue val(lay.E, lay.M);
        const int up = 127 - (int)uniform((uint32_t)lay.bias[pair]);
        const float inv_gain = lay.gain[2 * pair + 1];   // 1 unless the plan carries a scale
        float *dst = q + (uint64_t)u * q_stride + g.e0;
        if (full) {
#pragma unroll 4
            for (uint32_t e = 4 * lane; e < (uint32_t)kChunk; e += 256) {
                const uint32_t w = s_stage[(e >> 6) * kStageStride + ((e & 63u) >> 2)];
                f32x4 v;
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) v[b] = __fmul_rn(ldexpf(val(w, 8u * b), up), inv_gain);
                *reinterpret_cast<f32x4_any *>(dst + e) = v;
            }
        } else {
            for (uint32_t e = lane; e < g.n; e += 64)
                dst[e] = __fmul_rn(ldexpf(val(stage_b[(e >> 6) * (kStageStride * 4) + (e & 63u)], 0), up), inv_gain);
        }
    }
}

// A decode table of the values in LDS: the set's own where it was filled for this format, else from the symbols'.
__device__ inline void load_value_table(uint32_t *dst, const BookDev *__restrict__ book, const Layout &lay, uint32_t t,
                                        uint32_t nthreads)
{
    const uint32_t n = dec_table_entries(lay.A);
    if (book->format == dec_format(lay.E, lay.M)) {
        load_table(dst, book->dval, 4u * n, t, nthreads);
    } else {
        for (uint32_t i = t; i < n; i += nthreads) {
            const uint32_t e = book->dsym[i];
            dst[i] = dec_value_bits(e >> 8, lay.E, lay.M) | (e & 0xffu);
        }
    }
}

// Bits of the sum of n users' values in units of the smallest, the users' biases `spread` apart: an entry is below
// 2^(2^E - 1 + M).
__host__ __device__ inline int int_sum_bits(const Layout &lay, int spread, uint32_t n)
{
    return (1 << lay.E) - 1 + lay.M + spread + (n > 1 ? 32 - __builtin_clz(n - 1) : 0);
}

// Smallest and largest bias of the users in a layer, by one wavefront.
__device__ inline void bias_range(const Layout &lay, uint32_t seg, int &lo, int &hi)
{
    const uint32_t lane = threadIdx.x & 63;
    lo = 1 << 20;
    hi = -(1 << 20);
    for (uint32_t u = lane; u < lay.U; u += 64) {
        const int b = lay.bias[(uint64_t)u * lay.nseg + seg];
        lo = b < lo ? b : lo;
        hi = b > hi ? b : hi;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int l = __shfl_xor(lo, o, 64), h = __shfl_xor(hi, o, 64);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
}

constexpr int kAggWaves = 8;
// Users whose symbols a wavefront holds packed at most, 16 registers each.
constexpr int kPackUsers = 4;
// Pieces of the sums on their way out: element i of sub-chunk s at i * stride + s.
constexpr int kAcrossStride = 65, kAcrossBytes = 64 * kAcrossStride * 4;   // a workgroup's 64 rows (or 16 of fp64)
constexpr int kAloneStride = 68;                                           // a wavefront's 16 rows (8 of fp64)
static_assert(16 * kAloneStride <= (int)kStageWords, "the pieces go through the windows");

// Everything the parts of the kernel below share.
struct AggPart {
    const Layout &lay;
    const AggArgs &a;
    uint32_t *smem;
    int32_t *s_book;         // [3][kAggWaves], where a wavefront has a chunk: of its code table; notes
    double *s_all;           // [kSub][kAcrossStride] where the wavefronts' users come in several turns, else nullptr
    ChunkGeom g;
    uint64_t c;
    bool active;
    uint32_t wave, waves;
    // a wavefront's window where each has a chunk: behind the larger table
    __device__ inline uint32_t *alone_window() const
    {
        return smem + front_words(dec_table_entries(lay.A)) + wave * stage_window_words(lay.A);
    }
};

// Decodes users u0, u0 + 1, .. (kAcross: u0 + wave, u0 + wave + waves, ..), `users` of them as far as there are, one after
// the other: on_user(u, ix, st, tab, book) with the chunk started, on_none() in the turns that are left over.
// kBytes: tables of values (4) or of symbols (2).  kAcross: the wavefronts of the workgroup share a chunk; else each has
// a chunk of its own.  in_order: users u0, u0 + 1, .. with kAcross too.  place(i): where the lane goes on in its sub-chunk (see
// StreamPlaces); to_end: the sub-chunks are decoded to their ends.  kAhead: (kAcross) a user's index is asked for ahead of the user
// before, the first one's ahead of the table.
struct FromTheStart {
    __device__ inline uint32_t operator()(uint32_t) const { return 0u; }
};
template <bool kAcross, int kBytes, int kUsers, bool kAhead = true, class OnUser, class Place = FromTheStart>
__device__ inline void each_user(const AggPart &p, uint32_t u0, uint32_t users, OnUser on_user, bool in_order = false, Place place = Place{}, bool to_end = true)
{
    const Layout &lay = p.lay;
    const uint32_t t = threadIdx.x;
    const uint32_t tab_words = dec_table_entries(lay.A) * kBytes / 4u;
    auto load = [&](uint32_t *dst, const BookDev *book, uint32_t thread, uint32_t nthreads) {
        if (kBytes == 2) load_table(dst, book->dsym, 4u * tab_words, thread, nthreads);
        else load_value_table(dst, book, lay, thread, nthreads);
    };
    auto decode = [&](uint32_t i, uint32_t u, const ChunkIndex &ix, uint32_t *win, const DecTable<kBytes> &tab, const BookDev *book) {
        Stream st;
        const uint32_t from = place(i);
        start_chunk<kRowsByte>(st, p.g, ix, lds_address(win), window_rows(lay.A), from & 0x7fffu);
        st.bad = (from & 0x8000u) != 0u;
        on_user(i, u, ix, st, tab, book);
        if (to_end) finish_chunk(st, ix, p.a.status);
        else wave_lds_fence();
    };
    auto request_of = [&](uint32_t u) { return request_index(lay, p.c, uniform(u), p.a.chunk_offset, p.a.sub_bits); };
    DecTable<kBytes> tab;
    if constexpr (kAcross) {
        const bool own = lay.per_user_books != 0;
        uint32_t *my_tab = p.smem + (own ? p.wave * tab_words : 0u);
        uint32_t *win = p.smem + front_words((own ? p.waves : 1u) * tab_words) + p.wave * window_words(lay.A);
        tab.init(lds_address(my_tab), lay.A);
        auto user_of = [&](uint32_t i) { return u0 + (in_order ? i : p.wave + i * p.waves); };
        IndexAhead ahead;
        if (kAhead && user_of(0) < lay.U) ahead = request_of(user_of(0));
        if (!own) {
            load(my_tab, p.a.books + p.g.book, t, 64 * p.waves);
            __syncthreads();
        }
        auto turn = [&](uint32_t i) {
            const uint32_t u = user_of(i);
            if (u >= lay.U) return;
            const ChunkIndex ix = kAhead ? take_index(ahead, u, p.a.words, p.a.words_stride)
                                         : read_index(lay, p.c, u, p.a.words, p.a.words_stride, p.a.chunk_offset, p.a.sub_bits);
            if (kAhead && user_of(i + 1) < lay.U && i + 1 < users) ahead = request_of(user_of(i + 1));
            const BookDev *book = p.a.books + p.g.book;
            if (own) {
                book += (uint64_t)u * lay.books_per_user;
                load(my_tab, book, t & 63u, 64);
            }
            decode(i, u, ix, win, tab, book);
        };
        if constexpr (kUsers > 0) {
#pragma unroll
            for (uint32_t i = 0; i < (uint32_t)kUsers; ++i) turn(i);
        } else {
#pragma unroll 1
            for (uint32_t i = 0; i < users; ++i) turn(i);
        }
    } else {
        uint32_t *win = p.alone_window();
        tab.init(lds_address(p.smem), lay.A);
        // where the code table changes among the chunks (layers), one stretch after the other
        uint32_t w0 = 0;
        do {
            int32_t b = p.g.book;
            uint32_t w1 = kAggWaves;
            if (lay.books_per_user > 1) {
                b = __builtin_amdgcn_readfirstlane(p.s_book[w0]);
                for (w1 = w0 + 1; w1 < kAggWaves && __builtin_amdgcn_readfirstlane(p.s_book[w1]) == b;) ++w1;
            }
            const bool mine = p.active && p.wave >= w0 && p.wave < w1;
            IndexAhead ahead;
            if (mine && u0 < lay.U) ahead = request_of(u0);
            auto turn = [&](uint32_t i) {
                const uint32_t u = u0 + i;
                if (u >= lay.U) return;
                ChunkIndex ix;
                if (mine) {
                    ix = take_index(ahead, u, p.a.words, p.a.words_stride);
                    if (u + 1 < lay.U && i + 1 < users) ahead = request_of(u + 1);
                }
                const BookDev *book = p.a.books + (lay.per_user_books ? (uint64_t)u * lay.books_per_user : 0u) + b;
                if (i == 0 || lay.per_user_books) {
                    if (i || w0) __syncthreads();   // the table before is done with
                    load(p.smem, book, t, 64 * kAggWaves);
                    __syncthreads();
                }
                if (mine) decode(i, u, ix, win, tab, book);
            };
            if constexpr (kUsers > 0) {
#pragma unroll
                for (uint32_t i = 0; i < (uint32_t)kUsers; ++i) turn(i);
            } else {
#pragma unroll 1
                for (uint32_t i = 0; i < users; ++i) turn(i);
            }
            w0 = w1;
        } while (w0 < kAggWaves);
    }
}

// The sums leave the registers: of(j) is this lane's sum of element j as a T (j a constant in [J0, J1)), `unit` what a sum of 1 is
// worth.  kAcross: they are added up over the workgroup's wavefronts, fp64 in their order.  Where the users come in
// several turns (first .. last), p.s_all keeps the sums.  at_element: of j = 0.
template <bool kAcross, class T, int J0, int J1, class Of>
__device__ inline void write_sums(const AggPart &p, double unit, Of of, bool first = true, bool last = true, int at_element = 0)
{
    const uint32_t t = threadIdx.x, lane = t & 63;
    const double inv_u = 1.0 / (double)p.lay.U;
    const bool whole = p.g.n == (uint32_t)kChunk;
    constexpr int rows = sizeof(T) == 4 ? (kAcross ? 64 : 16) : (kAcross ? 16 : 8);
    constexpr uint32_t per = rows / 4;   // groups of four elements per sub-chunk
    if constexpr (kAcross) {
#pragma unroll
        for (int j = J0; j < J1; j += rows) {
            // over tables and windows, which are done with
            T *s_sum = p.s_all ? reinterpret_cast<T *>(p.s_all) + j * kAcrossStride : reinterpret_cast<T *>(p.smem);
            __syncthreads();
            T v[rows];
#pragma unroll
            for (int i = 0; i < rows; ++i) v[i] = sizeof(T) == 8 ? here(of(j + i)) : of(j + i);
            // (the sums are exact for any reasonable spread of the biases; up to four users keep their order anyhow)
            const uint32_t turns = sizeof(T) == 8 && p.lay.U <= 4u ? p.waves : 2u;
#pragma unroll 1
            for (uint32_t w = 0; w < turns; ++w) {
                if (turns == 2u && w ? p.wave > 0u : p.wave == w) {
#pragma unroll
                    for (int i = 0; i < rows; ++i) {
                        T *at = &s_sum[i * kAcrossStride + lane];
                        if (w == 0 && first) *at = v[i];
                        else __hip_atomic_fetch_add(at, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
                __syncthreads();
            }
#pragma unroll 1
            for (uint32_t k = here(t); last && k < 64 * per; k += 64 * p.waves) {
                const uint32_t s = k / per, i = 4 * (k % per);
                double avg[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) avg[b] = (double)s_sum[(i + b) * kAcrossStride + s] * unit * inv_u;
                write_four(p.g, p.a, s * kSub + (uint32_t)(at_element + j) + i, avg, whole);
            }
        }
    } else if (p.active) {
        T *s_sum = reinterpret_cast<T *>(p.alone_window());
#pragma unroll
        for (int j = J0; j < J1; j += rows) {
#pragma unroll
            for (int i = 0; i < rows; ++i) s_sum[i * kAloneStride + lane] = of(j + i);
            wave_lds_fence();
            const uint32_t l = here(lane);
            auto four = [&](uint32_t k, bool w) {
                const uint32_t s = k / per, i = 4 * (k % per);
                double avg[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) avg[b] = (double)s_sum[(i + b) * kAloneStride + s] * unit * inv_u;
                write_four(p.g, p.a, s * kSub + (uint32_t)(at_element + j) + i, avg, w);
            };
            if (whole) {
#pragma unroll
                for (uint32_t k = 0; k < 64 * per; k += 64) four(l + k, true);
            } else {
#pragma unroll 1
                for (uint32_t k = l; k < 64 * per; k += 64) four(k, false);
            }
            wave_lds_fence();
        }
    }
}

// Users a wavefront takes.  A chunk's wavefronts are as many as its users, or a power of two: no quotient, which would be found
// by an fp32 reciprocal while the conversions round toward zero.
__device__ inline uint32_t users_each(const Layout &lay, uint32_t waves, bool across)
{
    if (!across) return lay.U;
    return lay.U <= waves ? 1u : (lay.U + waves - 1u) >> (31 - __builtin_clz(waves));
}

// The value of a decoded entry's symbol where tables hold symbols.
struct SymbolEntry {
    __device__ inline uint32_t operator()(uint32_t s) const { return s << 8; }
};

// sum + fl32(value * inv_gain) of a symbol; val: its value at exponent bias 127, times `scale` at its own.
template <bool kGain>
__device__ inline double add_value(float val, double scale, float inv_gain, double sum)
{
    if constexpr (kGain) return sum + (double)__fmul_rn((float)((double)val * scale), inv_gain);
    return __builtin_fma((double)val, scale, sum);   // the product is exact
}

// Integer sums in units of 2^(1 - M - bias_hi), exact while they fit 32 bits; wide: the wavefronts' sums do, the
// workgroup's need fp64.
template <bool kAcross>
__device__ inline void aggregate_int(const AggPart &p, int bias_hi, bool wide)
{
    const int E = p.lay.E, M = p.lay.M;
    int32_t sum[kSub];
#pragma unroll
    for (int i = 0; i < kSub; ++i) sum[i] = 0;
    each_user<kAcross, 4, 0>(
        p, 0, users_each(p.lay, p.waves, kAcross),
        [&](uint32_t, uint32_t u, const ChunkIndex &ix, Stream &st, const DecTable<4> &tab, const BookDev *book) {
            const int shift = bias_hi - (int)uniform((uint32_t)p.lay.bias[(uint64_t)u * p.lay.nseg + p.g.seg]);
            auto value = [E, M](uint32_t s) { return dec_value_bits(s, E, M); };
            decode_started<true>(st, p.g, ix, p.lay.A, tab, book, value, [&](int gr, const uint32_t (&e)[kGroup]) {
#pragma unroll
                for (int b = 0; b < kGroup; ++b)
                    sum[gr * kGroup + b] = here(sum[gr * kGroup + b] + (((int32_t)e[b] >> 8) << shift));
            });
        });
    round_to_nearest();
    const double unit = __longlong_as_double((long long)(1023 + 1 - M - bias_hi) << 52);
    if (kAcross && wide) write_sums<kAcross, double, 0, kSub>(p, unit, [&](int j) { return (double)sum[j]; });
    else write_sums<kAcross, int32_t, 0, kSub>(p, unit, [&](int j) { return sum[j]; });
}

// Where the users' streams stand between the parts that aggregate_spread takes: a lane's place in its sub-chunk (below 2^15
// bits: half of it), in the top bit whether a code was damaged before it.
struct StreamPlaces {
    uint16_t *at;     // behind everything else in LDS
    uint32_t users;   // of a wavefront's; the others are decoded from the start in every part
    __device__ inline uint16_t &of(const AggPart &p, uint32_t i) const { return at[(p.wave * users + i) * 64u + (threadIdx.x & 63u)]; }
};

// Sums in fp64, from the packed symbols of up to kUsers users at a time; any format and bias, kGain: and scale.
template <int kUsers, bool kGain, bool kAcross>
__device__ inline void aggregate_packed(const AggPart &p)
{
    const Layout &lay = p.lay;
    u32x16 pk[kUsers];
    const uint32_t step = kAcross ? p.waves : 1u;
    const SymbolValue val(lay.E, lay.M);
    for (uint32_t u0 = 0; u0 < lay.U; u0 += step * kUsers) {
#pragma unroll
        for (int s = 0; s < kUsers; ++s) pk[s] = 0u;
        each_user<kAcross, 2, kUsers>(
            p, u0, kUsers,
            [&](uint32_t i, uint32_t, const ChunkIndex &ix, Stream &st, const DecTable<2> &tab, const BookDev *book) {
                decode_started<false>(st, p.g, ix, p.lay.A, tab, book, SymbolEntry{},
                                             [&](int gr, const uint32_t (&e)[kGroup]) { pack_group(pk[i], gr, e); });
            });
        round_to_nearest();
        auto pair_of = [&](int s) {
            const uint32_t u = u0 + (kAcross ? p.wave : 0u) + (uint32_t)s * step;
            return (uint64_t)(u < lay.U ? u : 0u) * lay.nseg + p.g.seg;
        };
        double scale[kUsers];
#pragma unroll
        for (int s = 0; s < kUsers; ++s) {
            const int bias = (int)uniform((uint32_t)lay.bias[pair_of(s)]);
            scale[s] = __longlong_as_double((long long)(1023 + 127 - bias) << 52);
        }
        const bool last = u0 + step * kUsers >= lay.U;
        if (kGain) {
            float inv_gain[kUsers];
#pragma unroll
            for (int s = 0; s < kUsers; ++s) inv_gain[s] = lay.gain[2 * pair_of(s) + 1];
            auto sum_of = [&](int j) {   // in the users' order; the products round: not before the mode is back
                double sum = 0.0;
#pragma unroll
                for (int s = 0; s < kUsers; ++s)
                    sum = add_value<true>(val(here(pk[s][j >> 2]), 8u * (uint32_t)(j & 3)), scale[s], inv_gain[s], sum);
                return sum;
            };
            write_sums<kAcross, double, 0, kSub>(p, 1.0, sum_of, u0 == 0, last);
        } else {
            auto sum_of = [&](int j) {
                double sum = 0.0;
#pragma unroll
                for (int s = 0; s < kUsers; ++s)
                    sum = add_value<false>(val(pk[s][j >> 2], 8u * (uint32_t)(j & 3)), scale[s], 1.0f, sum);
                return sum;
            };
            write_sums<kAcross, double, 0, kSub>(p, 1.0, sum_of, u0 == 0, last);
        }
        if (kAcross && !last) {
            round_toward_zero();
            __syncthreads();
        }
    }
}

// The same users where the biases lie too far apart for that, or (kGain) one carries a scale: fp64 sums, of one of kParts parts
// of every sub-chunk at a time, for more do not fit the registers.  ordered: in the users' order.
// A wavefront keeps where its users' streams stand, so that every symbol is decoded once: decoded anew with every part, eight
// users of 25 M elements in [1,4,3] with biases 14 binades apart 228 us, this way 177.
template <bool kAcross, bool kGain, int kParts>
__device__ inline void aggregate_spread(const AggPart &p, const StreamPlaces &places, bool ordered)
{
    constexpr int kPart = kSub / kParts, kPartGroups = kGroups / kParts;
    const SymbolValue val(p.lay.E, p.lay.M);
#pragma unroll 1
    for (int part = 0; part < kParts; ++part) {
        double sum[kPart];
#pragma unroll
        for (int i = 0; i < kPart; ++i) sum[i] = 0.0;
        const int from = part * kPartGroups;
        auto on_user = [&](uint32_t i, uint32_t u, const ChunkIndex &ix, Stream &st, const DecTable<2> &tab, const BookDev *book) {
            typedef uint32_t words_t __attribute__((ext_vector_type(kPart / 4)));
            const bool kept = i < places.users;
            words_t packed = 0u;
            decode_started<false>(
                st, p.g, ix, p.lay.A, tab, book, SymbolEntry{},
                [&](int gr, const uint32_t (&e)[kGroup]) {
                    if (gr >= from) pack_group(packed, gr - from, e);
                },
                kept ? from : 0, from + kPartGroups);
            if (kept && part + 1 < kParts)
                places.of(p, i) = (uint16_t)(((st.bit() - (st.end - ix.sb)) & 0x7fffu) | (st.bad ? 0x8000u : 0u));
            const uint64_t pair = (uint64_t)u * p.lay.nseg + p.g.seg;
            const int bias = (int)uniform((uint32_t)p.lay.bias[pair]);
            const double scale = __longlong_as_double((long long)(1023 + 127 - bias) << 52);
            const float inv_gain = kGain ? p.lay.gain[2 * pair + 1] : 1.0f;
            if constexpr (kGain) round_to_nearest();   // (the products round)
#pragma unroll
            for (int k = 0; k < kPart; ++k) {
                const uint32_t w = kGain ? here(packed[k >> 2]) : packed[k >> 2];
                sum[k] = here(add_value<kGain>(val(w, 8u * (uint32_t)(k & 3)), scale, inv_gain, sum[k]));
            }
            if constexpr (kGain) round_toward_zero();
        };
        auto place = [&](uint32_t i) { return part == 0 || i >= places.users ? 0u : (uint32_t)places.of(p, i); };
        each_user<kAcross, 2, 0>(p, 0, ordered ? (p.wave ? 0u : p.lay.U) : users_each(p.lay, p.waves, kAcross), on_user, ordered, place, part + 1 == kParts);
        round_to_nearest();
        write_sums<kAcross, double, 0, kPart>(p, 1.0, [&](int j) { return sum[j]; }, true, true, part * kPart);
        round_toward_zero();
        __syncthreads();
    }
}

// Users whose symbols meet in LDS at most: two a wavefront, 5 KB each, as many as a CU's 160 KB hold.  (Four a wavefront: sixteen
// users of 12 M elements in [1,5,2], a round 600 us from the sums, 794 this way.)
constexpr uint32_t kStageWaves = 16, kStageUsers = 31;
__host__ __device__ constexpr uint32_t stage_bytes(uint32_t U) { return 4u * U * kStageWords + kStageUsers * (uint32_t)(sizeof(double) + sizeof(float)); }
static_assert(kStageUsers <= 2 * kStageWaves && stage_bytes(kStageUsers) <= 160 * 1024, "a turn, and a CU");
// The same sums where the workgroup's wavefronts decode all users in one turn: the symbols meet in LDS, an eighth of what
// the fp64 sums would be, and every thread adds up its elements in the users' order, where the sums would be added up by
// one wavefront after the other (the others at barriers).  A small launch is one workgroup's way: a round of three users of
// 63 112 elements in [1,4,1] with a scale 29.5 -> 23.2 us, of four of 600 001 in [1,5,2] with a table each 47 -> 40, of ten
// of 10^6 in [1,4,3] with a scale 86 -> 70, of sixteen of 300 001 in [1,5,2] 66 -> 60.
template <int kUsers, bool kAhead>
__device__ inline void aggregate_staged(const AggPart &p)
{
    const Layout &lay = p.lay;
    double *s_scale = reinterpret_cast<double *>(p.smem + lay.U * kStageWords);   // [kStageUsers], behind the symbols
    float *s_inv_gain = reinterpret_cast<float *>(s_scale + kStageUsers);         // [kStageUsers]
    const uint32_t t = threadIdx.x, lane = t & 63u;
    int bias = 0;
    float inv_gain = 1.0f;
    if (t < lay.U) {   // a workgroup has as many threads; requested here, needed when the users are decoded
        const uint64_t pair = (uint64_t)t * lay.nseg + p.g.seg;
        bias = lay.bias[pair];
        inv_gain = lay.gain[2 * pair + 1];
    }
    u32x16 pk[kUsers];
#pragma unroll
    for (int s = 0; s < kUsers; ++s) pk[s] = 0u;
    each_user<true, 2, kUsers, kAhead>(
        p, 0, kUsers,
        [&](uint32_t i, uint32_t, const ChunkIndex &ix, Stream &st, const DecTable<2> &tab, const BookDev *book) {
            decode_started<false>(st, p.g, ix, lay.A, tab, book, SymbolEntry{},
                                         [&](int gr, const uint32_t (&e)[kGroup]) { pack_group(pk[i], gr, e); });
        });
    round_to_nearest();
    __syncthreads();   // tables and windows are done with
    if (t < lay.U) {
        s_scale[t] = __longlong_as_double((long long)(1023 + 127 - bias) << 52);
        s_inv_gain[t] = inv_gain;
    }
#pragma unroll
    for (int s = 0; s < kUsers; ++s) {
        const uint32_t u = p.wave + (uint32_t)s * p.waves;
        if (u >= lay.U) break;
        uint32_t *row = p.smem + u * kStageWords + lane * kStageStride;
#pragma unroll
        for (int i = 0; i < kSub / 16; ++i)
            *reinterpret_cast<u32x4 *>(row + 4 * i) = u32x4{pk[s][4 * i], pk[s][4 * i + 1], pk[s][4 * i + 2], pk[s][4 * i + 3]};
    }
    __syncthreads();
    const SymbolValue val(lay.E, lay.M);
    const double inv_u = 1.0 / (double)lay.U;
    const bool whole = p.g.n == (uint32_t)kChunk;
    for (uint32_t k = t; k < (uint32_t)kChunk / 4; k += 64 * p.waves) {   // elements 4 k .. 4 k + 3
        const uint32_t *at = p.smem + (k >> 4) * kStageStride + (k & 15u);
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
        if (__builtin_expect(p.g.scaled, 0)) {
#pragma unroll 4
            for (uint32_t u = 0; u < lay.U; ++u) {
                const uint32_t w = at[u * kStageWords];
                const double scale = s_scale[u];
                const float inv = s_inv_gain[u];
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) sum[b] = add_value<true>(val(w, 8u * b), scale, inv, sum[b]);
            }
        } else {
#pragma unroll 4
            for (uint32_t u = 0; u < lay.U; ++u) {
                const uint32_t w = at[u * kStageWords];
                const double scale = s_scale[u];
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) sum[b] = add_value<false>(val(w, 8u * b), scale, 1.0f, sum[b]);
            }
        }
        double avg[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) avg[b] = sum[b] * inv_u;
        write_four(p.g, p.a, 4 * k, avg, whole);
    }
}

// Shared by the kernels below: the wavefront's chunk.  kAcross: the wavefronts of a workgroup share a chunk and split
// the users, else each has a chunk.
template <bool kAcross>
__device__ inline AggPart agg_part(const Layout &lay, const AggArgs &a, uint32_t *smem, uint32_t all_at)
{
    const uint32_t wave = uniform(threadIdx.x >> 6);
    uint64_t c = blockIdx.x;
    if constexpr (!kAcross) c = c * kAggWaves + wave;
    const bool active = c < lay.nchunks;
    if (!active) c = lay.nchunks - 1;
    int32_t *s_book = reinterpret_cast<int32_t *>(smem + front_words(dec_table_entries(lay.A)) + kAggWaves * stage_window_words(lay.A));
    return AggPart{lay, a, smem, s_book, all_at ? reinterpret_cast<double *>(smem + all_at) : nullptr,
                   uniform(chunk_geom(lay, c)), c, active, wave, kAcross ? blockDim.x >> 6 : (uint32_t)kAggWaves};
}

// The layer's entry and biases say which way the sums take, and not the host: a captured launch may be replayed on a plan that
// has been given a scale or other biases since.
// Where each wavefront has a chunk of its own: tells the others its code table, and whether x; one of them takes all along
// (they meet at barriers).  note: 1 or 2, another with each call.
__device__ inline bool any_wave(const AggPart &p, bool x, int note)
{
    if ((threadIdx.x & 63) == 0) {
        p.s_book[p.wave] = p.g.book;
        p.s_book[note * kAggWaves + (int)p.wave] = x ? 1 : 0;
    }
    __syncthreads();
    return __any(p.s_book[note * kAggWaves + (int)(threadIdx.x & (kAggWaves - 1))] != 0);
}

// The way of what the kernels below are not made for: sums that do not fit integers, a scale that the host does not know of.
// It reads the kernel's arguments (Layout and AggArgs come first) anew and looks its chunk up again, so that nothing of its
// own is held in registers over the kernel's usual way (in k_aggregate_int: eight users of 10^6 elements in [1,4,3] 13.3 us
// with the kernel's own values, 12.6 this way).
template <bool kAcross>
__device__ __forceinline__ void aggregate_rare(uint32_t *smem, uint32_t places_at, uint32_t places)
{
    struct Arguments { Layout lay; AggArgs a; };
    uint64_t arguments = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(arguments));
    const Arguments *k = (const Arguments *)(const __attribute__((address_space(4))) Arguments *)arguments;
    const Layout lay = k->lay;
    const AggArgs a = k->a;
    const AggPart p = agg_part<kAcross>(lay, a, smem, 0);
    const StreamPlaces sp = {reinterpret_cast<uint16_t *>(smem + places_at), places};
    bool scaled = p.g.scaled, ordered = false;
    if constexpr (!kAcross) scaled = any_wave(p, scaled, 2);
    if constexpr (kAcross) {
        // up to four users keep their order where it can make a difference: sums of more than 53 bits, or with a scale
        int lo, hi;
        bias_range(lay, p.g.seg, lo, hi);
        ordered = lay.U <= 4u && p.waves < lay.U && (p.g.scaled || int_sum_bits(lay, hi - lo, lay.U) > 53);
        if (lay.U <= 2u * p.waves && stage_bytes(lay.U) <= 4u * places_at) return aggregate_staged<2, true>(p);
    }
    if (scaled) aggregate_spread<kAcross, true, 4>(p, sp, ordered);
    else aggregate_spread<kAcross, false, 2>(p, sp, ordered);
}

// co3_ps_aggregate with integer sums (formats of up to four exponent bits; layers without a real-valued scale).
template <bool kAcross>
__global__ __launch_bounds__(64 * kAggWaves, 4) void k_aggregate_int(Layout lay, AggArgs a, uint32_t places_at, uint32_t places)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const AggPart p = agg_part<kAcross>(lay, a, smem, 0);
    round_toward_zero();
    int lo, hi;
    bias_range(lay, p.g.seg, lo, hi);
    const bool fits = int_sum_bits(lay, hi - lo, users_each(lay, p.waves, kAcross)) <= 31;
    const bool wide = int_sum_bits(lay, hi - lo, lay.U) > 31;
    bool rare = p.g.scaled || !fits;
    if constexpr (!kAcross) rare = any_wave(p, rare, 1);
    if (__builtin_expect(rare, 0)) aggregate_rare<kAcross>(smem, places_at, places);
    else aggregate_int<kAcross>(p, hi, wide);
}

// co3_ps_aggregate for everything else.  kUsers: per wavefront and turn.
template <int kUsers, bool kGain, bool kAcross>
__global__ __launch_bounds__(64 * kAggWaves, 4) void k_aggregate(Layout lay, AggArgs a, uint32_t all_at, uint32_t places_at, uint32_t places)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const AggPart p = agg_part<kAcross>(lay, a, smem, all_at);
    round_toward_zero();
    bool rare = p.g.scaled;
    if constexpr (!kAcross) rare = any_wave(p, rare, 1);
    if constexpr (!kGain) {
        if (__builtin_expect(rare, 0)) return aggregate_rare<kAcross>(smem, places_at, places);
    }
    aggregate_packed<kUsers, kGain, kAcross>(p);
}

// The same where a workgroup's wavefronts take all users of a chunk in one turn, one or two each.
template <int kUsers, bool kAhead>
__global__ __launch_bounds__(64 * kStageWaves, kUsers == 1 ? 6 : 4) void k_aggregate_staged(Layout lay, AggArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const AggPart p = agg_part<true>(lay, a, smem, 0);
    round_toward_zero();
    aggregate_staged<kUsers, kAhead>(p);
}

__global__ __launch_bounds__(64) void k_mark_scaled(Layout lay, SegDev *__restrict__ segs)
{
    bool any = false;
    for (uint32_t u = threadIdx.x; u < lay.U; u += 64) any = any || lay.gain[2 * ((uint64_t)u * lay.nseg + blockIdx.x) + 1] != 1.0f;
    any = __any(any);
    if (threadIdx.x == 0) segs[blockIdx.x].scaled = any ? 1 : 0;
}

hipError_t launch_mark_scaled(const Layout &lay, SegDev *segs, hipStream_t s)
{
    hipLaunchKernelGGL(k_mark_scaled, dim3(lay.nseg), dim3(64), 0, s, lay, segs);
    return hipGetLastError();
}

static size_t decode_lds(const Layout &lay)
{
    return 4 * ((size_t)front_words(dec_table_entries(lay.A) / 2) + kDecWaves * stage_window_words(lay.A) + kBehindWords);
}

hipError_t launch_decode(const Layout &lay, const co3_decode_args &a, const BookDev *books, hipStream_t s)
{
    if (lay.U == 0 || lay.nchunks == 0) return hipSuccess;
    const uint64_t sym_stride = symbol_row_stride(lay.d);
    const size_t lds = decode_lds(lay);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_decode<false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(K_DECODE, s);
    // Where layers under tables of their own are short, the users' parts of a chunk go to one workgroup: it meets few tables,
    // which it takes one after the other (24 users of 353 444 elements in twelve layers, [1,5,2]: by user 28, by chunk 14 us).
    const bool by_chunk = lay.books_per_user > 1 && !lay.per_user_books;
    const uint64_t chunks = by_chunk ? lay.nchunks * lay.U : lay.nchunks;
    const dim3 grid((uint32_t)((chunks + kDecWaves - 1) / kDecWaves), by_chunk ? 1u : lay.U);
    hipLaunchKernelGGL(k_decode<false>, grid, dim3(64 * kDecWaves), lds, s, lay, a.words, a.words_stride, a.chunk_offset, a.sub_bits,
                       books, a.symbols, sym_stride, a.q, a.q_stride, a.status, by_chunk ? 1u : 0u, AggArgs{});
    return hipGetLastError();
}

// LDS of the averages' kernels: a table (or one for each wavefront with a user's own), windows, where the sums meet.
static size_t aggregate_lds(const Layout &lay, bool values, uint32_t waves, bool across)
{
    const uint32_t table = dec_table_entries(lay.A) / (values || !across ? 1 : 2);   // words
    if (!across) return 4 * ((size_t)front_words(table) + kAggWaves * stage_window_words(lay.A) + kBehindWords);
    const size_t lds = 4 * ((size_t)front_words((lay.per_user_books ? waves : 1) * table) + waves * window_words(lay.A) + kBehindWords);
    return lds > (size_t)kAcrossBytes ? lds : (size_t)kAcrossBytes;
}

template <class Kernel, class... Args>
static hipError_t launch_aggregate_k(Kernel k, const Layout &lay, uint32_t waves, bool across, size_t lds, hipStream_t s, Args... args)
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(K_AGGREGATE, s);
    const uint64_t grid = across ? lay.nchunks : (lay.nchunks + kAggWaves - 1) / kAggWaves;
    hipLaunchKernelGGL(k, dim3((uint32_t)grid), dim3(64 * waves), lds, s, lay, args...);
    return hipGetLastError();
}

// Launches one of the kernels that has aggregate_rare, with room for what that keeps in LDS as far as it costs no workgroup that
// the CU would hold beside (sixteen wavefronts, for the registers hold no more; a workgroup where there are no more than CUs):
// behind the `lds` bytes a place for each of a wavefront's users, and so many in all that the users' symbols can meet there.
template <class Kernel, class... Args>
static hipError_t launch_aggregate_places(Kernel k, const Layout &lay, uint32_t waves, bool across, size_t lds, hipStream_t s, Args... args)
{
    const uint32_t piece = 1280, pieces = 128;   // LDS is given out in pieces (26 880 bytes: six workgroups, 27 136: five)
    uint32_t groups = pieces / (((uint32_t)lds + piece - 1) / piece);
    const uint64_t grid = across ? lay.nchunks : (lay.nchunks + waves - 1) / waves;
    if (groups > 16 / waves) groups = 16 / waves;
    if (groups > (grid + 255) / 256) groups = (uint32_t)((grid + 255) / 256);
    const uint32_t share = pieces / groups * piece;
    if (across && lay.U <= 2 * waves && stage_bytes(lay.U) <= share && stage_bytes(lay.U) > lds) lds = stage_bytes(lay.U);
    const uint32_t at = (uint32_t)((lds + 15) / 16 * 4), per_user = waves * 64 * (uint32_t)sizeof(uint16_t);
    uint32_t places = share > 4 * at ? (share - 4 * at) / per_user : 0;
    const uint32_t users = across ? (lay.U + waves - 1) / waves : lay.U;
    if (places > users) places = users;
    return launch_aggregate_k(k, lay, waves, across, 4 * (size_t)at + (size_t)places * per_user, s, args..., at, places);
}

static size_t staged_lds(const Layout &lay, uint32_t waves)
{
    const size_t lds = aggregate_lds(lay, false, waves, true), stage = stage_bytes(lay.U);
    return lds > stage ? lds : stage;
}
static hipError_t launch_aggregate_staged(const Layout &lay, const AggArgs &a, uint32_t waves, hipStream_t s)
{
    const size_t lds = staged_lds(lay, waves);
    // One user a wavefront: there is none before to ask ahead of, and a launch of up to eight wavefronts a CU waits for the table's
    // first words behind the index (the average in [1,5,2], index ahead of the table and with the user: two users of 10^6 elements
    // 11.1 and 10.85 us, three of 2 M 12.9 and 12.75, four 12.0 and 12.05; eight 14.4 and 14.7; four of 10^7 33.0 and 33.3, of 25 10^7
    // 557 and 571).
    if (lay.U <= waves && (uint64_t)lay.U * lay.nchunks <= 2048) return launch_aggregate_k(k_aggregate_staged<1, false>, lay, waves, true, lds, s, a);
    if (lay.U <= waves) return launch_aggregate_k(k_aggregate_staged<1, true>, lay, waves, true, lds, s, a);
    return launch_aggregate_k(k_aggregate_staged<2, true>, lay, waves, true, lds, s, a);
}

// Wavefronts of a workgroup that takes all users of a chunk in one turn, one each or two, where that is the better way (else 0).  A launch
// of few chunks is a workgroup's way: one turn of decoding, and sums by all threads.  Beyond, it takes what the busiest CU does, a
// workgroup for every 256 chunks ("rounds"); nine to twelve wavefronts cost what twelve do, as one SIMD has three of them, and of
// thirteen and more a CU was seen to hold one workgroup, not two.  us in [1,4,3], this way and integer sums (launch_aggregate(): eight
// wavefronts a chunk up to 512 chunks, four to 1024, two to 2048, then one; each best at the end of its range, where its launch just
// fits the device):
//   rounds       1      2      3      4         5      6      7      8      9
//   8 users    11 12  14 15  18 21  24 23     28 36  32 39  37 58  41 60  45 67
//   10 users   12 17  17 20  25 27  30-34 29  38 42  47 46  53 68  60 71  70 80
//   12 users   12 17  18 20  26 27  31 31     39 48  45 52  51 78  58 82  64 93
//   14 users   14 18  24 22  35 33  47 37     57 53  68 58
// Tables of up to 64 symbols leave room in LDS for all workgroups of two wavefronts to 2048 chunks ([1,2,1], 6 to 8 rounds: 8 users
// 29 36, 34 36, 37 38; 9 users 37-40 41, 43 42, 48-52 43; 10 users 42-46 42, 49 43, 54-59 44).  The sums of other formats are
// left for more than twelve users where a workgroup of them takes sixteen in eight wavefronts and two such fit a CU (two rounds of
// 13 to 15 users, [1,5,2]: 24 22), at four rounds (16 users 50 48) and beyond 1280 or 1400 chunks.
// A table for every wavefront leaves less room in LDS and is a load more before every chunk's first symbol: beyond what the
// device holds (five users of 1264 chunks in [1,2,1] 22, integer sums 29) only tables of up to 64 symbols, to 1250 chunks (of [1,2,1] and [1,3,1], this way and integer
// sums: 1036 chunks of ten users 35 39, of eight 25 33; 1221 of ten 39 41; 1587 of ten 48 44, of eight 33 37; 1954 of ten 57 44,
// of six 34 31).
static uint32_t staged_waves(const Layout &lay, bool ints)
{
    if (lay.U < 2 || lay.U > kStageUsers) return 0;
    const uint32_t each = (lay.U + kStageWaves - 1) / kStageWaves;
    const uint32_t waves = (lay.U + each - 1) / each;
    const uint64_t pieces = (staged_lds(lay, waves) + 1279) / 1280;   // LDS is given out in pieces, 128 of them
    const uint32_t resident = (waves <= 12 ? 32 : 24) / waves;
    const uint64_t per_cu = 128 / pieces < resident ? 128 / pieces : resident;
    if (per_cu == 0) return 0;
    const uint64_t rounds = (lay.nchunks + 255) / 256;   // workgroups of the busiest CU
    const bool few = rounds <= per_cu, small = lay.A <= 64u;
    if (lay.per_user_books && !few && !(lay.U <= 10 && small && lay.nchunks <= 1250)) return 0;
    if (lay.per_user_books && (few || !ints)) return waves;
    if (ints) {
        if (lay.U > 10) return few ? waves : 0;
        if (lay.nchunks > 2500 || (lay.U > 8 && rounds > 9)) return 0;
        if (lay.U > 6 && rounds == 4) return 0;
        if (lay.U > 4 && small && rounds == 8) return 0;
        if (lay.U > 8 && (small ? rounds == 7 || (lay.U > 9 && rounds == 6) : rounds == 6)) return 0;
        return waves;
    }
    if (lay.U <= 12) return lay.U <= 10 || lay.nchunks <= 1400 ? waves : 0;
    if (rounds == 2) return lay.U > 15 ? waves : 0;
    return rounds != 4 && lay.nchunks <= (lay.U <= 16 ? 1400u : 1280u) ? waves : 0;
}

static hipError_t launch_average_of_one(const Layout &lay, const AggArgs &a, hipStream_t s)
{
    const size_t lds = decode_lds(lay);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_decode<true>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ProfScope prof(K_AGGREGATE, s);
    hipLaunchKernelGGL(k_decode<true>, dim3((uint32_t)((lay.nchunks + kDecWaves - 1) / kDecWaves)), dim3(64 * kDecWaves), lds, s, lay, a.words,
                       a.words_stride, a.chunk_offset, a.sub_bits, a.books, static_cast<uint8_t *>(nullptr), (uint64_t)0,
                       static_cast<float *>(nullptr), (uint64_t)0, a.status, 0u, a);
    return hipGetLastError();
}

template <bool kGain>
static hipError_t launch_aggregate_packed(const Layout &lay, const AggArgs &a, uint32_t waves, hipStream_t s)
{
    if (waves <= 1) {
        const size_t lds = aggregate_lds(lay, false, kAggWaves, false);
        return launch_aggregate_places(k_aggregate<kPackUsers, kGain, false>, lay, kAggWaves, false, lds, s, a, 0u);
    }
    if (lay.U <= 2 * waves) return launch_aggregate_staged(lay, a, waves, s);
    size_t lds = aggregate_lds(lay, false, waves, true);
    uint32_t all_at = 0;
    if (lay.U > waves * kPackUsers) {   // several turns: the sums need a place of their own
        all_at = (uint32_t)((lds + 15) / 16 * 4);
        lds = 4 * (size_t)all_at + (size_t)kSub * kAcrossStride * sizeof(double);
    }
    return launch_aggregate_places(k_aggregate<kPackUsers, kGain, true>, lay, waves, true, lds, s, a, all_at);
}

hipError_t launch_aggregate(const Layout &lay, const PlanFacts &facts, const co3_aggregate_args &a, const BookDev *books, hipStream_t s)
{
    if (lay.U == 0 || lay.nchunks == 0) return hipSuccess;
    const AggArgs args = {a.words, a.words_stride, a.chunk_offset, a.sub_bits, books, a.out, a.model, (double)a.eta, a.status};
    if (lay.U == 1) return launch_average_of_one(lay, args, s);
    if (const uint32_t w = staged_waves(lay, dec_value_is_int(lay.E) && !facts.has_gain)) return launch_aggregate_staged(lay, args, w, s);
    // What staged_waves() leaves: many users, or chunks enough to fill the device.
    // A wavefront per user where 4096 are resident at a time (sixteen a CU) and more would wait: what bounds a small
    // launch is one wavefront's way through its users (eight users of 10^6 elements in [1,4,3], eight, four, two
    // wavefronts and one a chunk: 13, 18, 28 and 53 us; of 4 M elements 30, 24, 33, 53).  Beyond, a wavefront per chunk
    // spares the meeting at the end (five users of 25 M: 80 us, two 104, four 109), unless it has many users: the chunks
    // are too few then for an even load (ten users of 25 M 147, 168, 160; sixteen 219, 244, 205; 24 of 12 M 175, 177, 146).
    const uint64_t resident = 4096;
    uint32_t waves = lay.U <= (uint32_t)kAggWaves && lay.nchunks * lay.U <= resident ? lay.U : kAggWaves;
    while (waves > 1 && (waves > lay.U || lay.nchunks * waves > resident)) waves = waves > 4 ? 4 : waves / 2;
    while (lay.U > 12u * waves && waves < kAggWaves) waves = waves < 4 ? 4 : kAggWaves;
    // (tables of their own in LDS per wavefront: the symbols' take half the room of the values'.  Biases set from device memory are
    // taken to lie close together; where they do not, the kernel takes aggregate_rare)
    const bool ints = dec_value_is_int(lay.E) && !facts.has_gain && (!lay.per_user_books || lay.A <= 64u) &&
                      int_sum_bits(lay, facts.bias_spread, (lay.U + waves - 1) / waves) <= 31;
    if (ints) {
        const bool across = waves > 1;
        if (!across) waves = kAggWaves;
        const size_t lds = aggregate_lds(lay, true, waves, across);
        return across ? launch_aggregate_places(k_aggregate_int<true>, lay, waves, true, lds, s, args)
                      : launch_aggregate_places(k_aggregate_int<false>, lay, waves, false, lds, s, args);
    }
    while (waves * kPackUsers < lay.U && waves < kAggWaves) waves = waves < 2 ? 2 : (waves < 4 ? 4 : kAggWaves);
    return facts.has_gain ? launch_aggregate_packed<true>(lay, args, waves, s) : launch_aggregate_packed<false>(lay, args, waves, s);
}

}  // namespace co3
