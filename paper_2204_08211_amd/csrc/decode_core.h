// Wavefront-level core of the decoder (Sec. II-B (iv)): lane j of a wavefront decodes sub-chunk j (64 symbols) of a
// chunk, eight symbols at a time, shared by co3_decode and the PS average (k_decode.hip).
//
// Table.  Canonical codes grow with their length, so the long codes are the largest prefixes.  With u the complement of
// the next 32 bits and k the number of its leading zeros, the codeword at the front has at most k + log2(A) bits: it is
// all ones (and not longer than k), or its first zero is at bit k; in the latter case the prefix of k + 1 ones behind it
// has to hold codes as long or longer, a share of 2^-(k+1) of the code space, at least 2^(len - k - 1) of them, and there
// are fewer than A.  So u's exponent and log2(A) - 1 bits behind its leading one - the top bits of u as a floating point
// number - index a table that resolves every code of up to 31 bits in one look-up: 32 binades of A / 2 entries, 16 KB
// for 256 symbols, 1 KB for 16.  (The binade of u < 4 holds no codes; longer codes, streams that are not one and the
// absent second codeword of a code of one symbol take the slow path.)
//
// Reader.  A lane's words lie complemented and in reverse order in its column of LDS, so that the stream is one large
// number read from its top: 32 bits at any bit address N are two LDS words and one v_alignbit, with nothing carried from
// symbol to symbol but N.  A window serves two symbols (together 31 bits at most: otherwise the group's lanes concerned
// take the slow path, one window per symbol).
//
// What bounds it: vector instructions (some nine per symbol of a wavefront, 27 in the form this replaced: two words and an
// offset in registers, an 11-bit table and second-level tables), the LDS look-ups of 64 lanes at unrelated addresses, and
// the chain of three LDS reads per pair.  Sixteen users of 25.6 M elements in [1,4,3] (6.9 bit/element): decoded to
// symbols 365 -> 172 us, averaged 380 -> 228 us; with the words of a chunk in order in LDS, where two of the lanes'
// reads in three met in a bank, 200 us.
#pragma once

#include "co3_internal.h"
#include "quantize_math.h"
#include "wave_ops.h"

namespace co3 {

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A wavefront's window: rows of 64 words, the word of lane j in column j, so that the lanes' reads never meet in a bank.
// Word k behind the one with the lane's position when the window was loaded lies k rows below the top row.
constexpr uint32_t kRowBytes = 256;
// Bits that a group reads at most, on the slow path too: eight of the longest codes an alphabet can have, and a window.
__host__ __device__ constexpr uint32_t group_bits(uint32_t A) { return 8u * (A > 64u ? 64u : A - 1u) + 64u; }
// Rows, a multiple of four: room for a sub-chunk of the bits its symbols have and an eighth more, and for a group.  A lane
// whose sub-chunk is longer loads again on the way.
__host__ __device__ constexpr uint32_t window_rows(uint32_t A)
{
    const uint32_t nbits = (uint32_t)(31 - __builtin_clz(A));
    return nbits > 8u ? 24u : (nbits >= 6u ? 20u : (2u * nbits + 5u) & ~3u);
}
__host__ __device__ constexpr bool holds_group(uint32_t A) { return 32u * (window_rows(A) - 1u) - 31u >= group_bits(A); }
static_assert(holds_group(8) && holds_group(16) && holds_group(32) && holds_group(64) && holds_group(128) && holds_group(256) && holds_group(4096),
              "wherever a window starts in its first word, it holds a group");
constexpr int kRowsByte = 20, kRowsWide = 24;   // at most; 8 at least: formats have three bits or more
__host__ __device__ constexpr uint32_t window_words(uint32_t A) { return window_rows(A) * 64u; }
// In front of the windows lies at least this much (tables): a group of a damaged stream reads up to eight rows below its
// window before it is found out.
constexpr uint32_t kFrontWords = 8 * kRowBytes / 4;
__host__ __device__ constexpr uint32_t front_words(uint32_t table_words) { return table_words < kFrontWords ? kFrontWords : table_words; }
constexpr uint32_t kBehindWords = 64;   // and a row behind them: the reader takes a word from the row above its place
constexpr int kGroup = 8;                           // symbols decoded between two checks
constexpr int kGroups = kSub / kGroup;

__device__ inline uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ inline uint32_t lds_word(uint32_t byte) { return *(const lds_u32 *)byte; }

__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Between the two, conversions to fp32 round toward zero, so that u's leading bits survive; nothing else there rounds in
// fp32.  (Register MODE, its two bits for fp32.)  The conversions take words read from LDS behind a fence and feed
// addresses of reads before one, so they stay where they are written.
__device__ inline void round_toward_zero() { __builtin_amdgcn_s_setreg(1 | (1 << 11), 3); }
__device__ inline void round_to_nearest() { __builtin_amdgcn_s_setreg(1 | (1 << 11), 0); }

// A value made here and not earlier (what depends on the lane alone would be computed once per kernel) or not later (a
// group's entries would wait for their use at the end): both would hold registers over the decoding.
template <class T>
__device__ inline T here(T x)
{
    asm volatile("" : "+v"(x));
    return x;
}
// The same for sixteen words, one by one: they need not lie side by side.  fp32 arithmetic on decoded symbols in registers
// stays behind round_to_nearest() by taking them from here: the compiler knows no order between MODE and arithmetic.
template <class Words>
__device__ inline void words_here(Words &w)
{
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = here(w[i]);
}

// Where an entry lies in its table: byte alphabets, bytes from the table's start (key: u as fp32, rounded toward zero) ...
__host__ __device__ inline uint32_t byte_table_shift(uint32_t A, uint32_t bytes)
{
    return 24u - (31u - (uint32_t)__builtin_clz(A)) - (bytes == 4u ? 2u : 1u);
}
__host__ __device__ inline uint32_t byte_table_mask(uint32_t A, uint32_t bytes) { return dec_table_entries(A) * bytes - bytes; }
__host__ __device__ inline uint32_t byte_table_at(uint32_t key, uint32_t shift, uint32_t mask) { return (key >> shift) & mask; }
// ... and wide ones, where the field `off`, `width` of the key (u itself, or the larger of u and this as fp32) is the index, less
// wide_table_first(bits)
constexpr uint32_t kWideTabLeast = 2u << kWideTabLow;   // the lowest binade holds nothing
__host__ __device__ inline uint32_t wide_table_off(uint32_t bits) { return bits ? 23u - bits : 32u - kWidePrefixBits; }
__host__ __device__ inline uint32_t wide_table_width(uint32_t bits) { return bits ? bits + 5u : kWidePrefixBits; }
__host__ __device__ inline uint32_t wide_table_first(uint32_t bits) { return bits ? kWideTabLow << bits : 0u; }

// Where the entries of a code lie in LDS.  Entry: code length in bits 0..7 (kLenSlow: slow path), above it what the sink
// asks for.  kBytes 4 or 2 per entry.  The table lies at a multiple of its size.
template <int kBytes>
struct DecTable {
    static constexpr int kMaxRows = kRowsByte;
    uint32_t base;    // LDS address
    uint32_t shift, mask;
    __device__ inline void init(uint32_t address, uint32_t A)
    {
        base = address;
        shift = byte_table_shift(A, kBytes);
        mask = here(byte_table_mask(A, kBytes));   // (v_and_or_b32 takes one scalar operand)
    }
    // u is a window's complement, whole: an entry of a code of 25 bits or more depends on its low byte too
    __device__ inline uint32_t operator()(uint32_t u) const
    {
        const float f = (float)u;
        const uint32_t a = byte_table_at(__float_as_uint(f), shift, mask) | base;
        if constexpr (kBytes == 4) return *(const lds_u32 *)a;
        else return *(const lds_u16 *)a;
    }
    // entry of a code of up to 31 bits that the table does not resolve: there is none
    __device__ inline uint32_t search(uint32_t, const BookDev *) const { return kLenSlow; }
};

// The same for alphabets of 9 to 12 bits, entries of four bytes with the symbol.  The full table would take 32 binades of
// up to 2048 entries, more than LDS has.  A code built from gradients needs fewer mantissa bits than the worst one (two to
// four fewer: its symbols come in groups of like weight), so the builder chooses them (BookWide::tab_bits, at most nine),
// and the binades below 2^12 are left out (one window in 2^20).  What the table does not resolve is found by a search of
// the lengths' limits, as costly as the former decoder was for every symbol.  A code whose symbols are all about as likely
// would need eleven bits; where a table by the first twelve bits of the window resolves more, it is that
// (prefixes; sixteen users of 4 M elements in [1,2,9], symbols all alike: averaged 231 us by the search, 75 by that table).
struct WideDecTable {
    static constexpr int kMaxRows = kRowsWide;
    uint32_t base, off, width;
    uint32_t limits;          // LDS address of the lengths' limits, 32 words
    bool prefixes;
    __device__ inline void init(uint32_t address, uint32_t bits, uint32_t limits_address)
    {
        limits = limits_address;
        prefixes = bits == 0;
        base = address - wide_table_first(bits) * 4u;
        off = wide_table_off(bits);
        width = here(wide_table_width(bits));   // (v_bfe_u32 takes one scalar operand)
    }
    __device__ inline uint32_t operator()(uint32_t u) const
    {
        const float f = (float)(u > kWideTabLeast ? u : kWideTabLeast);
        const uint32_t key = prefixes ? u : __float_as_uint(f);
        return *(const lds_u32 *)(__builtin_amdgcn_ubfe(key, off, width) * 4u + base);
    }
    __device__ inline uint32_t search(uint32_t u, const BookWide *__restrict__ book) const
    {
        uint32_t l = 0;   // the largest l whose codes, and shorter ones, lie below the window
#pragma unroll
        for (uint32_t k = 16; k; k >>= 1) l = u <= lds_word(limits + 4u * (l + k)) ? l + k : l;
        const uint32_t L = l + 1u;
        if (L > 31u) return kLenSlow;
        const uint32_t r = book->offset[L] + ((~u >> (32u - L)) - (uint32_t)book->first[L]);
        return ((uint32_t)book->sorted[r & (kWideMaxA - 1)] << 8) | L;
    }
};

// Loads that return zeros beyond `bytes`, without a branch.
__device__ inline __amdgpu_buffer_rsrc_t bounded(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}
__device__ inline u32x4 load16(__amdgpu_buffer_rsrc_t r, uint32_t byte) { return __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte, 0, 0); }

// A table of `bytes` (a multiple of 16) from device memory to LDS.
__device__ inline void load_table(uint32_t *dst, const void *src, uint32_t bytes, uint32_t thread, uint32_t nthreads)
{
    const __amdgpu_buffer_rsrc_t r = bounded(src, bytes);
    char *d = reinterpret_cast<char *>(dst);
    const uint32_t t = here(thread) * 16u, step = nthreads * 16u;
#pragma unroll 1
    for (uint32_t i = 0; i < bytes; i += 4u * step) {
        u32x4 v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = load16(r, t + i + k * step);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (t + i + k * step < bytes) *reinterpret_cast<u32x4 *>(d + t + i + k * step) = v[k];
    }
}

struct ChunkGeom {
    uint32_t seg;
    uint32_t n;       // elements in the chunk
    uint64_t e0;      // first element
    int32_t book;     // table id within a user's set
    bool scaled;      // a user of the layer carries a real-valued scale
};

__device__ inline ChunkGeom chunk_geom(const Layout &lay, uint64_t c)
{
    uint32_t lo = 0, hi = lay.nseg;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (lay.segs[mid].chunk_start <= c) lo = mid; else hi = mid;
    }
    ChunkGeom g;
    g.seg = lo;
    const SegDev sd = load_segment(lay.segs + lo);
    g.e0 = sd.offset + (c - sd.chunk_start) * kChunk;
    const uint64_t left = sd.offset + sd.length - g.e0;
    g.n = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
    g.book = sd.book;
    g.scaled = sd.scaled != 0;
    return g;
}


__device__ inline uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ inline uint64_t uniform(uint64_t x) { return ((uint64_t)uniform((uint32_t)(x >> 32)) << 32) | uniform((uint32_t)x); }

// The same in all lanes, said so: in the averages it spares spilled registers (k_aggregate_int<false> 6, k_aggregate_wide<2, false> 5 of
// 8; 24 users of 10^6 elements in [1,4,5] 32.6 -> 31.8 us); k_decode and k_decode_wide, which have none, lose 1 % by it.
__device__ inline ChunkGeom uniform(ChunkGeom g)
{
    g.e0 = uniform(g.e0);
    g.n = uniform(g.n);
    g.book = (int32_t)uniform((uint32_t)g.book);
    g.scaled = uniform(g.scaled ? 1u : 0u) != 0u;
    return g;
}

// What a wavefront needs to know about chunk c of user u before it can decode it.
struct ChunkIndex {
    const uint32_t *w;   // chunk's first word
    uint32_t nw;         // its words (0 if the index is malformed)
    uint32_t sb;         // this lane's sub-chunk bit count
    bool ok;             // 32-bit aligned, ordered, inside the buffer
};

// What read_index() asks for, requested a user ahead: between two users of a chunk stood two trips to memory, the index's
// and then the words', in which its wavefront issued nothing. The index is now on its way while the user before is decoded.
// The words' place is uniform and goes to scalar registers (one vector register more is held over the decoding, not five).
// The average of 4 x 1e8 values: 233.5 -> 228.2 us, of 8 x 4e7: 173.7 -> 170.8, of 10 x 11.7e6 with codes of a bit: 79.7 -> 77.7.
// The words' own lines asked for as well: 16 x 25.6e6 of 1+4+3 bits 205 -> 214 us, more registers than the sums leave.
struct IndexAhead {
    uint64_t off, end;
    uint32_t sb;
};
__device__ inline IndexAhead request_index(const Layout &lay, uint64_t c, uint32_t u, const uint64_t *__restrict__ chunk_offset,
                                           const uint16_t *__restrict__ sub_bits)
{
    IndexAhead a;
    typedef const __attribute__((address_space(4))) uint64_t *scalar_ptr;
    const scalar_ptr at = (scalar_ptr)(uintptr_t)(chunk_offset + (uint64_t)u * (lay.nchunks + 1) + c);
    a.off = at[0];
    a.end = at[1];
    a.sb = sub_bits[((uint64_t)u * lay.nchunks + c) * kSubsPerChunk + (threadIdx.x & 63)];
    return a;
}
__device__ inline ChunkIndex take_index(const IndexAhead &a, uint32_t u, const uint32_t *__restrict__ words, uint64_t words_stride)
{
    ChunkIndex ix;
    ix.sb = a.sb;
    ix.ok = !(a.off & 31u) && a.end >= a.off && (a.end >> 5) <= words_stride &&
            ((a.end - a.off) >> 5) <= (uint64_t)kChunk * CO3_MAX_CODE_LEN / 32;
    ix.nw = ix.ok ? (uint32_t)((a.end - a.off) >> 5) : 0u;
    ix.w = words + (uint64_t)u * words_stride + (ix.ok ? (a.off >> 5) : 0);
    return ix;
}

__device__ inline ChunkIndex read_index(const Layout &lay, uint64_t c, uint32_t u, const uint32_t *__restrict__ words,
                                        uint64_t words_stride, const uint64_t *__restrict__ chunk_offset,
                                        const uint16_t *__restrict__ sub_bits)
{
    ChunkIndex ix;
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t *at = chunk_offset + (uint64_t)u * (lay.nchunks + 1) + c;
    ix.sb = sub_bits[((uint64_t)u * lay.nchunks + c) * kSubsPerChunk + lane];
    const uint64_t off = uniform(at[0]), end = uniform(at[1]);
    ix.ok = !(off & 31u) && end >= off && (end >> 5) <= words_stride &&
            ((end - off) >> 5) <= (uint64_t)kChunk * CO3_MAX_CODE_LEN / 32;
    ix.nw = ix.ok ? (uint32_t)((end - off) >> 5) : 0u;
    ix.w = words + (uint64_t)u * words_stride + (ix.ok ? (off >> 5) : 0);
    return ix;
}

// A lane's place in its stream.
struct Stream {
    uint32_t N;       // bit address of the low end of the next 32 bits, counted in rows: LDS row N / 32, bit N % 32
    uint32_t first;   // word of the chunk that lies in the top row
    uint32_t end;     // bit of the chunk where the lane's sub-chunk ends
    uint32_t column;  // LDS address of the lane's column
    uint32_t row0, rows;   // the window's rows (the same in all lanes)
    int cnt;          // symbols to decode
    bool bad;         // a prefix matched no codeword
    __device__ inline uint32_t top() const { return 32u * (row0 + rows - 1u); }
    __device__ inline uint32_t bit() const { return 32u * first + (top() - N); }
    __device__ inline uint32_t word(uint32_t row) const { return lds_word(column + row * kRowBytes); }
    // the complements of 32 bits and of the 32 bits behind them
    __device__ inline uint32_t window(uint32_t n) const
    {
        const uint32_t r = n >> 5;
        return __builtin_amdgcn_alignbit(word(r + 1u), word(r), n);
    }
};

// Loads every lane's window from the word with its position on, 16 bytes a lane at a time (the lanes' pieces overlap or
// follow each other: the first request of a line serves the others from the cache), nothing beyond the chunk.
template <int kMaxRows>
__device__ inline void load_window(Stream &st, const ChunkIndex &ix, uint32_t bit)
{
    constexpr int n = kMaxRows / 4;
    st.first = bit >> 5;
    st.N = st.top() - (bit & 31u);
    const __amdgpu_buffer_rsrc_t r = bounded(ix.w, 4u * ix.nw);
    const uint32_t at = 4u * (st.first < ix.nw ? st.first : ix.nw);
    // pieces of four words: what the longest sub-chunk needs
    uint32_t pieces = 2;
#pragma unroll
    for (int k = 2; k < n; ++k) pieces += __any((st.first + 4u * (uint32_t)k) * 32u < st.end) ? 1u : 0u;
    pieces = pieces < st.rows / 4u ? pieces : st.rows / 4u;
    u32x4 v[n];
#pragma unroll
    for (int k = 0; k < n; ++k)
        if (k < 2 || (uint32_t)k < pieces) v[k] = load16(r, at + 16u * (uint32_t)k);
    // word 4 k + 3 - i lies i rows above the lowest of its piece
    const uint32_t low = st.column + (st.row0 + st.rows - 16u) * kRowBytes;
#pragma unroll
    for (int k = 0; k < n; ++k)
        if (k < 2 || (uint32_t)k < pieces) {
            const uint32_t at_row = k < 4 ? low + (uint32_t)(12 - 4 * k) * kRowBytes : low - (uint32_t)(4 * k - 12) * kRowBytes;
#pragma unroll
            for (int i = 0; i < 4; ++i) *(lds_u32 *)(at_row + (uint32_t)i * kRowBytes) = ~v[k][3 - i];
        }
    wave_lds_fence();
}

// Where some lane's sub-chunk does not fit its window: the windows are loaded anew unless every lane has the `bits` bits
// that a group reads at most, or all there is.
template <int kMaxRows>
__device__ inline void refill(Stream &st, const ChunkIndex &ix, uint32_t bits)
{
    const bool low = st.N < 32u * st.row0 + bits && 32u * (st.first + st.rows) < st.end;
    if (!__any(low)) return;
    wave_lds_fence();
    load_window<kMaxRows>(st, ix, st.bit());
}

// Symbols j0 .. j0 + 7, of which those from cnt on give the entry 0 and take no bits (full: cnt is kSub in every lane).
// Where bit 5, 6 or 7 of the result is set the lane's entries are not to be used: two symbols of 32 bits or more
// together, or a code the table does not hold.  n0: where the group started.
template <class Table>
__device__ inline uint32_t fast_group(Stream &st, uint32_t (&e)[kGroup], uint32_t &n0, int j0, const Table &tab, bool full)
{
    const uint32_t least = 32u * (st.row0 - 1u);   // (a damaged stream only)
    n0 = st.N > least ? st.N : least;
    uint32_t N = n0, over = 0;
#pragma unroll
    for (int b = 0; b < kGroup; b += 2) {
        const uint32_t u = st.window(N);
        const uint32_t x = tab(u);
        const uint32_t y = tab(u << (x & 31u));
        e[b] = x;
        e[b + 1] = y;
        const uint32_t both = x + y;   // bits 0..7: the two lengths, up to 64
        over |= both;
        N -= both & 0xffu;
    }
    if (!full) {
        N = n0;
#pragma unroll
        for (int b = 0; b < kGroup; ++b) {
            e[b] = j0 + b < st.cnt ? e[b] : 0u;
            N -= e[b] & 0xffu;
        }
        over = j0 < st.cnt ? over : 0u;
    }
    st.N = N;
    return over;
}

// The exact decoder, for the lanes `redo` of a group that started at n0: one window per symbol; a code the table does
// not hold is searched by all lanes together, lane l comparing the window with the codes of l + 1 bits.
template <class Table, class Book, class Value>
__device__ inline void slow_group(Stream &st, uint32_t (&e)[kGroup], uint32_t n0, bool redo, int j0, const Table &tab,
                                  const Book *__restrict__ book, Value value)
{
    const uint32_t lane = here(threadIdx.x & 63);
    st.N = redo ? n0 : st.N;
#pragma unroll 1
    for (int i = 0; i < kGroup; ++i) {
        const bool on = redo && j0 + i < st.cnt;
        const uint32_t least = 32u * (st.row0 - 1u);
        const uint32_t n = st.N > least ? st.N : least;
        const uint32_t u0 = st.window(n), u1 = st.window(n - 32u);
        uint32_t x = tab(u0);
        if (on && (x & 0xffu) == kLenSlow) x = tab.search(u0, book);
        uint64_t todo = __ballot(on && (x & 0xffu) == kLenSlow);
        while (todo) {
            const int src = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const uint64_t win = ~(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)u0, src) << 32) |
                                   (uint32_t)__builtin_amdgcn_readlane((int)u1, src));
            const uint64_t c = win >> (63u - lane), first = book->first[lane + 1u];
            const uint64_t hits = __ballot(c >= first && c - first < book->count[lane + 1u]);
            uint32_t y = 1u;   // nothing matches: one bit is passed over, as symbol 0
            if (hits) {
                const uint32_t L = (uint32_t)__ffsll((unsigned long long)hits);
                y = value(book->sorted[(book->offset[L] + (uint32_t)(win >> (64u - L)) - (uint32_t)book->first[L]) & ((uint32_t)(sizeof(book->sorted) / sizeof(book->sorted[0])) - 1u)]) | L;
            }
            if ((int)lane == src) {
                x = y;
                st.bad = st.bad || !hits;
            }
        }
        x = on ? x : 0u;
        st.N = on ? n - (x & 0xffu) : st.N;
        if (redo) {
#pragma unroll
            for (int b = 0; b + 1 < kGroup; ++b) e[b] = e[b + 1];
            e[kGroup - 1] = x;
        }
    }
}

// Where a wavefront decodes chunk (g, ix): `window` is the LDS address of its `rows` rows.  skip: bits of the lane's sub-chunk
// that are passed over.
template <int kMaxRows>
__device__ inline void start_chunk(Stream &st, const ChunkGeom &g, const ChunkIndex &ix, uint32_t window, uint32_t rows, uint32_t skip = 0)
{
    const uint32_t lane = threadIdx.x & 63;
    st.end = wave_inclusive_scan_dpp(ix.sb);
    st.row0 = window / kRowBytes;
    st.rows = rows;
    st.column = 4u * lane;
    const int left = (int)g.n - (int)lane * kSub;
    st.cnt = (int)here((uint32_t)(left < 0 ? 0 : (left > kSub ? kSub : left)));
    st.bad = false;
    load_window<kMaxRows>(st, ix, st.end - ix.sb + skip);
}
__device__ inline void finish_chunk(const Stream &st, const ChunkIndex &ix, uint64_t *__restrict__ status)
{
    if (!ix.ok || st.bad || st.bit() != st.end || (st.cnt > 0 && st.end > 32u * ix.nw))
        atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CORRUPT), 1ull);
    wave_lds_fence();   // the next chunk's words overwrite these
}

// on_group(gr, e) gets the entries of symbols 8 gr .. 8 gr + 7 of every lane, gr = 0 .. 7 (or from .. to - 1, where st stands
// before symbol 8 from).  kUnroll: gr is a constant there (sums in registers), at eight times the code, which a launch of few
// workgroups waits for.
template <bool kUnroll, class Table, class Book, class Value, class OnGroup>
__device__ inline void decode_started(Stream &st, const ChunkGeom &g, const ChunkIndex &ix, uint32_t A, const Table &tab,
                                      const Book *__restrict__ book, Value value, OnGroup on_group, int from = 0, int to = kGroups)
{
    const bool part = __any(32u * (st.first + st.rows) < st.end), full = g.n == (uint32_t)kChunk;
    auto group = [&](int gr) {
        uint32_t e[kGroup], n0;
        if (__builtin_expect(part, 0)) refill<Table::kMaxRows>(st, ix, group_bits(A));
        const uint32_t over = fast_group(st, e, n0, gr * kGroup, tab, full);
        const bool redo = (over & 0xe0u) != 0u;
        if (__builtin_expect(__any(redo), 0)) slow_group(st, e, n0, redo, gr * kGroup, tab, book, value);
        on_group(gr, e);
    };
    if constexpr (kUnroll) {
#pragma unroll
        for (int gr = 0; gr < kGroups; ++gr) group(gr);
    } else {
#pragma unroll 1
        for (int gr = from; gr < to; ++gr) group(gr);
    }
}

// ---- what becomes of the symbols ----

typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

// A symbol's value at exponent bias 127: its bits at their places in an fp32 pattern, so that the format's subnormals
// come out as fp32 ones, at their value.  Times 2^(127 - bias) it is the user's, exactly.
struct SymbolValue {
    uint32_t pattern, up, down;
    __device__ inline SymbolValue(int E, int M)
    {
        const uint32_t sign_shift = (uint32_t)(E + M);
        pattern = 0x80000000u | (((1u << sign_shift) - 1u) << (23 - M));
        up = 31u - sign_shift;
        down = 8u - (uint32_t)E;
    }
    // the symbol that lies `bit` bits up in a word (0, 8, 16, 24; of more than 8 bits: 0, 16)
    __device__ inline float operator()(uint32_t word, uint32_t bit) const
    {
        return __uint_as_float((uint32_t)((int32_t)(word << (up - bit)) >> down) & pattern);
    }
};

template <class Book>
struct AggArgsT {
    const uint32_t *words;
    uint64_t words_stride;
    const uint64_t *chunk_offset;
    const uint16_t *sub_bits;
    const Book *books;
    float *out;
    float *model;
    double eta;
    uint64_t *status;
};

// Four averages from sums, and with `model` the PS update w - eta * average (eq. (aggregate hat), Algorithm 1 line 14):
// products and difference in fp64, one rounding.  e: first of the four elements within the chunk; whole: so is the chunk.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));   // layers start anywhere: 16 bytes at any element
typedef u32x4 u32x4_u16 __attribute__((aligned(2)));
typedef u32x4 u32x4_u8 __attribute__((aligned(1)));
template <class Args>
__device__ inline void write_four(const ChunkGeom &g, const Args &a, uint32_t e, const double (&avg)[4], bool whole)
{
    if (whole) {
        if (a.out)
            *reinterpret_cast<f32x4_any *>(a.out + g.e0 + e) = f32x4{(float)avg[0], (float)avg[1], (float)avg[2], (float)avg[3]};
        if (a.model) {
            f32x4 w = *reinterpret_cast<const f32x4_any *>(a.model + g.e0 + e);
#pragma unroll
            for (int b = 0; b < 4; ++b) w[b] = (float)((double)w[b] - a.eta * avg[b]);
            *reinterpret_cast<f32x4_any *>(a.model + g.e0 + e) = w;
        }
    } else {
#pragma unroll
        for (uint32_t b = 0; b < 4; ++b) {
            if (e + b >= g.n) continue;
            if (a.out) a.out[g.e0 + e + b] = (float)avg[b];
            if (a.model) a.model[g.e0 + e + b] = (float)((double)a.model[g.e0 + e + b] - a.eta * avg[b]);
        }
    }
}

}  // namespace co3
