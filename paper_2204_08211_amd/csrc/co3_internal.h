// Internal declarations shared by the host API and the HIP kernels of libco3.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include "co3.h"

namespace co3 {

constexpr int kChunk = CO3_CHUNK;
constexpr int kSub = CO3_SUB;
constexpr int kSubsPerChunk = CO3_SUBS_PER_CHUNK;
constexpr int kMaxA = 256;          // alphabets of up to 8 bits: symbols are bytes
constexpr int kWideMaxA = 4096;     // alphabets of 9 to 12 bits: symbols are 16-bit words (k_wide.hip)
// Decode table of a wide alphabet (decode_core.h): binades 10 to 30 (binade 10 stands for all below and holds nothing) of
// up to 2^9 entries, 42 KB of the 160 that a CU's wavefronts share.
constexpr uint32_t kWideTabLow = 10, kWideTabBinades = 21;
__host__ __device__ constexpr uint32_t wide_tab_bits_max(uint32_t A) { return A > 512u ? 9u : 8u; }
constexpr uint32_t kWideTabMax = kWideTabBinades << 9;
constexpr uint32_t kWidePrefixBits = 12;   // of a code for which a table by prefixes resolves more
__host__ __device__ constexpr uint32_t wide_tab_entries(uint32_t bits) { return bits ? kWideTabBinades << bits : 1u << kWidePrefixBits; }
// Decode tables of byte alphabets (decode_core.h): 32 binades of A / 2 entries.
constexpr uint32_t kDecTableMax = 16 * kMaxA;
__host__ __device__ constexpr uint32_t dec_table_entries(uint32_t A) { return 16u * A; }
__host__ __device__ constexpr uint32_t dec_format(int E, int M) { return ((uint32_t)E << 8) | (uint32_t)M; }
constexpr uint32_t kLenSlow = 32;   // an entry's length field: none of the codes of up to 31 bits
// Symbols between two users' rows of a symbol buffer: the row length rounded up to 128 symbols, so that rows
// start on 128-byte lines (of a 256-byte-aligned buffer).
inline uint64_t symbol_row_stride(uint64_t d) { return (d + 127) & ~(uint64_t)127; }

constexpr int kHistGlobalRep = 64;   // copies of the global symbol-count table the workgroups spread over
constexpr int kFastLen = 24;        // longest code held in the 32-bit encode entry
constexpr uint32_t kFastSlow = 0xFFu;  // length field marking "use the 64-bit table"

constexpr uint32_t kWFastCodeBits = 25;   // longest code held in a wide alphabet's encode entry ...
constexpr uint32_t kWFastSlow = 127;      // ... and the length field of the others

// One Huffman code table as the kernels read it.
struct BookDev {
    uint64_t code[kMaxA];        // right-aligned codeword of each symbol
    uint64_t first[65];          // first[L]: first canonical code of length L (L = 1..64)
    uint32_t fast[kMaxA];        // (len << 24) | code for len <= 24; len field 0xFF: a longer code, or none
    uint32_t count[65];          // count[L]: symbols with length L
    uint32_t offset[65];         // offset[L]: index of the first length-L symbol in sorted[]
    uint8_t len[kMaxA];          // codeword length, 0 = no code
    uint8_t sorted[kMaxA];       // symbols ordered by (length, symbol)
    uint32_t maxlen;
    uint32_t nactive;
    uint32_t format;             // (E << 8) | M that dval[] was filled for (dec_value_is_int(E), else it is not)
    // Decode tables over the complement u of the next 32 bits: entry i serves the u whose leading bits, as a floating
    // point number of log2(A) - 1 mantissa bits, are i = (exponent mod 32) * A / 2 + mantissa.
    // (symbol << 8) | length, and (what the PS sums (dec_value_bits) | length); kLenSlow: no code of up to 31 bits
    alignas(16) uint16_t dsym[kDecTableMax];
    alignas(16) uint32_t dval[kDecTableMax];
};

// One Huffman code table of a wide alphabet (9 to 12 symbol bits) as the wide kernels read it.
struct BookWide {
    uint64_t code[kWideMaxA];             // right-aligned codeword of each symbol
    uint64_t first[65];                   // first[L]: first canonical code of length L
    uint32_t count[65];                   // symbols with length L
    uint32_t offset[65];                  // index of the first length-L symbol in sorted[]
    uint16_t sorted[kWideMaxA];           // symbols ordered by (length, symbol)
    uint8_t len[kWideMaxA];               // codeword length, 0 = no code
    alignas(16) uint32_t fast[kWideMaxA]; // (len << kWFastCodeBits) | code; length field kWFastSlow: a longer code, or none
    uint32_t maxlen;
    uint32_t nactive;
    uint32_t tab_bits;                    // mantissa bits of the decode table's index; 0: indexed by the complement's top 12 bits
    uint32_t limit[32];                   // a window's complement <= limit[l] (and not 0): its code has more than l bits
    // (symbol << 8) | length, kLenSlow: a code the table does not resolve; entry i belongs to binade kWideTabLow + i >> tab_bits
    alignas(16) uint32_t tab[kWideTabMax];
};

// One layer of the flat vector as the kernels read it.
struct SegDev {
    uint64_t offset;       // first element
    uint64_t length;
    uint64_t chunk_start;  // index of the segment's first chunk within a user
    int32_t book;          // code table id within a user's (or the shared) set
    int32_t scaled;        // whether a user's real-valued scale of the layer is not 1 (launch_mark_scaled)
};

// How the wide coder (k_wide.hip) cuts a user's chunks into workgroups: at every change of the code table, and after
// kWgChunks (or kWgChunksSmall) chunks.  A run is a longest stretch of chunks under one table.
struct RunDev {
    uint64_t chunk_start;             // its first chunk
    uint32_t wg_start, wg_small_start;   // its first workgroup of up to kWgChunks, of up to kWgChunksSmall chunks
    int32_t book;                     // code table id within a user's (or the shared) set
    uint32_t seg;                     // its first layer
};
struct WideCut {
    const RunDev *runs;               // device [nrun + 1] (last entry: chunk_start = nchunks, seg = nseg)
    uint32_t nrun;
    uint32_t nwg, nwg_small;          // workgroups per user
};
constexpr uint32_t kWgChunks = 16, kWgChunksSmall = 4;

// Constants of Q_fp for one (format, bias), derived on the device from E, M and bias.
struct Layout {
    uint32_t U;
    uint32_t nseg;
    uint64_t d;
    uint64_t nchunks;          // per user
    int32_t E, M;
    uint32_t A;
    uint32_t books_per_user;   // 1 + max segment.codebook
    uint32_t per_user_books;
    uint32_t nbooks;           // tables in a set
    uint32_t wide;             // alphabet above 8 bits: 16-bit symbols, the kernels of k_wide.hip
    uint32_t vec_aligned;      // every layer starts at a multiple of 4 elements (16-byte vectors never straddle a layer start)
    uint32_t tile_aligned;     // every layer starts at a multiple of 2048 elements (a tile of the wide quantizer lies in one chunk)
    const SegDev *segs;        // device [nseg + 1] (last entry: offset = d, chunk_start = nchunks)
    const int32_t *bias;       // device [U][nseg]
    const float *gain;         // device [U][nseg][2]: (gain, inv_gain) of the real-valued scale; (1, 1) when unused
};
// Every kernel takes a Layout and looks its layers up, so what one kernel needs alone stays out of both: at 40 and 96
// bytes, with the wide coder's cut in them, sixteen users' round of 25.6 M elements took 1347 instead of 1336 us, the
// wide average of the same size 941 instead of 909 us.
static_assert(sizeof(SegDev) == 32 && sizeof(Layout) == 88, "read by every kernel");

// A layer's entry, requested as a whole; left to itself the compiler requests its parts where they are used (three users of
// 11.3 M elements in eleven layers in [1,5,6], the former wide decoder: 187 -> 183 us).
__device__ inline SegDev load_segment(const SegDev *p)
{
    typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));
    const u64x4 e = *reinterpret_cast<const u64x4 *>(p);   // entries of 32 bytes from a 256-byte boundary on
    SegDev sd;
    sd.offset = e[0];
    sd.length = e[1];
    sd.chunk_start = e[2];
    sd.book = (int32_t)(uint32_t)e[3];
    sd.scaled = (int32_t)(uint32_t)(e[3] >> 32);
    return sd;
}

}  // namespace co3

namespace co3 {
// What the host knows of a plan beside its layout.  It chooses between kernels by that, for speed only: a captured launch may
// be replayed when it is out of date, so every kernel looks at the device's tables.
struct PlanFacts {
    bool has_gain = false;     // a gain other than (1, 1) was installed
    int32_t bias_spread = 0;   // how far the users' biases of a layer lie apart at most; 0 where they came from device memory
};
}  // namespace co3

struct co3_plan {
    co3::Layout lay;
    co3::SegDev *d_segs = nullptr;
    co3::RunDev *d_runs = nullptr;   // wide alphabets only: wide.runs
    co3::WideCut wide = {};
    int32_t *d_bias = nullptr;
    float *d_gain = nullptr;
    co3::PlanFacts facts;
    int device = 0;
};

struct co3_codebook {
    co3_format format;
    uint32_t nbooks = 0;
    uint32_t A = 0;
    co3::BookDev *d_books = nullptr;    // byte alphabets
    co3::BookWide *d_wide = nullptr;    // wide alphabets (exactly one of the two is set)
    int device = 0;
};

namespace co3 {

// Per-kernel event timing (profile.cpp).  A ProfScope around a launch records two events on
// the stream when profiling is on, and does nothing otherwise.
enum KernelId { K_ZERO = 0, K_QUANTIZE, K_REDUCE_HIST, K_BUILD_BOOKS, K_CHUNK_BITS, K_SCAN, K_PACK, K_DECODE, K_AGGREGATE, K_FUSED, K_MOMENTS, K_FIT, K_MODEL_WEIGHTS, K_MODEL_BIAS, K_COUNT };
bool profile_enabled();
class ProfScope {
public:
    ProfScope(int kid, hipStream_t s);
    ~ProfScope();
private:
    int kid_;
    hipStream_t s_;
    hipEvent_t start_;
};

// Host Huffman builder (host_codebook.cpp): fills one table; returns a co3_status.
int build_book_host(const uint64_t *weights, uint32_t A, int E, int M, BookDev *out);
int build_wide_host(const uint64_t *weights, uint32_t A, BookWide *out);


// Kernel launchers (one per .hip file).  All return a hipError_t from hipGetLastError().
struct EncodeWs {
    uint64_t *hist_rep;     // [kHistGlobalRep][nbooks][A] partial symbol counts
    uint32_t *chunk_bits;   // [U][nchunks] payload bits of every chunk
    uint16_t *chunk_hist;   // [U][nchunks][A] symbol counts of every chunk, or nullptr (single-layer vectors only)
};
// bytes of the three-step encoder's workspace: what it cannot do without, and what it takes when it gets it (the
// per-chunk symbol counts spare it a sweep over the symbols)
size_t three_step_workspace_min(const Layout &lay);
size_t three_step_workspace_full(const Layout &lay);
EncodeWs three_step_workspace(const Layout &lay, void *workspace, size_t bytes);

hipError_t launch_zero_u64(uint64_t *p, uint64_t n, hipStream_t s);
hipError_t launch_reduce_hist(const uint64_t *hist_rep, uint64_t *hist, uint64_t n, hipStream_t s);   // hist[i] = sum of the partial tables
hipError_t launch_quantize(const Layout &lay, const co3_encode_args &a, const EncodeWs &ws, hipStream_t s);
hipError_t launch_build_books(BookDev *books, uint32_t nbooks, int E, int M, const uint64_t *weights, uint64_t *counts,
                              uint64_t *status, hipStream_t s);
hipError_t launch_pack(const Layout &lay, const co3_encode_args &a, const BookDev *books,
                       const EncodeWs &ws, hipStream_t s);
// exclusive scan of the 32-bit-rounded chunk sizes of every user (k_pack.hip), shared with the wide path
hipError_t launch_scan_chunks(const Layout &lay, const uint32_t *chunk_bits, uint64_t *chunk_offset,
                              uint64_t *payload_bits, hipStream_t s);
// single-sweep encoder for a fixed code (k_fused.hip); its workspace need in bytes
hipError_t launch_encode_fused(const Layout &lay, const co3_encode_args &a, const BookDev *books, hipStream_t s);
size_t fused_workspace_bytes(const Layout &lay);
// GenNorm fit and model weights (k_fit.hip); partial: fit_workspace_bytes() of device memory
size_t fit_workspace_bytes(const Layout &lay);
hipError_t launch_fit(const Layout &lay, const float *g, const float *m, uint64_t row_stride, float gamma,
                      co3_gennorm_params *params, double *partial, hipStream_t s);
hipError_t launch_model_weights(const Layout &lay, const co3_gennorm_params *params, uint64_t *weights,
                                hipStream_t s);
size_t bias_workspace_bytes(const Layout &lay);
hipError_t launch_model_bias(const Layout &lay, const co3_gennorm_params *params, int32_t *bias, double *error,
                             double *errors_ws, hipStream_t s);
size_t scale_workspace_bytes(const Layout &lay);
hipError_t launch_model_scale(const Layout &lay, const co3_gennorm_params *params, int32_t *bias, float *gain_pairs,
                              double *error, double *workspace, hipStream_t s);
hipError_t launch_decode(const Layout &lay, const co3_decode_args &a, const BookDev *books, hipStream_t s);
// says in every layer's entry whether the plan's gain table has a scale for it
hipError_t launch_mark_scaled(const Layout &lay, SegDev *segs, hipStream_t s);
hipError_t launch_aggregate(const Layout &lay, const PlanFacts &facts, const co3_aggregate_args &a, const BookDev *books,
                            hipStream_t s);
// wide alphabets (k_wide.hip): the same steps with 16-bit symbols and tables in device memory
size_t wide_workspace_bytes(const Layout &lay);
hipError_t launch_encode_wide(const Layout &lay, const WideCut &cut, const co3_encode_args &a, BookWide *books, void *workspace,
                              hipStream_t s);
hipError_t launch_build_books_wide(BookWide *books, uint32_t nbooks, uint32_t A, const uint64_t *weights,
                                   uint64_t *status, hipStream_t s);
hipError_t launch_decode_wide(const Layout &lay, const co3_decode_args &a, const BookWide *books, hipStream_t s);
hipError_t launch_aggregate_wide(const Layout &lay, const co3_aggregate_args &a, const BookWide *books,
                                 hipStream_t s);

}  // namespace co3
