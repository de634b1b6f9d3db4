// h_Hf: element-wise Huffman coding of the quantized symbols into one binary string per user
// (Sec. II-B (iii), Sec. IV-A (ii); Algorithm 1 line 9).  r, the length the paper's
// communication overhead counts, is the sum of the codeword lengths.
//
// Container: codewords in element order, MSB-first in 32-bit words.  A chunk (4096 elements,
// restarting at each layer) starts on a 32-bit boundary, so wavefronts own disjoint words of the
// output and no global atomics touch the stream.
//
// Coder for symbols stored by the quantize sweep.  Three steps:
//   k_chunk_bits   sum of the code lengths of every chunk: a wavefront per chunk, coalesced loads, a
//                  byte table of lengths in LDS (k_chunk_bits_hist: the same sums from the per-chunk symbol
//                  counts the quantize sweep writes for single-layer vectors, without touching the symbols)
//   k_scan_chunks  exclusive scan of the 32-bit-rounded chunk sizes (64-bit offsets), payload r; left out where a user has so
//                  few chunks that the coder's workgroups add the sizes up themselves
//   k_pack_chunk   four wavefronts per chunk, a thread a run of sixteen symbols: the codewords go to their place in the
//                  chunk's words in LDS (run_coder.h), which are then copied out coalesced; the sums over four threads are
//                  the sub-chunk index
#include "co3_internal.h"
#include "pack_core.h"
#include "run_coder.h"

namespace co3 {

constexpr int kPkWaves = 4;                         // wavefronts (chunks) per workgroup
constexpr int kPkThreads = 64 * kPkWaves;
constexpr int kSymLoads = (kChunk / 4 + 1 + 63) / 64;  // dword loads per lane to cover a chunk at any byte offset (17)

__device__ inline uint32_t wave_sum(uint32_t x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// Where chunk c of user u lies: first symbol byte (within the symbol buffer), element count, code table.
struct PkChunk {
    uint64_t byte0;
    uint64_t left;   // elements from there to the layer's end
    uint32_t n;
    uint32_t book;
    uint32_t seg;
};

__device__ inline PkChunk pk_layer_chunk(const Layout &lay, uint32_t seg, const SegDev &sd, uint64_t first, uint32_t u, uint64_t sym_stride)
{
    // the same in all lanes of a wavefront, and kept so: k_pack_chunk has no vector registers to spare
    auto scalar = [](uint64_t x) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32;
    };
    PkChunk k;
    k.byte0 = scalar((uint64_t)u * sym_stride + sd.offset + first);
    k.left = scalar(sd.length - first);
    k.n = k.left < (uint64_t)kChunk ? (uint32_t)k.left : (uint32_t)kChunk;
    k.book = (uint32_t)__builtin_amdgcn_readfirstlane((int)((lay.per_user_books ? u * lay.books_per_user : 0u) + (uint32_t)sd.book));
    k.seg = (uint32_t)__builtin_amdgcn_readfirstlane((int)seg);
    return k;
}

__device__ inline PkChunk pk_chunk(const Layout &lay, uint64_t c, uint32_t u, uint64_t sym_stride)
{
    const uint32_t seg = wave_find_chunk_segment(lay.segs, lay.nseg, c);
    const SegDev sd = load_segment(lay.segs + seg);
    return pk_layer_chunk(lay, seg, sd, (c - sd.chunk_start) * kChunk, u, sym_stride);
}

// The user's chunk behind k, of which there is one; only where k ends its layer is a layer's entry read.  (Searched for with every
// chunk, three loads that the next symbols' waited for: k_pack_chunk of ten users of 8 M elements in [1,3,0] in one layer 39 us,
// in three at odd elements 48; so 36.5 and 39.)
__device__ inline void pk_next_chunk(PkChunk &k, const Layout &lay, uint32_t u, uint64_t sym_stride)
{
    if (k.left > (uint64_t)kChunk) {
        k.byte0 += kChunk;
        k.left -= kChunk;
        k.n = k.left < (uint64_t)kChunk ? (uint32_t)k.left : (uint32_t)kChunk;
        return;
    }
    SegDev sd;
    uint32_t seg = k.seg;
    do sd = load_segment(lay.segs + ++seg); while (sd.length == 0);
    k = pk_layer_chunk(lay, seg, sd, 0, u, sym_stride);
}

// chunk_bits[u][c] = sum of the code lengths of the chunk's symbols (symbols without a code add nothing;
// they are counted where they are coded).  Lane l takes dwords l, l + 64, ... of the chunk's bytes.
__global__ __launch_bounds__(kPkThreads) void k_chunk_bits(Layout lay, const uint8_t *__restrict__ sym, uint64_t sym_stride,
                                                          const BookDev *__restrict__ books,
                                                          uint32_t *__restrict__ chunk_bits)
{
    __shared__ uint8_t s_len_all[kPkWaves][kMaxA];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t c = (uint64_t)blockIdx.x * kPkWaves + wave;
    const uint32_t u = blockIdx.y;
    if (c >= lay.nchunks) return;  // whole wavefront; no workgroup barriers below
    const PkChunk k = pk_chunk(lay, c, u, sym_stride);
    uint8_t *s_len = s_len_all[wave];
    const uint32_t len4 = reinterpret_cast<const uint32_t *>(books[k.book].len)[lane];
    const uint32_t shift = (uint32_t)(k.byte0 & 3u);
    const uint32_t *src = reinterpret_cast<const uint32_t *>(sym + (k.byte0 - shift));
    const uint32_t ndw = (shift + k.n + 3u) >> 2;
    uint32_t w[kSymLoads];
#pragma unroll
    for (int r = 0; r < kSymLoads; ++r) {
        const uint32_t i = lane + 64u * r;
        w[r] = i < ndw ? __builtin_nontemporal_load(src + i) : 0u;
    }
    reinterpret_cast<uint32_t *>(s_len)[lane] = len4;
    pc_wave_sync_lds();
    uint32_t total = 0;
    if (shift == 0 && k.n == (uint32_t)kChunk) {
#pragma unroll
        for (int r = 0; r < kChunk / 4 / 64; ++r)
#pragma unroll
            for (int b = 0; b < 4; ++b) total += s_len[(w[r] >> (8 * b)) & 0xffu];
    } else {
#pragma unroll
        for (int r = 0; r < kSymLoads; ++r) {
            const uint32_t i = lane + 64u * r;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t pos = 4u * i + b;                       // byte within the loaded dwords
                const bool in = pos >= shift && pos < shift + k.n;
                total += in ? s_len[(w[r] >> (8 * b)) & 0xffu] : 0u;
            }
        }
    }
    total = wave_sum(total);
    if (lane == 0) chunk_bits[(uint64_t)u * lay.nchunks + c] = total;
}

// The same sizes from the symbol counts of every chunk that the quantize sweep left behind (single-layer
// vectors): chunk_bits[u][c] = sum over symbols of count x code length.  A wavefront per chunk, four bins per lane.
__global__ __launch_bounds__(kPkThreads) void k_chunk_bits_hist(Layout lay, const uint16_t *__restrict__ chunk_hist,
                                                               const BookDev *__restrict__ books,
                                                               uint32_t *__restrict__ chunk_bits)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t c = (uint64_t)blockIdx.x * kPkWaves + wave;
    const uint32_t u = blockIdx.y;
    if (c >= lay.nchunks) return;
    const BookDev &book = books[(lay.per_user_books ? u * lay.books_per_user : 0u) + (uint32_t)lay.segs[0].book];
    const uint16_t *h = chunk_hist + ((uint64_t)u * lay.nchunks + c) * lay.A;
    uint32_t total = 0;
    for (uint32_t b0 = 4u * lane; b0 < lay.A; b0 += 256u) {   // A is a power of two, at least 8
        const uint2 cnt = *reinterpret_cast<const uint2 *>(h + b0);
        const uint32_t len4 = *reinterpret_cast<const uint32_t *>(book.len + b0);
        total += (cnt.x & 0xffffu) * (len4 & 0xffu) + (cnt.x >> 16) * ((len4 >> 8) & 0xffu) +
                 (cnt.y & 0xffffu) * ((len4 >> 16) & 0xffu) + (cnt.y >> 16) * (len4 >> 24);
    }
    total = wave_sum(total);
    if (lane == 0) chunk_bits[(uint64_t)u * lay.nchunks + c] = total;
}

// The coder proper.  chunk_offset comes from k_scan_chunks, or (kOffsets) every workgroup adds up the sizes of its user's chunks ahead
// of its own and writes its chunks' offsets, the last one the payload.  A workgroup takes `per_wg` consecutive chunks of a user, a team of four
// wavefronts on each in turn: a thread loads the 16 symbols of its run at once, at any byte, those of the next chunk before
// it codes these.  (A ragged chunk's last run is loaded whole as well: the symbols' buffer ends 16 bytes behind the last row.)  Two windows take turns; a thread clears the words that it has copied out.
// What bounds it: vector instructions, some 13 per symbol (17.5 where a lane coded 64 symbols into a row of its own and moved it).
// Sixteen users of 25.6 M elements in [1,4,3]: 229 -> 200 us.
template <bool kOffsets>
__global__ __launch_bounds__(kPkThreads, 8) void k_pack_chunk(
    Layout lay, const uint8_t *__restrict__ sym, uint64_t sym_stride, const BookDev *__restrict__ books,
    uint64_t *__restrict__ chunk_offset, uint16_t *__restrict__ sub_bits, uint32_t *__restrict__ words,
    uint64_t words_stride, uint64_t *__restrict__ status, uint32_t per_wg, const uint32_t *__restrict__ chunk_bits,
    uint64_t *__restrict__ payload_bits)
{
    __shared__ __align__(16) uint32_t s_win[2][kRunWindowStride];
    __shared__ uint32_t s_entry[kMaxA];
    __shared__ uint32_t s_part[2][kPkWaves];
    static_assert(kPkThreads == kMaxA && kPkThreads * kRun == kChunk, "an entry and a run for every thread");

    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t part = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t u = blockIdx.y;
    const uint64_t c0 = (uint64_t)blockIdx.x * per_wg;
    const uint32_t n = lay.nchunks - c0 < per_wg ? (uint32_t)(lay.nchunks - c0) : per_wg;
    uint64_t *offsets = chunk_offset + (uint64_t)u * (lay.nchunks + 1) + c0;
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef u4 u4_any __attribute__((aligned(1)));
    auto request = [&](const PkChunk &k) {
        return (uint32_t)kRun * t < k.n ? __builtin_nontemporal_load(reinterpret_cast<const u4_any *>(sym + k.byte0 + (uint32_t)kRun * t))
                                        : u4{0u, 0u, 0u, 0u};
    };
    PkChunk k = pk_chunk(lay, c0, u, sym_stride);
    u4 next = request(k);
    uint32_t tab = books[k.book].fast[t];
    for (uint32_t i = 4u * t; i < (uint32_t)kRunWindowStride; i += 4u * kPkThreads)
        *reinterpret_cast<u4 *>(&s_win[0][i]) = *reinterpret_cast<u4 *>(&s_win[1][i]) = u4{0u, 0u, 0u, 0u};
    uint32_t ahead = 0, payload = 0;   // (kOffsets) bits of the chunks before this one, rounded up to words each, and as they are
    if constexpr (kOffsets) {
        __shared__ uint32_t s_ahead[kPkWaves], s_payload[kPkWaves];
        const uint32_t *size = chunk_bits + (uint64_t)u * lay.nchunks;
        for (uint32_t i = t; i < (uint32_t)c0; i += kPkThreads) {
            ahead += (size[i] + 31u) & ~31u;
            payload += size[i];
        }
        ahead = wave_sum(ahead);
        payload = wave_sum(payload);
        if (lane == 0) {
            s_ahead[part] = ahead;
            s_payload[part] = payload;
        }
        __syncthreads();
        ahead = payload = 0;
#pragma unroll
        for (int j = 0; j < kPkWaves; ++j) {
            ahead += s_ahead[j];
            payload += s_payload[j];
        }
        ahead = (uint32_t)__builtin_amdgcn_readfirstlane((int)ahead);
        payload = (uint32_t)__builtin_amdgcn_readfirstlane((int)payload);
    }
    uint32_t book = ~0u;
    for (uint32_t i = 0; i < n; ++i) {
        const PkChunk cur = k;
        const BookDev &table = books[cur.book];
        if (cur.book != book) {   // the same in all threads
            if (i) {
                __syncthreads();   // the table before is done with
                tab = table.fast[t];
            }
            s_entry[t] = run_entry(tab);
            book = cur.book;
            __syncthreads();
        }
        TeamRun run;
#pragma unroll
        for (int j = 0; j < 4; ++j) run.w[j] = next[j];
        if (i + 1 < n) {
            pk_next_chunk(k, lay, u, sym_stride);
            next = request(k);
        }
        uint64_t off_words = 0;
        if constexpr (!kOffsets) off_words = offsets[i] >> 5;
        uint32_t head;
        team_lengths<false>(run, 64u * kRun * part, cur.n, cur.n == (uint32_t)kChunk, 0, s_entry, table, head, status);
        uint32_t *win = s_win[i & 1u], *share = s_part[i & 1u];
        if (lane == 0) share[part] = run.total;
        __syncthreads();
        uint32_t base = 0, bits = 0;
#pragma unroll
        for (uint32_t j = 0; j < (uint32_t)kPkWaves; ++j) {
            base += j < part ? share[j] : 0u;
            bits += share[j];
        }
        bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)bits);
        const uint32_t excl = base + run.excl, nwords = (bits + 31u) >> 5;
        if constexpr (kOffsets) {
            off_words = ahead >> 5;
            if (t == 0) offsets[i] = ahead;
            ahead += nwords << 5;
            payload += bits;
        }
        const uint32_t sub = quad_sum(run.bits);
        if ((lane & 3u) == 0) sub_bits[((uint64_t)u * lay.nchunks + c0 + i) * kSubsPerChunk + (t >> 2)] = (uint16_t)sub;
        const bool fits = off_words + nwords <= words_stride;
        if (!fits && t == 0) atomicAdd(reinterpret_cast<unsigned long long *>(status + CO3_STAT_CAPACITY), 1ull);
        uint32_t *dst = words + (uint64_t)u * words_stride + off_words;
        // window by window where the chunk's words are more than one holds
        for (uint32_t wbase = 0; wbase < nwords; wbase += kRunWindow) {
            if (wbase) __syncthreads();   // the window before is out
            // (a pair too long takes that way as well: singly from the entries, which the next symbols leave no registers for, 32 spill)
            if (run.wide || nwords > (uint32_t)kRunWindow) run_append_exact(run.w, 0, (int)run.to, s_entry, table, excl, win, wbase, kRunWindow);
            else if (run.bits) run_append<2>(run.e, excl, win);
            __syncthreads();
            const uint32_t left = nwords - wbase, wn = left < (uint32_t)kRunWindow ? left : (uint32_t)kRunWindow;
            for (uint32_t j = t; j < wn; j += kPkThreads) {
                if (fits) __builtin_nontemporal_store(win[j], dst + wbase + j);
                win[j] = 0u;
            }
        }
        if (t < 1) win[kRunWindow] = 0u;
    }
    if constexpr (kOffsets) {
        if (t == 0 && c0 + n == lay.nchunks) {
            offsets[n] = ahead;
            payload_bits[u] = payload;
        }
    }
}

// Exclusive scan of the chunks' sizes (rounded up to 32 bits) of one user; payload_bits = r.
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void k_scan_chunks(uint64_t nchunks, const uint32_t *__restrict__ chunk_bits,
                                                            uint64_t *__restrict__ chunk_offset,
                                                            uint64_t *__restrict__ payload_bits)
{
    __shared__ uint32_t s_wave[kScanThreads / 64];
    __shared__ uint32_t s_pay[kScanThreads / 64];
    const uint32_t u = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t *cb = chunk_bits + (uint64_t)u * nchunks;
    uint64_t *co = chunk_offset + (uint64_t)u * (nchunks + 1);
    uint64_t running = 0, payload = 0;
    for (uint64_t base = 0; base < nchunks; base += kScanThreads) {
        const uint64_t i = base + t;
        const uint32_t b = (i < nchunks) ? cb[i] : 0u;
        const uint32_t a = (b + 31u) & ~31u;
        const uint32_t incl_w = pc_wave_inclusive_scan(a, lane);
        const uint32_t pay = wave_sum(b);
        __syncthreads();  // previous iteration's reads of s_wave are done
        if (lane == 63) { s_wave[wave] = incl_w; s_pay[wave] = pay; }
        __syncthreads();
        uint32_t wave_base = 0, tot = 0, ptot = 0;
        for (uint32_t k = 0; k < kScanThreads / 64; ++k) {
            if (k < wave) wave_base += s_wave[k];
            tot += s_wave[k];
            ptot += s_pay[k];
        }
        if (i < nchunks) co[i] = running + wave_base + incl_w - a;
        running += tot;
        payload += ptot;
    }
    if (t == 0) { co[nchunks] = running; payload_bits[u] = payload; }
}

hipError_t launch_scan_chunks(const Layout &lay, const uint32_t *chunk_bits, uint64_t *chunk_offset,
                              uint64_t *payload_bits, hipStream_t s)
{
    if (lay.U == 0) return hipSuccess;
    ProfScope prof(K_SCAN, s);
    hipLaunchKernelGGL(k_scan_chunks, dim3(lay.U), dim3(kScanThreads), 0, s, lay.nchunks, chunk_bits, chunk_offset,
                       payload_bits);
    return hipGetLastError();
}

// One while the workgroups fit the device at a time; then several, whose symbols are requested ahead (k_pack_chunk of 256 chunks with
// one, two and four a workgroup 3.8, 5.1, 7.9 us; of 10 360 25.3, 22.4, 22.1; of 28 540 62, 57, 54; of 99 840 227, 203, 200; with
// eight 13.4, 25.4, 55, 203).
constexpr uint64_t kPkSums = 1024;
static uint32_t pack_chunks_per_workgroup(const Layout &lay)
{
    const uint64_t chunks = lay.nchunks * lay.U;
    return chunks >= 8192 ? 4 : (chunks >= 4096 ? 2 : 1);
}

hipError_t launch_pack(const Layout &lay, const co3_encode_args &a, const BookDev *books, const EncodeWs &ws,
                       hipStream_t s)
{
    if (lay.U == 0) return hipSuccess;
    const uint64_t sym_stride = symbol_row_stride(lay.d);
    const uint32_t gx = (uint32_t)((lay.nchunks + kPkWaves - 1) / kPkWaves);
    if (lay.nchunks) {
        ProfScope prof(K_CHUNK_BITS, s);
        if (ws.chunk_hist)
            hipLaunchKernelGGL(k_chunk_bits_hist, dim3(gx, lay.U), dim3(kPkThreads), 0, s, lay, ws.chunk_hist, books,
                               ws.chunk_bits);
        else
            hipLaunchKernelGGL(k_chunk_bits, dim3(gx, lay.U), dim3(kPkThreads), 0, s, lay, a.symbols, sym_stride, books,
                               ws.chunk_bits);
    }
    // Up to kPkSums chunks a user the coder's workgroups add up the sizes themselves: a launch less (one user of 256 chunks in [1,3,0], a
    // round 46.7 -> 41.0 us with the coder above; a workgroup's loads, four a thread at most, are answered while its symbols are on their way).
    const bool sums = lay.nchunks && lay.nchunks <= kPkSums;
    if (!sums && launch_scan_chunks(lay, ws.chunk_bits, a.chunk_offset, a.payload_bits, s) != hipSuccess) return hipGetLastError();
    if (lay.nchunks) {
        ProfScope prof(K_PACK, s);
        const uint32_t per_wg = pack_chunks_per_workgroup(lay);
        hipLaunchKernelGGL(sums ? k_pack_chunk<true> : k_pack_chunk<false>, dim3((uint32_t)((lay.nchunks + per_wg - 1) / per_wg), lay.U),
                           dim3(kPkThreads), 0, s, lay, a.symbols, sym_stride, books, a.chunk_offset, a.sub_bits, a.words, a.words_stride,
                           a.status, per_wg, ws.chunk_bits, a.payload_bits);
    }
    return hipGetLastError();
}

}  // namespace co3
