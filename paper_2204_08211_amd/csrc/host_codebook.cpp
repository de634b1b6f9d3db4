// Host construction of one Huffman code table (Sec. IV-A (ii): element-wise Huffman coding of
// the quantized gradient; optimal for a known source, Sec. II-E).
//
// Tie rule: nodes are ordered by (weight, key); a leaf's key is its symbol, an internal node's
// key is A + its creation order; the two smallest are merged.  With the leaves sorted once by
// (weight, symbol) and the internal nodes kept in creation order (their weights never
// decrease), the smallest node is always at the head of one of the two lists, and on equal
// weight the leaf comes first because every leaf key is below every internal key.
#include <algorithm>
#include <cstring>
#include <vector>

#include "co3_internal.h"
#include "quantize_math.h"

namespace co3 {

// Fill every derived table of `b` from b->len[] (lengths) for alphabet size A.
static void finish_tables(BookDev *b, uint32_t A, int E, int M)
{
    std::memset(b->count, 0, sizeof(b->count));
    std::memset(b->first, 0, sizeof(b->first));
    std::memset(b->offset, 0, sizeof(b->offset));
    std::memset(b->code, 0, sizeof(b->code));
    for (uint32_t s = 0; s < (uint32_t)kMaxA; ++s) b->fast[s] = kFastSlow << 24;  // no code: the coders' general path counts it
    std::memset(b->sorted, 0, sizeof(b->sorted));
    b->maxlen = 0;
    b->nactive = 0;
    for (uint32_t s = 0; s < A; ++s) {
        if (!b->len[s]) continue;
        b->count[b->len[s]]++;
        b->nactive++;
        if (b->len[s] > b->maxlen) b->maxlen = b->len[s];
    }
    // canonical codes: first[L] = (first[L-1] + count[L-1]) << 1
    uint64_t code = 0;
    uint32_t off = 0;
    for (int L = 1; L <= 64; ++L) {
        code = (code + b->count[L - 1]) << 1;
        b->first[L] = code;
        b->offset[L] = off;
        off += b->count[L];
    }
    uint32_t next[65];
    std::memset(next, 0, sizeof(next));
    for (uint32_t s = 0; s < A; ++s) {  // ascending symbol within each length
        const int L = b->len[s];
        if (!L) continue;
        const uint32_t rank = next[L]++;
        b->code[s] = b->first[L] + rank;
        b->sorted[b->offset[L] + rank] = (uint8_t)s;
        if (L <= kFastLen) b->fast[s] = ((uint32_t)L << 24) | (uint32_t)b->code[s];
        else b->fast[s] = kFastSlow << 24;
    }
    // decode tables: entry i belongs to the windows whose complement u has exponent i / (A / 2) mod 32 and, behind its
    // leading one, the bits i mod (A / 2); a code of up to 31 bits covers whole entries
    const uint32_t half = A / 2;
    int nm = 0;
    while ((1u << nm) < half) ++nm;
    b->format = dec_format(E, M);
    for (uint32_t i = 0; i < dec_table_entries(A); ++i) {
        const uint32_t binade = i / half;
        const int ex = binade == 31 ? 0 : (int)binade + 1;   // exponent of u
        const uint64_t lead = (uint64_t)(half + i % half);   // leading one and mantissa
        const uint32_t x = ~(uint32_t)(ex >= nm ? lead << (ex - nm) : lead >> (nm - ex));
        uint32_t len = kLenSlow, sym = 0;
        for (int L = 1; binade != 0 && L <= 31; ++L) {
            const uint64_t c = x >> (32 - L);
            if (c < b->first[L] || c - b->first[L] >= b->count[L]) continue;
            len = (uint32_t)L;
            sym = b->sorted[b->offset[L] + (uint32_t)(c - b->first[L])];
            break;
        }
        b->dsym[i] = (uint16_t)((sym << 8) | len);
        if (dec_value_is_int(E)) b->dval[i] = dec_value_bits(sym, E, M) | len;
    }
}

// Huffman code lengths by the two-queue merge (leaves sorted by (weight, symbol), internal nodes in creation
// order, leaves first on equal weight); len must hold A zeros.
static int huffman_lengths_host(const uint64_t *w, uint32_t A, uint8_t *len)
{
    struct Leaf { uint64_t w; uint32_t s; };
    std::vector<Leaf> leaves;
    uint64_t total = 0;
    for (uint32_t s = 0; s < A; ++s) {
        if (!w[s]) continue;
        if (total + w[s] < total || total + w[s] == ~0ull) return CO3_ERR_ARG;
        total += w[s];
        leaves.push_back({w[s], s});
    }
    const int n = (int)leaves.size();
    if (n == 0) return CO3_OK;
    if (n == 1) { len[leaves[0].s] = 1; return CO3_OK; }
    std::sort(leaves.begin(), leaves.end(),
              [](const Leaf &x, const Leaf &y) { return x.w != y.w ? x.w < y.w : x.s < y.s; });
    std::vector<uint64_t> nw(2 * n - 1);
    std::vector<int> parent(2 * n - 1, -1);
    for (int i = 0; i < n; ++i) nw[i] = leaves[i].w;
    int li = 0, ii = n, made = n;
    for (int step = 0; step < n - 1; ++step) {
        int pick[2];
        for (int r = 0; r < 2; ++r) {
            const bool have_leaf = li < n, have_int = ii < made;
            if (have_leaf && (!have_int || nw[li] <= nw[ii])) pick[r] = li++;
            else pick[r] = ii++;
        }
        nw[made] = nw[pick[0]] + nw[pick[1]];
        parent[pick[0]] = made;
        parent[pick[1]] = made;
        ++made;
    }
    for (int i = 0; i < n; ++i) {
        int depth = 0;
        for (int p = parent[i]; p >= 0; p = parent[p]) ++depth;
        if (depth > CO3_MAX_CODE_LEN) return CO3_ERR_CODELEN;
        len[leaves[i].s] = (uint8_t)depth;
    }
    return CO3_OK;
}

// The decode table of `b` from its lengths, codes and order.
static void finish_wide_table(BookWide *b, uint32_t A)
{
    // mantissa bits: what the codes with up to ten leading ones need
    uint32_t nm = 2;
    for (uint32_t s = 0; s < A; ++s) {
        const uint32_t L = b->len[s];
        if (!L) continue;
        uint32_t k = 0;
        while (k < L && ((b->code[s] >> (L - 1 - k)) & 1u)) ++k;
        if (k <= 10 && k < L && L - k - 1 > nm) nm = L - k - 1;
    }
    if (nm > wide_tab_bits_max(A)) nm = wide_tab_bits_max(A);
    uint64_t end[33];   // codes of up to l bits lie below end[l], left-aligned in 32 bits
    end[0] = 0;
    for (int l = 1; l <= 32; ++l) end[l] = (b->first[l] + b->count[l]) << (32 - l);
    for (int l = 0; l < 32; ++l) b->limit[l] = end[l] >> 32 ? 0u : 0xffffffffu - (uint32_t)end[l];
    uint64_t missing = 0;   // share of the code space the table leaves to the search, in 2^-32
    auto entry = [&](uint32_t x, uint32_t longest) {   // window, longest code that covers the entry
        uint32_t L = 1;
        while (L < 32 && (uint64_t)x >= end[L]) ++L;
        if (L > 31 || L > longest) return kLenSlow;
        return ((uint32_t)b->sorted[b->offset[L] + ((x >> (32 - L)) - (uint32_t)b->first[L])] << 8) | L;
    };
    b->tab_bits = nm;
    std::fill(b->tab, b->tab + kWideTabMax, kLenSlow);
    for (uint32_t i = 1u << nm; i < wide_tab_entries(nm); ++i) {
        const uint32_t ex = kWideTabLow + (i >> nm) + 1;   // exponent of the window's complement
        b->tab[i] = entry(~(uint32_t)((uint64_t)((1u << nm) | (i & ((1u << nm) - 1u))) << (ex - nm)), 32 - ex + nm);
        if (b->tab[i] == kLenSlow) missing += 1ull << (ex - nm);
    }
    // (the device's builder has the rule and why fewer bits never meet it)
    if (nm == wide_tab_bits_max(A) && missing > (1ull << 32) - end[kWidePrefixBits]) {
        b->tab_bits = 0;
        std::fill(b->tab, b->tab + kWideTabMax, kLenSlow);
        for (uint32_t i = 0; i < wide_tab_entries(0); ++i) b->tab[i] = entry(~(i << (32 - kWidePrefixBits)), kWidePrefixBits);
    }
}

int build_wide_host(const uint64_t *w, uint32_t A, BookWide *b)
{
    std::memset(b, 0, sizeof(*b));
    std::fill(b->fast, b->fast + kWideMaxA, kWFastSlow << kWFastCodeBits);
    int rc = huffman_lengths_host(w, A, b->len);
    if (rc != CO3_OK) { std::memset(b, 0, sizeof(*b)); return rc; }
    for (uint32_t s = 0; s < A; ++s) {
        if (!b->len[s]) continue;
        b->count[b->len[s]]++;
        b->nactive++;
        if (b->len[s] > b->maxlen) b->maxlen = b->len[s];
    }
    uint64_t code = 0;
    uint32_t off = 0;
    for (int L = 1; L <= 64; ++L) {   // canonical codes: first[L] = (first[L-1] + count[L-1]) << 1
        code = (code + b->count[L - 1]) << 1;
        b->first[L] = code;
        b->offset[L] = off;
        off += b->count[L];
    }
    uint32_t next[65];
    std::memset(next, 0, sizeof(next));
    for (uint32_t s = 0; s < A; ++s) {  // ascending symbol within each length
        const int L = b->len[s];
        if (!L) continue;
        const uint32_t rank = next[L]++;
        b->code[s] = b->first[L] + rank;
        if ((uint32_t)L <= kWFastCodeBits) b->fast[s] = ((uint32_t)L << kWFastCodeBits) | (uint32_t)b->code[s];
        b->sorted[b->offset[L] + rank] = (uint16_t)s;
    }
    finish_wide_table(b, A);
    return CO3_OK;
}

int build_book_host(const uint64_t *w, uint32_t A, int E, int M, BookDev *b)
{
    std::memset(b, 0, sizeof(*b));
    struct Leaf { uint64_t w; uint32_t s; };
    std::vector<Leaf> leaves;
    uint64_t total = 0;
    for (uint32_t s = 0; s < A; ++s) {
        if (!w[s]) continue;
        if (total + w[s] < total || total + w[s] == ~0ull) return CO3_ERR_ARG;
        total += w[s];
        leaves.push_back({w[s], s});
    }
    const int n = (int)leaves.size();
    if (n == 0) { finish_tables(b, A, E, M); return CO3_OK; }
    if (n == 1) { b->len[leaves[0].s] = 1; finish_tables(b, A, E, M); return CO3_OK; }
    std::sort(leaves.begin(), leaves.end(),
              [](const Leaf &x, const Leaf &y) { return x.w != y.w ? x.w < y.w : x.s < y.s; });
    // nodes 0..n-1: sorted leaves; n..2n-2: internal nodes in creation order
    std::vector<uint64_t> nw(2 * n - 1);
    std::vector<int> parent(2 * n - 1, -1);
    for (int i = 0; i < n; ++i) nw[i] = leaves[i].w;
    int li = 0, ii = n, made = n;
    for (int step = 0; step < n - 1; ++step) {
        int pick[2];
        for (int r = 0; r < 2; ++r) {
            const bool have_leaf = li < n, have_int = ii < made;
            if (have_leaf && (!have_int || nw[li] <= nw[ii])) pick[r] = li++;
            else pick[r] = ii++;
        }
        nw[made] = nw[pick[0]] + nw[pick[1]];
        parent[pick[0]] = made;
        parent[pick[1]] = made;
        ++made;
    }
    for (int i = 0; i < n; ++i) {
        int depth = 0;
        for (int p = parent[i]; p >= 0; p = parent[p]) ++depth;
        if (depth > CO3_MAX_CODE_LEN) return CO3_ERR_CODELEN;
        b->len[leaves[i].s] = (uint8_t)depth;
    }
    finish_tables(b, A, E, M);
    return CO3_OK;
}

}  // namespace co3
