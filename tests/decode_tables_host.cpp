// The host's code builders and the decode tables' index rules of the library, for tests/test_decode_table_model.py: built for
// the CPU, the conversion to fp32 rounding toward zero as the decoders set it.
#include <cfenv>
#include <cstring>

#include "co3_internal.h"
#include "decode_core.h"

static uint32_t key_of(uint32_t u)
{
    const int mode = std::fegetround();
    std::fesetround(FE_TOWARDZERO);
    volatile uint32_t in = u;
    volatile float f = (float)in;
    std::fesetround(mode);
    const float g = f;
    uint32_t bits;
    std::memcpy(&bits, &g, 4);
    return bits;
}

extern "C" {

// Table of a byte alphabet: lengths and codes, and for every window complement u the entries of symbols and of values.
int byte_lookup(const uint64_t *weights, int E, int M, uint8_t *len, uint64_t *code, const uint32_t *u, uint64_t n, uint32_t *sym,
                uint32_t *val, int *values_filled)
{
    static co3::BookDev book;
    const uint32_t A = 1u << (1 + E + M);
    const int rc = co3::build_book_host(weights, A, E, M, &book);
    if (rc) return rc;
    std::memcpy(len, book.len, A);
    std::memcpy(code, book.code, A * sizeof(uint64_t));
    *values_filled = 0;
    for (uint32_t i = 0; i < co3::dec_table_entries(A); ++i) *values_filled += book.dval[i] != 0;
    const uint32_t shift2 = co3::byte_table_shift(A, 2), mask2 = co3::byte_table_mask(A, 2);
    const uint32_t shift4 = co3::byte_table_shift(A, 4), mask4 = co3::byte_table_mask(A, 4);
    for (uint64_t k = 0; k < n; ++k) {
        const uint32_t key = key_of(u[k]);
        sym[k] = book.dsym[co3::byte_table_at(key, shift2, mask2) / 2];
        val[k] = book.dval[co3::byte_table_at(key, shift4, mask4) / 4];
    }
    return 0;
}

uint32_t byte_value(uint32_t sym, int E, int M) { return co3::dec_value_bits(sym, E, M); }
uint32_t slow_entry() { return co3::kLenSlow; }

// The same of a wide alphabet; limit: the lengths' limits that the search uses.
int wide_lookup(const uint64_t *weights, uint32_t A, uint8_t *len, uint64_t *code, const uint32_t *u, uint64_t n, uint32_t *entry,
                uint32_t *limit, uint32_t *bits)
{
    static co3::BookWide book;
    const int rc = co3::build_wide_host(weights, A, &book);
    if (rc) return rc;
    std::memcpy(len, book.len, A);
    std::memcpy(code, book.code, A * sizeof(uint64_t));
    std::memcpy(limit, book.limit, sizeof(book.limit));
    *bits = book.tab_bits;
    const uint32_t off = co3::wide_table_off(*bits), width = co3::wide_table_width(*bits), first = co3::wide_table_first(*bits);
    for (uint64_t k = 0; k < n; ++k) {
        const uint32_t key = *bits ? key_of(u[k] > co3::kWideTabLeast ? u[k] : co3::kWideTabLeast) : u[k];
        entry[k] = book.tab[((key >> off) & ((1u << width) - 1u)) - first];
    }
    return 0;
}

}
