"""The decoder's table rule without a GPU: with u the complement of the next bits and k its leading zeros, the codeword at
the front of a complete canonical code has at most k + log2(A) bits, so that u's exponent and log2(A) - 1 bits behind its
leading one name it (codes of up to 31 bits, u of at least 4)."""
import numpy as np
import pytest

from oracle import co3_oracle as orc


def weights(kind, A, rng):
    if kind == "uniform":
        return np.ones(A)
    if kind == "steep":
        return np.floor(2.0 ** np.maximum(40 - np.arange(A) * 0.7, 0)) + 1
    if kind == "geometric":
        return np.floor(1e12 * 0.9 ** np.arange(A)) + 1
    if kind == "random":
        return rng.integers(1, 1 << 30, A)
    if kind == "few":
        w = np.zeros(A)
        w[rng.choice(A, 3, replace=False)] = [5, 1, 9]
        return w
    w = np.zeros(A)     # Fibonacci: the longest codes there are
    a, b = 1, 1
    for i in range(min(A, 60)):
        w[i] = a
        a, b = b, a + b
    return w


@pytest.mark.parametrize("nbits", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("kind", ["uniform", "steep", "geometric", "random", "few", "fibonacci"])
def test_leading_bits_name_the_code(nbits, kind):
    A = 1 << nbits
    rng = np.random.default_rng(nbits)
    lens = orc.huffman_lengths(weights(kind, A, rng).astype(np.uint64))
    codes = orc.canonical_codes(lens)
    half = A // 2
    table = {}
    for s in range(A):
        L = int(lens[s])
        if L == 0 or L > 31:
            continue
        c = int(codes[s])
        top = (1 << 32) - (c << (32 - L))            # complements of the windows with this code in front: (low, top]
        low = top - (1 << (32 - L))
        k = 32 - (top - 1).bit_length() if top > 1 else 32
        ones = c == (1 << L) - 1
        assert ones or L <= k + nbits
        for u in {low, top - 1, (low + top - 1) // 2, *(int(x) for x in rng.integers(low, top, 40))}:
            if u < 4:
                continue
            e = u.bit_length() - 1
            key = (e, (u >> (e - nbits + 1)) % half if e >= nbits - 1 else (u << (nbits - 1 - e)) % half)
            assert table.setdefault(key, s) == s, "two codes under one entry"
