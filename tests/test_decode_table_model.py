"""The decode tables without a GPU: the library's host builders and the index rules of decode_core.h, compiled for the CPU,
against a canonical decode of the oracle's codes.  With u the complement of the next bits and k its leading zeros, the codeword
at the front of a complete canonical code has at most k + log2(A) bits, so that u's exponent and log2(A) - 1 bits behind its
leading one name it (codes of up to 31 bits, u of at least 4)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from oracle import co3_oracle as orc
from paper_2204_08211_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = tmp_path_factory.mktemp("tables") / "tables.so"
    flags = [f for f in hip_build.FLAGS if not f.startswith("--offload-arch")]
    flags = [f for k, f in enumerate(flags) if f not in ("-Xclang", "-target-feature", "-packed-fp32-ops")]
    subprocess.run([hip_build.HIPCC, "-x", "hip", "--cuda-host-only", "-shared", os.path.join(HERE, "decode_tables_host.cpp"),
                    os.path.join(hip_build.CSRC, "host_codebook.cpp"), "-o", str(so)] + flags, check=True)
    return C.CDLL(str(so))


def weights(kind, A, rng):
    if kind == "uniform":
        return np.ones(A)
    if kind == "steep":
        return np.floor(2.0 ** np.maximum(40 - np.arange(A) * 0.7, 0)) + 1
    if kind == "geometric":
        return np.floor(1e12 * 0.9 ** np.arange(A)) + 1
    if kind == "random":
        return rng.integers(1, 1 << 30, A)
    if kind == "tail":       # a few short words, then many of 18 bits and more
        return np.concatenate([2.0 ** np.arange(58, 58 - min(18, A // 2), -1), np.full(A - min(18, A // 2), 2.0 ** 33)])
    w = np.zeros(A)
    if kind == "few":
        w[rng.choice(A, 3, replace=False)] = [5, 1, 9]
    elif kind == "one":
        w[rng.integers(A)] = 7
    elif kind == "short":    # words of up to twelve bits, some of more than ten ones
        n = min(A, 4)
        w[:n] = [1 << 20, 1 << 19, 1 << 18, 1 << 18][:n]
        w[n:min(A, 64)] = 256
    else:                    # Fibonacci: the longest codes there are
        a, b = 1, 1
        for i in range(min(A, 60)):
            w[i] = a
            a, b = b, a + b
    return w


KINDS = ["uniform", "steep", "geometric", "random", "tail", "few", "one", "short", "fibonacci"]


def windows(lens, codes, rng):
    """Complements of windows: both ends of every code's, the bits behind every code shifted to the front, at random in every
    binade, and all near the binades' ends."""
    x = []
    for s in np.flatnonzero(lens):
        L, c = int(lens[s]), int(codes[s])
        if L <= 31:
            lo = c << (32 - L)
            x += [lo, lo + (1 << (32 - L)) - 1, lo | int(rng.integers(1 << (32 - L)))]
        else:
            x.append(c >> (L - 32))
    u = [0xffffffff - v for v in x]
    u += [(v << int(lens[s])) & 0xffffffff for v, s in zip(u, rng.choice(np.flatnonzero(lens), len(u)))]
    for k in range(32):
        top = 1 << k
        u += [top, top | (top - 1), top | 1] + list(top + rng.integers(0, top, 200))
    return np.array(u + [0], np.uint64).astype(np.uint32)


def canonical(u, lens, codes):
    """Symbol and length of the word of up to 31 bits at the front of each window (length 0: none)."""
    x = (~u).astype(np.uint64)
    sym = np.zeros(u.size, np.int64)
    length = np.zeros(u.size, np.int64)
    for L in range(1, 32):
        at = np.flatnonzero(lens == L)
        if at.size:
            first = int(codes[at].min())
            c = (x >> np.uint64(32 - L)).astype(np.int64) - first
            hit = (length == 0) & (c >= 0) & (c < at.size)
            sym[hit] = at[c[hit]]
            length[hit] = L
    return sym, length


def ptr(a):
    return a.ctypes.data_as(C.c_void_p)


@pytest.mark.parametrize("E,M", [(2, 0), (2, 1), (3, 1), (4, 1), (3, 3), (4, 3), (5, 1), (5, 2), (6, 1)])
@pytest.mark.parametrize("kind", KINDS)
def test_byte_tables(host, E, M, kind):
    A = 1 << (1 + E + M)
    rng = np.random.default_rng(A + len(kind))
    w = np.ascontiguousarray(weights(kind, A, rng).astype(np.uint64))
    lens = orc.huffman_lengths(w)
    codes = orc.canonical_codes(lens)
    u = windows(lens, codes, rng)
    sym, val = np.zeros(u.size, np.uint32), np.zeros(u.size, np.uint32)
    got_len, got_code, filled = np.zeros(A, np.uint8), np.zeros(A, np.uint64), C.c_int(0)
    assert host.byte_lookup(ptr(w), E, M, ptr(got_len), ptr(got_code), ptr(u), C.c_uint64(u.size), ptr(sym), ptr(val), C.byref(filled)) == 0
    assert np.array_equal(got_len, lens) and np.array_equal(got_code[lens > 0], np.asarray(codes, np.uint64)[lens > 0])
    want, length = canonical(u, lens, codes)
    slow = host.slow_entry()
    named = (length > 0) & (u >= 4)
    assert np.array_equal(sym[named], (want[named] << 8) | length[named])
    # the others are slow, but for the windows of less than 4 that a short word of ones covers
    assert np.all((sym[~named] == slow) | (length[~named] > 0))
    if E <= 4:       # the formats with integer sums
        v = np.array([host.byte_value(C.c_uint32(s), E, M) & 0xffffffff for s in range(A)], np.uint32)
        assert np.array_equal(val[named], v[want[named]] | length[named].astype(np.uint32))
        value = np.array([orc.value(s, E, M, 0) for s in range(A)], np.float64) * 2.0 ** (M - 1)
        emit = ((np.arange(A) & (A // 2 - 1)) < orc.num_magnitudes(E, M)) & (np.arange(A) != A // 2)   # (no negative zero)
        assert np.array_equal(v.view(np.int32)[emit] >> 8, value[emit].astype(np.int64))
    else:
        assert filled.value == 0


@pytest.mark.parametrize("nbits", [9, 10, 11, 12])
@pytest.mark.parametrize("kind", KINDS)
def test_wide_tables(host, nbits, kind):
    A = 1 << nbits
    rng = np.random.default_rng(A + len(kind))
    w = np.ascontiguousarray(weights(kind, A, rng).astype(np.uint64))
    lens = orc.huffman_lengths(w)
    codes = orc.canonical_codes(lens)
    u = windows(lens, codes, rng)
    entry, limit, bits = np.zeros(u.size, np.uint32), np.zeros(32, np.uint32), C.c_uint32(0)
    got_len, got_code = np.zeros(A, np.uint8), np.zeros(A, np.uint64)
    assert host.wide_lookup(ptr(w), C.c_uint32(A), ptr(got_len), ptr(got_code), ptr(u), C.c_uint64(u.size), ptr(entry), ptr(limit), C.byref(bits)) == 0
    assert np.array_equal(got_len, lens)
    want, length = canonical(u, lens, codes)
    slow = host.slow_entry()
    resolved = entry != slow
    assert np.array_equal(entry[resolved], (want[resolved] << 8) | length[resolved])
    # what the table leaves is found by the limits: a code's length is one more than the limits that u does not exceed
    left = ~resolved & (length > 0) & (u > 0)
    found = 1 + np.sum(u[left, None] <= limit[None, 1:], axis=1)
    assert np.array_equal(found, length[left])
    # where the mantissa bits suffice the table by binades is taken, and it leaves no code with up to ten leading ones
    need = 2
    for s in np.flatnonzero(lens):
        L = int(lens[s])
        ones = len(bin((int(codes[s]) ^ ((1 << L) - 1)) | (1 << L))[3:].split("1")[0])
        if ones <= 10 and ones < L:
            need = max(need, L - ones - 1)
    most = 9 if A > 512 else 8
    if need < most:
        assert bits.value == need
        assert np.all(resolved[(u >= 1 << 21) & (length > 0)])
