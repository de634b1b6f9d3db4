"""The decoder's windows and tables and the averages' sums at the places where they change, against the oracle."""
import numpy as np
import pytest

import gpu_util as gu
from oracle import co3_oracle as orc

pytestmark = pytest.mark.gpu
BOOK_FIXED, BOOK_EMPIRICAL = 0, 1


def on_grid(rng, E, M, bias, d, p=None):
    """Gradients that are representatives of the users' grids, magnitudes drawn with probabilities p."""
    g = np.empty((len(bias), d), np.float32)
    for u, b in enumerate(bias):
        grid = orc.grid(E, M, int(b))
        g[u] = (grid[rng.choice(grid.size, d, p=p)] * rng.choice([-1.0, 1.0], d)).astype(np.float32)
    return g


@pytest.mark.parametrize("E,M", [(2, 0), (2, 1), (3, 1), (3, 2), (3, 3), (4, 3), (5, 2), (4, 4), (5, 5), (4, 7)])
@pytest.mark.parametrize("U", [1, 3])
def test_sub_chunks_longer_than_a_window(E, M, U):
    # a held code that gives the frequent symbols its long words: a sub-chunk takes up to several windows, some lanes'
    # do and others' do not, in whole chunks and in a ragged one
    rng = np.random.default_rng(100 * E + M)
    d = 2 * 4096 + 1000
    bias = np.full((U, 1), 2 ** (E - 1) - 1 + 6, np.int32)
    nm = orc.num_magnitudes(E, M)
    p = 0.55 ** np.minimum(np.arange(nm)[::-1], 60)
    g = on_grid(rng, E, M, bias[:, 0], d, p / p.sum())
    g[:, 4096:4096 + 64 * 20] = 0.0             # twenty lanes with the shortest word only
    m = np.zeros_like(g)
    A = 1 << (1 + E + M)
    w = np.zeros(A, np.uint64)
    emit = [0] + [s for s in range(A) if 0 < (s & (A // 2 - 1)) < nm]
    order = sorted(emit, key=lambda s: s & (A // 2 - 1))
    w[order] = [max(1, int(2.0 ** (45 - 45.0 * i / len(order)))) for i in range(len(order))]
    kw = dict(E=E, M=M, U=U, d=d, bias=bias)
    gpu, _ = gu.gpu_round(kw, g, m, 0.9, BOOK_FIXED, weights=w[None, :], max_code_len=64)
    ref = gu.oracle_round(kw, g, m, 0.9, weights=w[None, :])
    rows = {3: 8, 4: 12, 5: 12}.get(1 + E + M, 20 if E + M < 8 else 24)
    if (E, M) != (2, 0):
        assert ref["sub_bits"].max() > 32 * rows
    assert ref["sub_bits"].min() < 32 * rows
    gu.compare_round(gpu, ref, d)


@pytest.mark.parametrize("U", [2, 4, 5, 8, 11, 34])
@pytest.mark.parametrize("spread", [0, 9, 12, 13, 60])
@pytest.mark.parametrize("own", [False, True])
def test_average_over_users_whose_biases_lie_apart(U, spread, own):
    # integer sums per wavefront and workgroup, fp64 sums where they would not fit, more users than one turn holds;
    # with a few chunks (a wavefront per user) and a plan that learns its biases on the device
    import torch
    from paper_2204_08211_amd import binding as B
    E, M, d = 4, 3, 4096 + 333
    rng = np.random.default_rng(1000 * U + spread)
    bias = (10 + rng.integers(0, spread + 1, (U, 1))).astype(np.int32)
    bias[0], bias[-1] = 10, 10 + spread
    g = np.concatenate([rng.standard_normal((1, d)) * orc.grid(E, M, int(b))[-1] / 3 for b in bias[:, 0]]).astype(np.float32)
    m = np.zeros_like(g)
    kw = dict(E=E, M=M, U=U, d=d, bias=bias, per_user_books=own)
    gpu, (plan, books, buf, _, _) = gu.gpu_round(kw, g, m, 0.9, BOOK_EMPIRICAL)
    ref = gu.oracle_round(kw, g, m, 0.9)
    # beyond 53 bits the last one may depend on the order of the users
    gu.compare_round(gpu, ref, d, avg_exact=spread < 30)
    same = torch.from_numpy(bias).to("cuda:0")
    plan_near = B.Plan(E, M, U, d, np.full((U, 1), 10, np.int32), per_user_books=own)   # as the host knows it: no spread
    B._check("co3_plan_set_bias_device", B.lib().co3_plan_set_bias_device(plan_near.handle, same.data_ptr(), B._stream()))
    again = torch.zeros(d, dtype=torch.float32, device="cuda:0")
    B.co3_ps_aggregate(plan_near, books, buf, again)
    torch.cuda.synchronize()
    if spread < 30:
        gu.assert_bits_equal(again.cpu().numpy(), ref["avg"], "average, biases set on the device")
    else:
        scale = np.maximum(np.abs(ref["avg"]), np.abs(ref["dec_q"]).mean(axis=0))
        assert np.all(np.abs(again.cpu().numpy().astype(np.float64) - ref["avg"]) <= 1e-6 * scale)


@pytest.mark.parametrize("chunks", [520, 1100])
@pytest.mark.parametrize("U,E,M", [(3, 4, 3), (4, 5, 2), (7, 3, 2), (13, 2, 1)])
def test_average_on_both_sides_of_the_wavefronts_rule(chunks, U, E, M):
    # a wavefront per user, several users a wavefront, a wavefront per chunk; layers of different tables that start and
    # end inside a workgroup's chunks, the average at any element
    rng = np.random.default_rng(chunks + U)
    seg_len = [4096 * 3 + 17, 0, 5, 4096 * (chunks - 9), 4096 * 4 + 1]
    d = sum(seg_len)
    bias = rng.integers(14, 18, (U, len(seg_len))).astype(np.int32)
    sym_top = np.float32(orc.grid(E, M, 16)[-1])
    g = (rng.standard_normal((U, d)) * sym_top / 4).astype(np.float32)
    m = np.zeros_like(g)
    kw = dict(E=E, M=M, U=U, d=d, bias=bias, seg_len=seg_len, seg_book=[0, 1, 1, 2, 0])
    gpu, _ = gu.gpu_round(kw, g, m, 0.9, BOOK_EMPIRICAL)
    check_against_own_symbols(gpu, U, E, M, seg_len, bias)


def test_table_set_of_another_format_of_the_same_alphabet():
    # a code names symbols, not values: a set made for [1,5,2] serves a plan in [1,4,3]
    import torch
    from paper_2204_08211_amd import binding as B
    E, M, U, d = 4, 3, 3, 9000
    rng = np.random.default_rng(5)
    bias = np.array([[12], [14], [13]], np.int32)
    g = (rng.standard_normal((U, d)) * 2.0).astype(np.float32)
    m = np.zeros_like(g)
    kw = dict(E=E, M=M, U=U, d=d, bias=bias)
    w = gu.oracle_round(kw, g, m, 0.9)["hist"]
    ref = gu.oracle_round(kw, g, m, 0.9, weights=w)
    gpu, _ = gu.gpu_round(kw, g, m, 0.9, BOOK_FIXED, weights=w, books=B.co3_build_codebook(5, 2, 1, w))
    gu.compare_round(gpu, ref, d)


def check_against_own_symbols(gpu, U, E, M, seg_len, bias):
    """The decoded symbols are the coded ones, the average is the oracle's of them."""
    d = sum(seg_len)
    vals = np.zeros(d)
    off = 0
    for k, n in enumerate(seg_len):
        for u in range(U):
            lut = np.array([orc.value(s, E, M, int(bias[u, k])) for s in range(1 << (1 + E + M))], np.float64)
            vals[off:off + n] += lut[gpu["sym"][u, off:off + n]]
        off += n
    gu.assert_bits_equal(gpu["dec_sym"], gpu["sym"], "decoded symbols")
    gu.assert_bits_equal(gpu["avg"], (vals * (1.0 / U)).astype(np.float32), "average")
    assert int(gpu["status"][5]) == 0


@pytest.mark.parametrize("U,E,M,seg_len,own", [
    (4, 4, 5, [4096 * 2100 + 77], False),                          # several sets of chunks a workgroup
    (4, 5, 4, [4096 * 900 + 5, 7, 4096 * 1203 + 1, 4096], False),  # and tables that change between and within them
    (3, 4, 4, [4096 * 1190 + 3, 4096 * 12], True),                 # a table per user, shared by a workgroup's wavefronts
    (2, 5, 6, [4096 * 1201], True),
    (7, 4, 5, [4096 * 30 + 9], True),                              # and two wavefronts with a table each, in turns
    (1, 4, 5, [4096 * 5], True),
    (35, 3, 6, [4096 * 2 + 11], False),                            # more users than a turn takes
])
def test_wide_sets_splits_and_tables(U, E, M, seg_len, own):
    rng = np.random.default_rng(U + E)
    d = sum(seg_len)
    bias = rng.integers(2 ** (E - 1), 2 ** (E - 1) + 3, (U, len(seg_len))).astype(np.int32)
    g = (rng.standard_normal((U, d)) * np.float32(orc.grid(E, M, int(bias.max()))[-1]) / 4).astype(np.float32)
    kw = dict(E=E, M=M, U=U, d=d, bias=bias, seg_len=seg_len, seg_book=list(range(len(seg_len))), per_user_books=own)
    gpu, _ = gu.gpu_round(kw, g, np.zeros_like(g), 0.9, BOOK_EMPIRICAL)
    check_against_own_symbols(gpu, U, E, M, seg_len, bias)


@pytest.mark.parametrize("E,M", [(4, 4), (4, 5), (5, 5), (4, 7), (5, 6)])
@pytest.mark.parametrize("kind", ["alike", "one", "two", "steep"])
def test_wide_codes_the_table_does_not_resolve(E, M, kind):
    # codes whose symbols are all about as likely need more mantissa bits than the table has (they are searched for), codes
    # of one and two symbols fewer than any, a steep one has words of more than 31 bits; host's and device's tables
    import torch
    from paper_2204_08211_amd import binding as B
    rng = np.random.default_rng(E * 16 + M)
    U, d, b = 3, 4096 + 900, 2 ** (E - 1)
    A, nm = 1 << (1 + E + M), orc.num_magnitudes(E, M)
    emit = np.array([0] + [s for s in range(A) if 0 < (s & (A // 2 - 1)) < nm])
    w = np.zeros(A, np.uint64)
    if kind == "alike":
        w[emit] = rng.integers(1000, 1003, emit.size)
        mags = np.arange(nm)
    elif kind == "steep":
        w[emit] = [max(1, int(2.0 ** (50 - 0.5 * (int(s) & (A // 2 - 1)) / max(1, nm // 256)))) for s in emit]
        mags = np.concatenate([np.arange(nm // 2), np.arange(nm)])
    else:
        mags = np.array([0] if kind == "one" else [0, 3])
        w[0] = 7
        if kind == "two":
            w[[3, 3 + A // 2]] = [4, 2]
    grid = orc.grid(E, M, b)
    g = (grid[rng.choice(mags, (U, d))] * rng.choice([-1.0, 1.0], (U, d))).astype(np.float32)
    m = np.zeros_like(g)
    bias = np.full((U, 1), b, np.int32)
    kw = dict(E=E, M=M, U=U, d=d, bias=bias)
    ref = gu.oracle_round(kw, g, m, 0.9, weights=w[None, :])
    books = B.co3_build_codebook(E, M, 1, None)
    status = torch.zeros(B.STATUS_WORDS, dtype=torch.int64, device="cuda:0")
    B.co3_build_codebook_device(books, torch.from_numpy(w.view(np.int64)).to("cuda:0"), status)
    for made in (None, books):
        gpu, _ = gu.gpu_round(kw, g, m, 0.9, BOOK_FIXED, weights=w[None, :], max_code_len=64, books=made)
        gu.compare_round(gpu, ref, d)


@pytest.mark.parametrize("U", [2, 3, 8, 9, 16, 17])
@pytest.mark.parametrize("gain", [False, True])
@pytest.mark.parametrize("own", [False, True])
def test_average_whose_users_meet_in_lds(U, gain, own):
    # formats without integer sums, and plans with a scale: a user per wavefront, two, and one more than meet in LDS; whole,
    # shifted and ragged chunks.  The fp64 sums in the users' order of the values that co3_decode gives, rounded once.
    import torch
    from paper_2204_08211_amd import binding as B
    E, M, seg_len = 5, 2, [4096 + 77, 5, 2 * 4096]
    d, nseg = sum(seg_len), len(seg_len)
    rng = np.random.default_rng(7000 + U)
    bias = rng.integers(20, 29, (U, nseg)).astype(np.int32)
    plan = B.Plan(E=E, M=M, U=U, d=d, bias=bias, seg_len=seg_len, seg_book=[0, 1, 0], per_user_books=own)
    if gain:
        inv = (2.0 ** rng.uniform(-0.5, 0.5, (U, nseg))).astype(np.float32)
        plan.set_gain((np.float32(1.0) / inv).astype(np.float32), inv)
    dev = torch.device("cuda:0")
    stride = (d + 3) // 4 * 4
    g = torch.zeros((U, stride), dtype=torch.float32, device=dev)
    g[:, :d] = torch.from_numpy((rng.laplace(size=(U, d)) * 1e-3).astype(np.float32)).to(dev)
    m = torch.zeros_like(g)
    books = B.co3_build_codebook(E, M, plan.num_books, None)
    buf = B.RoundBuffers(plan, dev, max_code_len=32)
    buf.status.zero_()
    B.co3_encode(plan, books, g, m, m, 0.9, buf, mode=BOOK_EMPIRICAL)
    q = torch.zeros((U, stride), dtype=torch.float32, device=dev)
    B.co3_decode(plan, books, buf, q=q)
    out = torch.full((d,), float("nan"), dtype=torch.float32, device=dev)
    model = torch.from_numpy(rng.standard_normal(d).astype(np.float32)).to(dev)
    before = model.cpu().numpy().astype(np.float64)
    B.co3_ps_aggregate(plan, books, buf, out, model=model, eta=0.25)
    torch.cuda.synchronize()
    assert not buf.status.cpu().numpy().any()
    total = np.zeros(d)
    for row in q[:, :d].cpu().numpy().astype(np.float64):
        total += row
    mean = total * (1.0 / U)
    if U <= 16 or not gain:      # (scaled values are no exact sums; beyond 16 users their order is not defined)
        gu.assert_bits_equal(out.cpu().numpy(), mean.astype(np.float32), "average")
        gu.assert_bits_equal(model.cpu().numpy(), (before - 0.25 * mean).astype(np.float32), "model")
    else:
        size = np.abs(q[:, :d].cpu().numpy()).mean(axis=0)
        assert np.all(np.abs(out.cpu().numpy() - mean) <= 2.0 ** -23 * np.maximum(np.abs(mean), 2.0 ** -20 * size))


@pytest.mark.parametrize("E,M", [(5, 2), (5, 1), (4, 3)])
@pytest.mark.parametrize("U", [1, 3, 8, 13, 17, 40])
@pytest.mark.parametrize("own", [False, True])
def test_average_with_a_scale_and_words_of_25_to_31_bits(E, M, U, own):
    # a held code with twenty words of one to twenty bits and many of 25 bits and more, which differ in the low byte of the
    # window's leading bits; most elements have one of those.  With a scale: a wavefront per chunk, the users' symbols
    # meeting in LDS, a turn and several turns of four a wavefront.  The average of the values that co3_decode gives.
    import torch
    from paper_2204_08211_amd import binding as B
    rng = np.random.default_rng(900 + 10 * E + U)
    A, nm, b0 = 1 << (1 + E + M), orc.num_magnitudes(E, M), 2 ** (E - 1) + 3
    seg_len = [4096 + 77, 5, 2 * 4096]
    d, nseg = sum(seg_len), len(seg_len)
    emit = np.array([0] + [s for s in range(A) if 0 < (s & (A // 2 - 1)) < nm])
    order = rng.permutation(emit)
    w = np.zeros(A, np.uint64)
    w[order[:18]] = [1 << (58 - i) for i in range(18)]
    rest = order[18:]
    w[rest] = [(1 << 33) >> (3 * (i * 3 // rest.size)) for i in range(rest.size)]    # three groups of equal weights
    lens = orc.huffman_lengths(w)
    assert ((lens >= 25) & (lens <= 31)).sum() > 20
    plan = B.Plan(E=E, M=M, U=U, d=d, bias=np.full((U, nseg), b0, np.int32), seg_len=seg_len, seg_book=[0, 1, 0], per_user_books=own)
    # (above sixteen users the order of the sums is not defined: powers of two, so that they are exact)
    inv = (2.0 ** (rng.uniform(-0.5, 0.5, (U, nseg)) if U <= 16 else rng.integers(-1, 2, (U, nseg)))).astype(np.float32)
    gain = (np.float32(1.0) / inv).astype(np.float32)
    plan.set_gain(gain, inv)
    grid = orc.grid(E, M, b0).astype(np.float64)
    p = np.where(rng.random((U, d)) < 0.8, rng.choice(rest, (U, d)), rng.choice(emit, (U, d)))
    v = grid[p & (A // 2 - 1)] * np.where(p >= A // 2, -1.0, 1.0) * np.repeat(inv.astype(np.float64), seg_len, axis=1)
    dev = torch.device("cuda:0")
    stride = (d + 3) // 4 * 4
    g = torch.zeros((U, stride), dtype=torch.float32, device=dev)
    g[:, :d] = torch.from_numpy(v.astype(np.float32)).to(dev)
    m = torch.zeros_like(g)
    books = B.co3_build_codebook(E, M, plan.num_books, np.tile(w, (plan.num_books, 1)))
    buf = B.RoundBuffers(plan, dev, max_code_len=64)
    B.co3_encode(plan, books, g, m, m, 0.9, buf, mode=BOOK_FIXED)
    sym = torch.zeros(plan.symbols_bytes, dtype=torch.uint8, device=dev)
    q = torch.zeros((U, stride), dtype=torch.float32, device=dev)
    B.co3_decode(plan, books, buf, symbols=sym, q=q)
    out = torch.full((d,), float("nan"), dtype=torch.float32, device=dev)
    B.co3_ps_aggregate(plan, books, buf, out)
    torch.cuda.synchronize()
    assert not buf.status.cpu().numpy()[2:].any()      # (a top value times its scale may be clamped by a rounding)
    gu.assert_bits_equal(gu._sym_numpy(B.symbols_2d(plan, sym)), gu._sym_numpy(buf.symbols_2d()), "decoded symbols")
    assert np.mean(lens[gu._sym_numpy(buf.symbols_2d())] >= 25) > 0.5
    total = np.zeros(d)
    for row in q[:, :d].cpu().numpy().astype(np.float64):
        total += row
    gu.assert_bits_equal(out.cpu().numpy(), (total * (1.0 / U)).astype(np.float32), "average")


def device_bias(plan, bias):
    import torch
    from paper_2204_08211_amd import binding as B
    t = torch.from_numpy(np.ascontiguousarray(bias, np.int32)).to("cuda:0")
    B._check("co3_plan_set_bias_device", B.lib().co3_plan_set_bias_device(plan.handle, t.data_ptr(), B._stream()))
    torch.cuda.synchronize()


def coded(E, M, g, bias, own=False, seg_len=None, max_code_len=40):
    """A round's streams of given gradients under a plan that knows the biases (memory zero)."""
    import torch
    from paper_2204_08211_amd import binding as B
    U, d = g.shape
    plan = B.Plan(E, M, U, d, bias, seg_len=seg_len, per_user_books=own)
    books = B.co3_build_codebook(E, M, plan.num_books, None)
    buf = B.RoundBuffers(plan, "cuda:0", max_code_len=max_code_len)
    gt = torch.zeros((U, (d + 3) // 4 * 4), dtype=torch.float32, device="cuda:0")
    gt[:, :d] = torch.from_numpy(g).to("cuda:0") if isinstance(g, np.ndarray) else g
    m = torch.zeros_like(gt)
    B.co3_encode(plan, books, gt, m, m, 0.0, buf, mode=BOOK_EMPIRICAL)
    return plan, books, buf


def in_order_average(plan, books, buf):
    import torch
    from paper_2204_08211_amd import binding as B
    q = torch.zeros((plan.U, (plan.d + 3) // 4 * 4), dtype=torch.float32, device="cuda:0")
    B.co3_decode(plan, books, buf, q=q)
    total = torch.zeros(plan.d, dtype=torch.float64, device="cuda:0")
    for u in range(plan.U):
        total += q[u, :plan.d].double()
    return (total * (1.0 / plan.U)).float().cpu().numpy()


def cancelling(U, d, bias, top, seed):
    """Gradients whose sums depend on the order: users 0 and 2 cancel but for a few elements, 1 and 3 are far below them."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    g = torch.randn((U, d), generator=gen, device="cuda:0") * (top / 4)
    g[2] = torch.where(torch.rand(d, generator=gen, device="cuda:0") < 0.9, -g[0], g[2])
    scale = torch.tensor([2.0 ** (int(bias[0, 0]) - int(b)) for b in bias[:, 0]], device="cuda:0")
    return (g * scale[:, None]).float()


@pytest.mark.parametrize("U", [3, 4])
@pytest.mark.parametrize("E,M,chunks", [(4, 3, 5), (4, 3, 1500), (2, 1, 1500), (4, 3, 2100)])
def test_few_users_keep_their_order(U, E, M, chunks):
    # biases from the device so far apart that fp64 sums depend on the order: the users', with a wavefront each, two for the
    # chunk (whose symbols meet in LDS, or do not fit there), one
    import torch
    from paper_2204_08211_amd import binding as B
    d = 4096 * chunks + 100
    bias = np.array([[10], [66], [10], [64]], np.int32)[:U]
    plan, books, buf = coded(E, M, cancelling(U, d, bias, float(orc.grid(E, M, 10)[-1]), U + chunks), bias)
    want = in_order_average(plan, books, buf)
    near = B.Plan(E, M, U, d, np.full((U, 1), 10, np.int32))
    device_bias(near, bias)
    out = torch.zeros(d, dtype=torch.float32, device="cuda:0")
    B.co3_ps_aggregate(near, books, buf, out)
    torch.cuda.synchronize()
    assert not buf.status.cpu().numpy()[2:].any()
    gu.assert_bits_equal(out.cpu().numpy(), want, "average")


@pytest.mark.parametrize("E,M,U,chunks,own", [(4, 3, 1, 3, False), (4, 3, 3, 2, True), (4, 3, 11, 2, False), (4, 3, 40, 2, False),
                                              (4, 3, 300, 1, False), (2, 1, 9, 2, True), (4, 3, 6, 2100, False), (3, 3, 12, 700, False)])
def test_average_of_biases_far_apart_decodes_parts(E, M, U, chunks, own):
    # the fp64 sums take a sub-chunk in parts and go on where a user's part ended: more users than a wavefront keeps places for,
    # sub-chunks longer than a window in some lanes, a ragged chunk; a damaged index is counted as the integer sums count it
    import torch
    from paper_2204_08211_amd import binding as B
    rng = np.random.default_rng(40 * E + U)
    d, b0 = 4096 * chunks + 1500, 2 ** (E - 1)
    nm = orc.num_magnitudes(E, M)
    bias = (b0 + rng.integers(0, 22, (U, 1))).astype(np.int32)
    bias[0], bias[-1] = b0, b0 + (21 if U > 1 else 0)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(U)
    scale = torch.tensor([2.0 ** (b0 - int(b)) for b in bias[:, 0]], device="cuda:0")
    x = torch.randn((U, d), generator=gen, device="cuda:0") * float(orc.grid(E, M, b0)[-1]) / 2
    x[:, 128:128 + 640] = 0.0                                # sub-chunks of the shortest word
    plan, books, buf = coded(E, M, (x * scale[:, None]).float(), bias, own=own)
    if not own:                                              # a code that gives the frequent symbols long words
        w = np.zeros(1 << (1 + E + M), np.uint64)
        A = w.size
        emit = sorted([0] + [s for s in range(A) if 0 < (s & (A // 2 - 1)) < nm], key=lambda s: s & (A // 2 - 1))
        w[emit] = [max(1, int(2.0 ** (40 - 40.0 * i / len(emit)))) for i in range(len(emit))]
        books = B.co3_build_codebook(E, M, 1, w[None, :])
        buf = B.RoundBuffers(plan, "cuda:0", max_code_len=64)
        g = torch.zeros((U, (d + 3) // 4 * 4), dtype=torch.float32, device="cuda:0")
        g[:, :d] = x * scale[:, None]
        m = torch.zeros_like(g)
        B.co3_encode(plan, books, g, m, m, 0.0, buf, mode=BOOK_FIXED)
    want = in_order_average(plan, books, buf)
    near = B.Plan(E, M, U, d, np.full((U, 1), b0, np.int32), per_user_books=own)
    device_bias(near, bias)
    out = torch.full((d,), float("nan"), dtype=torch.float32, device="cuda:0")
    B.co3_ps_aggregate(near, books, buf, out)
    torch.cuda.synchronize()
    assert not buf.status.cpu().numpy()[2:].any()
    gu.assert_bits_equal(out.cpu().numpy(), want, "average")
    # lanes of sub-chunks 3 and 4 of every user's second chunk start and end beside a codeword
    buf.sub_bits[:, 64 + 3] += 1
    buf.sub_bits[:, 64 + 4] -= 1
    counts = []
    for biases in (bias, np.full((U, 1), b0, np.int32)):
        buf.status.zero_()
        device_bias(near, biases)
        B.co3_ps_aggregate(near, books, buf, out)
        torch.cuda.synchronize()
        counts.append(int(buf.status[5]))
    assert counts[0] == counts[1] >= (U + 1) // 2 and not buf.status.cpu().numpy()[[2, 3, 6]].any()


@pytest.mark.parametrize("U", [3, 4])
@pytest.mark.parametrize("chunks,own,gain", [(520, False, False), (1100, False, True), (9, True, False), (1210, True, True)])
def test_few_users_keep_their_order_wide(U, chunks, own, gain):
    # 16-bit symbols, sums that depend on the order (biases far apart, or a scale): two wavefronts a chunk, several chunks a
    # workgroup, a table each, the users one after the other
    import torch
    from paper_2204_08211_amd import binding as B
    E, M, d = 4, 5, 4096 * chunks + 100
    bias = np.array([[10], [66], [10], [64]], np.int32)[:U]
    g = cancelling(U, d, bias, float(orc.grid(E, M, 10)[-1]), U + chunks)
    plan, books, buf = coded(E, M, g, bias, own=own)
    if gain:
        rng = np.random.default_rng(chunks)
        inv = (2.0 ** rng.uniform(-0.5, 0.5, (U, 1))).astype(np.float32)
        plan.set_gain((np.float32(1.0) / inv).astype(np.float32), inv)
    want = in_order_average(plan, books, buf)
    out = torch.zeros(d, dtype=torch.float32, device="cuda:0")
    B.co3_ps_aggregate(plan, books, buf, out)
    torch.cuda.synchronize()
    assert not buf.status.cpu().numpy()[2:].any()
    gu.assert_bits_equal(out.cpu().numpy(), want, "average")


@pytest.mark.parametrize("U,E,M,chunks,own", [(8, 4, 5, 1100, False), (1, 5, 6, 4200, False), (18, 4, 4, 2, False),   # sets of chunks, more than a turn
                                              (6, 4, 5, 1210, True), (2, 5, 6, 1201, True), (7, 4, 4, 30, True)])      # the users in turns, two wavefronts
def test_wide_average_with_a_scale(U, E, M, chunks, own):
    # 16-bit symbols with a scale where a workgroup takes several chunks or the users one after the other
    rng = np.random.default_rng(60 + U)
    seg_len = [4096 * chunks + 3, 4096 + 9]
    d, b0 = sum(seg_len), 2 ** (E - 1)
    import torch
    from paper_2204_08211_amd import binding as B
    bias = (b0 + rng.integers(0, 3, (U, 2))).astype(np.int32)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(U)
    plan, books, buf = coded(E, M, torch.randn((U, d), generator=gen, device="cuda:0") * float(orc.grid(E, M, b0 + 2)[-1]) / 4, bias,
                             own=own, seg_len=seg_len)
    # (the order of the users is defined up to four, and where they come one after the other)
    exact = U > 4 and not (own and chunks >= 1200)
    inv = (2.0 ** (rng.integers(-1, 2, (U, 2)) if exact else rng.uniform(-0.5, 0.5, (U, 2)))).astype(np.float32)
    inv[:, 1] = 1.0
    plan.set_gain((np.float32(1.0) / inv).astype(np.float32), inv)
    want = in_order_average(plan, books, buf)
    out = torch.full((d,), float("nan"), dtype=torch.float32, device="cuda:0")
    B.co3_ps_aggregate(plan, books, buf, out)
    torch.cuda.synchronize()
    assert not buf.status.cpu().numpy()[2:].any()
    gu.assert_bits_equal(out.cpu().numpy(), want, "average")


@pytest.mark.parametrize("U,chunks,E,M,own,gain", [
    (1, 1, 5, 2, False, False), (1, 9, 4, 3, False, True), (1, 2051, 2, 1, True, False),                     # the decoder writes them
    (10, 2500, 4, 3, False, False), (10, 2501, 4, 3, False, False), (11, 515, 5, 2, False, False),           # in LDS, integer sums
    (17, 1400, 5, 2, False, False), (17, 1401, 5, 2, False, False), (32, 250, 3, 2, False, False), (33, 250, 3, 2, False, False),
    (10, 2304, 4, 3, False, False), (10, 2305, 4, 3, False, False), (8, 2500, 4, 3, False, False), (8, 2501, 4, 3, False, False),
    (7, 768, 3, 2, False, False), (7, 769, 3, 2, False, False), (7, 1025, 3, 2, False, False),               # in LDS, integer sums
    (10, 1280, 2, 1, False, False), (10, 1281, 2, 1, False, False), (14, 256, 4, 3, False, True), (14, 257, 4, 3, False, True),
    (12, 1400, 5, 2, False, False), (12, 1401, 5, 2, False, False), (17, 1280, 5, 2, False, False), (17, 1281, 5, 2, False, False),
    (8, 256, 5, 2, False, False), (8, 257, 5, 2, False, False), (2, 1024, 4, 3, False, True), (2, 1025, 4, 3, True, False), (5, 1264, 2, 1, True, False),   # one a wavefront
    (31, 250, 3, 2, False, False), (31, 120, 5, 2, False, True), (32, 120, 5, 2, False, True),
    (10, 1250, 3, 1, True, False), (10, 1251, 3, 1, True, False), (6, 1100, 5, 2, True, False), (31, 70, 4, 3, True, False)])
def test_average_at_the_edges_of_its_rules(U, chunks, E, M, own, gain):
    # one user, users of a chunk in one workgroup and the other forms, on both sides of where they change; a ragged chunk in
    # front, so that the others lie at an odd offset, and one behind; two tables.  Values and sums are exact in fp64.
    import torch
    from paper_2204_08211_amd import binding as B
    seg_len = [5, 4096 * max(chunks - 2, 0), 3001] if chunks > 1 else [3001]
    d, nseg = sum(seg_len), len(seg_len)
    rng = np.random.default_rng(U + chunks)
    bias = rng.integers(14, 18, (U, nseg)).astype(np.int32)
    plan = B.Plan(E=E, M=M, U=U, d=d, bias=bias, seg_len=seg_len, seg_book=[0, 1, 0][:nseg], per_user_books=own)
    if gain:
        inv = (2.0 ** rng.uniform(-0.5, 0.5, (U, nseg))).astype(np.float32)
        plan.set_gain((np.float32(1.0) / inv).astype(np.float32), inv)
    dev, stride = torch.device("cuda:0"), (d + 3) // 4 * 4
    top = float(orc.grid(E, M, 16)[-1])
    gen = torch.Generator(device=dev); gen.manual_seed(chunks)
    g = torch.randn((U, stride), device=dev, generator=gen) * (top / 4)
    m = torch.zeros_like(g)
    books = B.co3_build_codebook(E, M, plan.num_books, None)
    buf = B.RoundBuffers(plan, dev, max_code_len=16)
    buf.status.zero_()
    B.co3_encode(plan, books, g, m, m, 0.9, buf, mode=BOOK_EMPIRICAL)
    del g
    B.co3_decode(plan, books, buf, q=m)
    out = torch.full((d,), float("nan"), dtype=torch.float32, device=dev)
    model = torch.randn((d,), device=dev, generator=gen)
    before = model.double()
    B.co3_ps_aggregate(plan, books, buf, out, model=model, eta=0.25)
    total = torch.zeros(d, dtype=torch.float64, device=dev)
    for u in range(U):
        total += m[u, :d].double()
    mean = total * (1.0 / U)
    assert not buf.status[2:].any()      # (the words in front count clipped values)
    assert torch.equal(out, mean.float()) and torch.equal(model, (before - 0.25 * mean).float())
    assert bool((out != 0).any())
