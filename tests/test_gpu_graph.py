"""A whole round (co3_encode + co3_ps_aggregate) captured in a HIP graph and replayed (pytest -m gpu).
The library clears its counters with fill kernels, not memset nodes, so the sequence may be
captured; every replay, with fresh inputs written into the captured buffers and eager work and
synchronisations in between, must reproduce the eager result bit for bit."""
import numpy as np
import pytest

import co3_synth as syn
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("single_sweep,E,M", [(False, 4, 3), (True, 4, 3), (False, 5, 5)])
def test_round_in_a_graph_equals_eager(single_sweep, E, M):
    # (5, 5): 16-bit symbols, the code rebuilt per round (the model code below is for alphabets of up to 8 bits)
    import torch
    from paper_2204_08211_amd import binding as B
    U, d = 4, 4096 * 11 + 321
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(77)
    stride = (d + 3) // 4 * 4
    bias0 = 16 if E == 4 else 24
    plan = B.Plan(E, M, U, d, [[bias0]] * U)
    # a model code (every producible symbol has a codeword) for the fixed mode; rebuilt per round otherwise
    books = B.co3_build_codebook(E, M, plan.num_books,
                                 B.co3_gennorm_weights(E, M, 16, 0.0, 5e-3, 1.0)[None, :] if single_sweep else None)
    buf = B.RoundBuffers(plan, dev, max_code_len=64)
    g = torch.zeros((U, stride), dtype=torch.float32, device=dev)
    m = torch.zeros((U, stride), dtype=torch.float32, device=dev)
    out = torch.zeros(d, dtype=torch.float32, device=dev)
    mode = B.BOOK_FIXED if single_sweep else B.BOOK_EMPIRICAL

    def fresh(it):
        return torch.from_numpy(np.stack([syn.gennorm_numpy(rng, d, 1.0, 2e-3 * (1 + it)) for _ in range(U)])).to(dev)

    def step():   # the binding enqueues on torch's current stream
        B.co3_encode(plan, books, g, m, m, 0.9, buf, mode=mode, single_sweep=single_sweep)
        B.co3_ps_aggregate(plan, books, buf, out)

    g[:, :d] = fresh(0)

    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                              # warm-up on the capture stream
        side.synchronize()
        m.zero_()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()

    m_eager = torch.zeros_like(m)
    for it in range(4):
        g[:, :d] = fresh(it + 1)
        # eager reference on copies of the state the replay starts from
        m_ref = m.clone()
        buf_ref = B.RoundBuffers(plan, dev, max_code_len=64)
        out_ref = torch.zeros_like(out)
        B.co3_encode(plan, books, g, m_ref, m_ref, 0.9, buf_ref, mode=mode, single_sweep=single_sweep)
        B.co3_ps_aggregate(plan, books, buf_ref, out_ref)
        torch.cuda.synchronize()
        buf.words.zero_(); out.fill_(float("nan"))             # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(m, m_ref), f"memory, replay {it}"
        assert torch.equal(buf.chunk_offset, buf_ref.chunk_offset) and torch.equal(buf.sub_bits, buf_ref.sub_bits)
        assert torch.equal(buf.payload_bits, buf_ref.payload_bits)
        for u in range(U):
            nw = int(buf_ref.chunk_offset[u, -1].item()) // 32
            assert torch.equal(buf.words[u, :nw], buf_ref.words[u, :nw]), f"stream {u}, replay {it}"
        assert torch.equal(out, out_ref), f"average, replay {it}"
        if not single_sweep:
            assert torch.equal(buf.hist, buf_ref.hist)
    st = buf.status.cpu().numpy()
    assert st[B.STAT_NOCODE] == 0 and st[B.STAT_CORRUPT] == 0 and st[B.STAT_STALLED] == 0 and st[B.STAT_CAPACITY] == 0


@pytest.mark.parametrize("E,M,U,chunks,own", [
    (4, 3, 3, 3, False), (4, 3, 8, 2, False), (4, 3, 20, 2, False), (2, 1, 5, 2, True),   # integer sums, users side by side
    (4, 3, 2, 2100, False),                                                              # a wavefront per chunk
    (4, 3, 4, 1500, False), (2, 1, 4, 1500, False),                                      # two wavefronts, four users
    (5, 2, 3, 3, False), (5, 2, 13, 2, True), (5, 2, 40, 2, False),                      # symbols met in LDS, turns of four users
    (5, 2, 4, 2100, False), (5, 2, 1, 5, True),                                          # a wavefront per chunk
    (4, 5, 3, 3, False),                                                                 # 16-bit symbols
])
def test_scale_and_bias_installed_between_replays(E, M, U, chunks, own):
    # a captured round follows what the plan carries when it is replayed: no scale, a scale in some layers from the host, a
    # scale and other biases from the device, biases far apart, no scale again.  The average is that of co3_decode's values.
    import torch
    from paper_2204_08211_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(E * 100 + U)
    seg_len = [4096 * 2 + 7, 4096 * chunks + 5, 3000]
    d, nseg, b0 = sum(seg_len), len(seg_len), 2 ** (E - 1)
    near = (b0 + rng.integers(0, 3, (U, nseg))).astype(np.int32)
    far = near.copy()
    far[0, 1] += 14
    plan = B.Plan(E, M, U, d, near, seg_len=seg_len, seg_book=[0, 1, 0], per_user_books=own)
    books = B.co3_build_codebook(E, M, plan.num_books, None)
    buf = B.RoundBuffers(plan, dev, max_code_len=40)
    stride = (d + 3) // 4 * 4
    gen = torch.Generator(device=dev)
    gen.manual_seed(U)
    g = torch.randn((U, stride), generator=gen, device=dev) * 0.7
    m = torch.zeros_like(g)
    out = torch.zeros(d, dtype=torch.float32, device=dev)
    q = torch.zeros_like(g)

    def step():
        B.co3_encode(plan, books, g, m, m, 0.9, buf)
        B.co3_ps_aggregate(plan, books, buf, out)

    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()

    # the fp64 sums of up to four users are in their order; of more, powers of two keep them exact
    inv = (2.0 ** (rng.uniform(-0.5, 0.5, (U, nseg)) if U <= 4 else rng.integers(-1, 2, (U, nseg)))).astype(np.float32)
    inv[:, 0] = 1.0
    gain = (np.float32(1.0) / inv).astype(np.float32)
    pairs = torch.from_numpy(np.stack([gain, inv], axis=2)).to(dev)
    bias_near, bias_far = torch.from_numpy(near + 1).to(dev), torch.from_numpy(far).to(dev)
    L = B.lib()
    states = [
        ("none", lambda: None),
        ("scale from the host", lambda: plan.set_gain(gain, inv)),
        ("no scale", lambda: plan.set_gain(None, None)),
        ("scale and biases from the device", lambda: (B._check("gain", L.co3_plan_set_gain_device(plan.handle, pairs.data_ptr(), B._stream())),
                                                      B._check("bias", L.co3_plan_set_bias_device(plan.handle, bias_near.data_ptr(), B._stream())))),
        ("and biases far apart", lambda: B._check("bias", L.co3_plan_set_bias_device(plan.handle, bias_far.data_ptr(), B._stream()))),
        ("biases far apart, no scale", lambda: plan.set_gain(None, None)),
        ("none again", lambda: plan.set_bias(near)),
    ]
    for what, install in states:
        install()
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        B.co3_decode(plan, books, buf, q=q)
        total = torch.zeros(d, dtype=torch.float64, device=dev)
        for u in range(U):
            total += q[u, :d].double()
        want = (total * (1.0 / U)).float()
        torch.cuda.synchronize()
        assert not buf.status.cpu().numpy()[2:].any(), what
        gu.assert_bits_equal(out.cpu().numpy(), want.cpu().numpy(), f"average, {what}")
