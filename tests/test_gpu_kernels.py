"""GPU parity of the full-step kernels (bf16 GEMM with its epilogues, flash
attention) against the oracle's primitives, through the C ABI.

Small shapes span several tiles and a ragged tail in every dimension; the
workload-sized cases run the exact launch shapes of the FLUX-1024 step and
compare sampled outputs computed one by one in float64."""
import numpy as np
import pytest

from oracle import dit
from oracle.numerics import round_bf16
from paper_2608_09231_amd import binding
from tests._gpu import assert_bf16_close, dev, host_bf16, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(2024)


def bf16_bits(x):
    """float64 -> bf16 bit patterns of round_bf16(x) (exact)."""
    r = round_bf16(x).astype(np.float32)
    return (r.view(np.uint32) >> 16).astype(np.uint16)


def bits_to_f64(b):
    return (b.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def make(shape, scale=1.0):
    b = bf16_bits(RNG.standard_normal(shape) * scale)
    return b, bits_to_f64(b)


@pytest.mark.parametrize("M,N,K", [(300, 392, 200), (37, 136, 64), (1, 8, 8), (513, 256, 3072)])
def test_gemm_store_and_bias(M, N, K):
    torch = torch_cuda()
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    out = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K)
    assert_bf16_close(host_bf16(out), round_bf16(a @ w.T + b))


def test_gemm_epilogues_gelu_silu_f32():
    torch = torch_cuda()
    M, N, K = 260, 300, 136
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.1)
    b_b, b = make((N,), 0.1)
    y = a @ w.T + b
    out = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K, gelu_from=100)
    ref = round_bf16(np.concatenate([y[:, :100], dit.gelu_tanh(y[:, 100:])], axis=1))
    assert_bf16_close(host_bf16(out), ref)
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K,
                      flags=binding.EPI_SILU)
    assert_bf16_close(host_bf16(out), round_bf16(dit.silu(y)))
    of = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), of, M=M, N=N, K=K,
                      flags=binding.EPI_F32)
    np.testing.assert_allclose(of.cpu().numpy(), y, rtol=1e-5, atol=1e-5)


def test_gemm_qkv_rms_and_gated_residual():
    torch = torch_cuda()
    M, H = 203, 256
    N, K = 3 * H + 512, H
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    y = a @ w.T + b
    ld = 4 * H + 512
    out = torch.zeros((M, ld), dtype=torch.int16, device="cuda")
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K, ldc=ld,
                      rms_cols=2 * H, gelu_from=3 * H, gap_at=3 * H, gap=H)
    got = host_bf16(out)
    assert_bf16_close(got[:, :2 * H], round_bf16(dit.rms_heads(y[:, :2 * H], 2 * H // 128, 128)))
    assert_bf16_close(got[:, 2 * H:3 * H], round_bf16(y[:, 2 * H:3 * H]))
    assert_bf16_close(got[:, 4 * H:], round_bf16(dit.gelu_tanh(y[:, 3 * H:])))
    assert np.all(got[:, 3 * H:4 * H] == 0)          # the hole is left untouched
    # gated residual in place: C = S(C + g * (A W^T + b))
    N2 = H
    w2_b, w2 = make((N2, K), 0.05)
    b2_b, b2 = make((N2,), 0.1)
    c0_b, c0 = make((M, N2))
    g = RNG.standard_normal(N2).astype(np.float32)
    cbuf = dev(torch, c0_b)
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w2_b), dev(torch, b2_b), cbuf, M=M, N=N2, K=K,
                      flags=binding.EPI_GATED_RES, gate=dev(torch, g))
    ref = round_bf16(c0 + g.astype(np.float64) * (a @ w2.T + b2))
    assert_bf16_close(host_bf16(cbuf), ref)


@pytest.mark.parametrize("gated", [False, True])
def test_gemm_ring_pipeline_ragged(gated):
    """256 x 256 tiles with the five-slice LDS ring (chosen for this shape:
    one full wave of 16 x 16 tiles), ragged M and N, K = 320 = five 64-deep
    slices (prologue, steady slices and the peeled tail); plain and gated
    residual epilogues against float64."""
    torch = torch_cuda()
    M, N, K = 3999, 3992, 320
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    y = a @ w.T + b
    if not gated:
        out = torch.zeros((M, N), dtype=torch.int16, device="cuda")
        binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K)
        assert_bf16_close(host_bf16(out), round_bf16(y))
    else:
        c0_b, c0 = make((M, N))
        g = RNG.standard_normal(N).astype(np.float32)
        cbuf = dev(torch, c0_b)
        binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), cbuf, M=M, N=N, K=K,
                          flags=binding.EPI_GATED_RES, gate=dev(torch, g))
        assert_bf16_close(host_bf16(cbuf), round_bf16(c0 + g.astype(np.float64) * y))


@pytest.mark.parametrize("K", [128, 192])
@pytest.mark.parametrize("flags", [binding.EPI_STORE, binding.EPI_F32, binding.EPI_GATED_RES])
def test_gemm_ring_shortest_pipelines(K, flags):
    """The ring kernel at its two and three slices of K (prologue and peeled
    tail only; one steady slice), one ragged row of 256 x 256 tiles that fills
    the chip once, with each of its three epilogues."""
    torch = torch_cuda()
    M, N = 250, 65528
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    y = a @ w.T + b
    args = dict(M=M, N=N, K=K, flags=flags)
    if flags == binding.EPI_F32:
        out = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, **args)
        np.testing.assert_allclose(out.cpu().numpy(), y, rtol=1e-5, atol=1e-5)
        return
    c0_b, c0 = make((M, N))
    g = RNG.standard_normal(N).astype(np.float32)
    gated = flags == binding.EPI_GATED_RES
    out = dev(torch, c0_b)
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, gate=dev(torch, g) if gated else None,
                      **args)
    assert_bf16_close(host_bf16(out), round_bf16(c0 + g.astype(np.float64) * y if gated else y))


@pytest.mark.parametrize("flags", [binding.EPI_STORE, binding.EPI_F32, binding.EPI_GATED_RES, binding.EPI_SILU])
@pytest.mark.parametrize("M,N,K", [
    (33, 392, 40),      # small kernel: a ragged second row tile, less than one step for some waves
    (5, 1000, 3072),    # the same, all K shared out, a ragged last column tile
    (31, 16392, 128),   # 32 x 128 tiles: fewer slices than the pipeline holds
    (100, 16392, 448),  # the same, past the pipeline's depth
])
def test_gemm_few_rows(M, N, K, flags):
    """The kernels for few rows and few tiles, every epilogue, against float64."""
    torch = torch_cuda()
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    y = a @ w.T + b
    args = dict(M=M, N=N, K=K, flags=flags)
    if flags == binding.EPI_F32:
        out = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, **args)
        np.testing.assert_allclose(out.cpu().numpy(), y, rtol=1e-5, atol=2e-5)
        return
    c0_b, c0 = make((M, N))
    g = RNG.standard_normal(N).astype(np.float32)
    out, gate = dev(torch, c0_b), None
    if flags == binding.EPI_GATED_RES:
        y, gate = c0 + g.astype(np.float64) * y, dev(torch, g)
    elif flags == binding.EPI_SILU:
        y = dit.silu(y)
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, gate=gate, **args)
    assert_bf16_close(host_bf16(out), round_bf16(y))


LAST_ROUND_GEMMS = [
    (4300, 4104, 2112, binding.EPI_STORE),       # 289 tiles: 33 shared out in 7 uneven parts of 33 slices
    (4300, 4104, 2112, binding.EPI_GATED_RES),
    (4100, 4360, 2112, binding.EPI_F32),         # 306 tiles: 50 in 5
    (4100, 4360, 2112, binding.EPI_SILU),
    (4096, 6144, 4096, binding.EPI_STORE),       # 384 tiles: 128 in 2
]


@pytest.mark.parametrize("M,N,K,flags", [(4100, 4360, 1600, binding.EPI_F32)] + LAST_ROUND_GEMMS)  # (first: whole tiles)
def test_gemm_ring_last_round(M, N, K, flags):
    """Tiles past the last whole round in shares of K, added by the finishing
    kernel with the ring kernel's epilogues (norm, GELU and column gap too):
    sampled rows against float64."""
    torch = torch_cuda()
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    rows = np.unique(np.concatenate([np.arange(M - 300, M, 7), RNG.choice(M, 60)]))
    y = a[rows] @ w.T + b
    gap = 512 if flags == binding.EPI_STORE else 0
    out = torch.zeros((M, N + gap), dtype=torch.float32 if flags == binding.EPI_F32 else torch.int16, device="cuda")
    args = dict(M=M, N=N, K=K, ldc=N + gap, flags=flags)
    if flags == binding.EPI_STORE:
        args.update(rms_cols=2048, gelu_from=3072, gap_at=3072, gap=gap)
        ref = np.concatenate([dit.rms_heads(y[:, :2048], 16, 128), y[:, 2048:3072],
                              np.zeros((len(rows), gap)), dit.gelu_tanh(y[:, 3072:])], axis=1)
    elif flags == binding.EPI_SILU:
        ref = dit.silu(y)
    else:
        ref = y
    gate = None
    if flags == binding.EPI_GATED_RES:
        c0_b, c0 = make((M, N))
        g = RNG.standard_normal(N).astype(np.float32)
        out, gate, ref = dev(torch, c0_b), dev(torch, g), c0[rows] + g.astype(np.float64) * y
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, gate=gate, **args)
    if flags == binding.EPI_F32:
        np.testing.assert_allclose(out.cpu().numpy()[rows], ref, rtol=1e-5, atol=3e-5)
    else:
        assert_bf16_close(host_bf16(out)[rows], round_bf16(ref))


def test_gemm_ring_rms_gelu_gap_ragged():
    """The ring kernel's store epilogue with the single-block projection's
    column roles at a ragged M: per-head RMS on the first 2 H columns, GELU
    on the MLP half, written past a hole of H columns."""
    torch = torch_cuda()
    M, H, F, K = 3999, 1024, 1024, 320
    N, ld = 3 * H + F, 4 * H + F
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    y = a @ w.T + b
    out = torch.zeros((M, ld), dtype=torch.int16, device="cuda")
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K, ldc=ld,
                      rms_cols=2 * H, gelu_from=3 * H, gap_at=3 * H, gap=H)
    got = host_bf16(out)
    assert_bf16_close(got[:, :2 * H], round_bf16(dit.rms_heads(y[:, :2 * H], 2 * H // 128, 128)))
    assert_bf16_close(got[:, 2 * H:3 * H], round_bf16(y[:, 2 * H:3 * H]))
    assert_bf16_close(got[:, 4 * H:], round_bf16(dit.gelu_tanh(y[:, 3 * H:])))
    assert np.all(got[:, 3 * H:4 * H] == 0)


def attn_case(torch, Lq, Lk, heads, sample_rows=None):
    H = heads * 128
    q_b, q = make((Lq, H))
    k_b, k = make((Lk, H))
    v_b, v = make((Lk, H))
    o = torch.zeros((Lq, H), dtype=torch.int16, device="cuda")
    ws = torch.zeros(heads * 128 * ((Lk + 63) // 64 * 64), dtype=torch.int16, device="cuda")
    binding.attention_bf16(dev(torch, q_b), dev(torch, k_b), dev(torch, v_b), o, Lq=Lq, Lk=Lk, heads=heads,
                           ldq=H, ldk=H, ldv=H, ldo=H, vt_ws=ws)
    got = host_bf16(o)
    rows = np.arange(Lq) if sample_rows is None else sample_rows
    ref = round_bf16(dit.attention(q[rows], k, v, heads, 128))
    return got[rows], ref


@pytest.mark.parametrize("Lq,Lk,heads", [(200, 200, 2), (130, 33, 1), (1, 1, 1), (64, 300, 3)])
def test_attention_small_ragged(Lq, Lk, heads):
    torch = torch_cuda()
    got, ref = attn_case(torch, Lq, Lk, heads)
    assert rel_l2(got, ref) < 4e-3
    assert np.max(np.abs(got - ref)) <= 3 * 2.0 ** -8 * np.max(np.abs(ref))


def test_attention_flux1024_joint_shape_sampled():
    """FLUX-1024 joint attention: 4608 tokens, 24 heads; 96 sampled queries."""
    torch = torch_cuda()
    L, heads = 4096 + 512, 24
    rows = np.sort(RNG.choice(L, 96, replace=False))
    got, ref = attn_case(torch, L, L, heads, rows)
    assert rel_l2(got, ref) < 4e-3


def test_gemm_flux1024_single_block_shape_sampled():
    """Single-block input projection of FLUX-1024: [4608 x 3072] x [21504 x 3072]^T
    with the fused RMS / GELU / gap epilogue; 2048 sampled outputs per region."""
    torch = torch_cuda()
    M, H, F = 4608, 3072, 12288
    N, K = 3 * H + F, H
    a_b = bf16_bits(RNG.standard_normal((M, K)))
    w_b = bf16_bits(RNG.standard_normal((N, K)) * 0.02)
    b_b = bf16_bits(RNG.standard_normal(N) * 0.02)
    ld = 4 * H + F
    out = torch.zeros((M, ld), dtype=torch.int16, device="cuda")
    binding.gemm_bf16(dev(torch, a_b), dev(torch, w_b), dev(torch, b_b), out, M=M, N=N, K=K, ldc=ld,
                      rms_cols=2 * H, gelu_from=3 * H, gap_at=3 * H, gap=H)
    got = host_bf16(out)
    a, w, b = bits_to_f64(a_b), bits_to_f64(w_b), bits_to_f64(b_b)
    rows = RNG.choice(M, 16, replace=False)
    # q/k heads need the whole head row for the RMS norm: sample rows x heads
    for r in rows:
        y = a[r] @ w.T + b
        qk = round_bf16(dit.rms_heads(y[None, :2 * H], 2 * H // 128, 128))[0]
        assert_bf16_close(got[r, :2 * H], qk, frac_exact=0.8)
        assert_bf16_close(got[r, 2 * H:3 * H], round_bf16(y[2 * H:3 * H]), frac_exact=0.8)
        assert_bf16_close(got[r, 4 * H:], round_bf16(dit.gelu_tanh(y[3 * H:])), frac_exact=0.8)


@pytest.mark.parametrize("L,heads", [(4608, 24), (333, 2)])
def test_attention_bounded_logits_rms_normalised(L, heads):
    """The sampler's path: q and k leave a unit-gain RMS norm, so the kernel
    may replace the running max by a fixed shift (DIT_ATTN_BOUNDED_LOGITS)."""
    torch = torch_cuda()
    H = heads * 128
    def mk(n, norm):
        x = RNG.standard_normal((n, H)) * 3.0
        if norm:
            x = dit.rms_heads(x, heads, 128)
        b = bf16_bits(x)
        return b, bits_to_f64(b)
    q_b, q = mk(L, True)
    k_b, k = mk(L, True)
    v_b, v = mk(L, False)
    o = torch.zeros((L, H), dtype=torch.int16, device="cuda")
    ws = torch.zeros(heads * 128 * ((L + 63) // 64 * 64), dtype=torch.int16, device="cuda")
    binding.attention_bf16(dev(torch, q_b), dev(torch, k_b), dev(torch, v_b), o, Lq=L, Lk=L, heads=heads,
                           ldq=H, ldk=H, ldv=H, ldo=H, vt_ws=ws, flags=binding.ATTN_BOUNDED_LOGITS)
    got = host_bf16(o)
    rows = np.sort(RNG.choice(L, min(L, 64), replace=False))
    ref = round_bf16(dit.attention(q[rows], k, v, heads, 128))
    assert rel_l2(got[rows], ref) < 4e-3


def bounded_case(torch, Lq, Lk, heads, bounded):
    H = heads * 128

    def mk(n, norm):
        x = RNG.standard_normal((n, H)) * 2.0
        b = bf16_bits(dit.rms_heads(x, heads, 128) if norm else x)
        return b, bits_to_f64(b)
    (q_b, q), (k_b, k), (v_b, v) = mk(Lq, bounded), mk(Lk, bounded), mk(Lk, False)
    args = dict(Lq=Lq, Lk=Lk, heads=heads, ldq=H, ldk=H, ldv=H, ldo=H,
                flags=binding.ATTN_BOUNDED_LOGITS if bounded else 0)
    rows = np.unique(np.concatenate([[0, Lq - 1], RNG.choice(Lq, min(Lq, 40), replace=False)]))
    ref = round_bf16(dit.attention(q[rows], k, v, heads, 128))
    return [dev(torch, t) for t in (q_b, k_b, v_b)], args, rows, ref


LAST_ROUND_ATTENTION = [  # Lq, Lk, heads, whole rounds before it, shares that hold parts of two items (None: not shared)
    (1, 64 * 30, 1, 0, False),    # one item, shared in seven
    (256, 768, 40, 0, False),     # items in three shares each, the fewest that a shared item has
    (257, 4100, 3, 0, False),     # a ragged second query block, shares of one XCD in several pieces
    (5000, 2001, 8, 0, True),     # 20 items an XCD in 32 shares, ragged queries and keys
    (9300, 750, 8, 1, False),     # a whole round, then five items in fifteen
    (13200, 2001, 8, 1, True),    # a whole round, then 20 items in 32
    (8300, 700, 8, 1, None),      # 33 items an XCD, eleven tiles: a whole round, one whole item
    (8192, 130, 10, 1, None),     # 40 an XCD, three tiles: whole items in the last round
    (2048, 2050, 1, 0, False),    # eight items, a last tile of two keys
]


@pytest.mark.parametrize("bounded", [True, False])
@pytest.mark.parametrize("Lq,Lk,heads", [(1, 64 * 9, 1)] + [c[:3] for c in LAST_ROUND_ATTENTION])  # (first: small kernel)
def test_attention_last_round(Lq, Lk, heads, bounded):
    """Items per work-group, the shared last round and its pieces, ragged
    queries and keys: sampled rows against float64."""
    torch = torch_cuda()
    (q, k, v), args, rows, ref = bounded_case(torch, Lq, Lk, heads, bounded)
    o = torch.full((Lq, heads * 128), 0x7fc0, dtype=torch.int16, device="cuda")  # NaN: every row written
    ws = torch.zeros(heads * 128 * ((Lk + 63) // 64 * 64), dtype=torch.int16, device="cuda")
    binding.attention_bf16(q, k, v, o, vt_ws=ws, **args)
    got = host_bf16(o)
    assert np.all(np.isfinite(got))
    assert rel_l2(got[rows], ref) < 4e-3


SMALL_ATTENTION = [
    (1, 1, 1), (31, 31, 2), (33, 257, 3),   # waves without keys, one key past a block
    (700, 1279, 2),                         # as many keys as the small kernel takes, uneven blocks
    (3000, 95, 5),                          # two rounds of work-groups
]


@pytest.mark.parametrize("bounded", [True, False])
@pytest.mark.parametrize("Lq,Lk,heads", SMALL_ATTENTION)
def test_attention_small(Lq, Lk, heads, bounded):
    """The kernel for few, short sequences against float64, NaN beyond the
    last key and query (rows of the buffers that belong to someone else)."""
    torch = torch_cuda()
    (q, k, v), args, rows, ref = bounded_case(torch, Lq, Lk, heads, bounded)
    H = heads * 128

    def padded(t, n):  # a NaN row behind the last one
        p = torch.full((n + 1, H), 0x7fc0, dtype=torch.int16, device="cuda")
        p[:n] = t
        return p
    o = torch.full((Lq + 1, H), 0x7fc0, dtype=torch.int16, device="cuda")
    ws = torch.zeros(H * ((Lk + 63) // 64 * 64), dtype=torch.int16, device="cuda")
    binding.attention_bf16(padded(q, Lq), padded(k, Lk), padded(v, Lk), o, vt_ws=ws, **args)
    got = host_bf16(o)
    assert np.all(np.isnan(got[Lq])) and np.all(np.isfinite(got[:Lq]))
    assert rel_l2(got[rows], ref) < 4e-3


def test_attention_calls_in_flight():
    """Four threads with streams of their own, each call with memory of its
    own for the shared items."""
    import threading
    torch = torch_cuda()
    cases, errs = [bounded_case(torch, 600, 3000, 2, True) for _ in range(4)], []

    def work(case):
        try:
            (q, k, v), args, rows, ref = case
            s = torch.cuda.Stream()
            o = torch.zeros((600, 256), dtype=torch.int16, device="cuda")
            ws = torch.zeros(256 * 3008, dtype=torch.int16, device="cuda")
            torch.cuda.synchronize()
            for _ in range(20):
                binding.attention_bf16(q, k, v, o, vt_ws=ws, stream=s, **args)
                assert rel_l2(host_bf16(o)[rows], ref) < 4e-3
        except Exception as e:  # reported by the main thread
            errs.append(e)
    ts = [threading.Thread(target=work, args=(c,)) for c in cases]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not errs, errs


@pytest.mark.parametrize("Lq,Lk,heads,first", [
    (40, 300, 2, 64),      # small kernel: whole 32-key blocks of a wave without a finite logit
    (40, 300, 2, 0),       # the same from the first key on
    (300, 3000, 2, 64),    # list kernel, last round shared: whole pieces without one
    (300, 3000, 2, 0),     # the same, the first tiles of a piece included
    (9000, 700, 8, 64),    # whole items: some of a wave's queries raise their maximum, others have none
    (9000, 700, 8, 0),
])
def test_attention_overflowing_logits(Lq, Lk, heads, first):
    """Logits that overflow to -inf weigh nothing: every second query against
    the keys from `first` on, but for the last 70."""
    torch = torch_cuda()
    H = heads * 128
    q = RNG.standard_normal((Lq, heads, 128))
    k = RNG.standard_normal((Lk, heads, 128))
    v = RNG.standard_normal((Lk, H))
    huge = np.arange(Lk)
    huge = (huge >= first) & (huge < Lk - 70)
    q[:, :, 0] = 0.0
    q[::2, :, 0] = 2e20
    k[:, :, 0] = np.where(huge[:, None], -1e20, 0.0)
    q_b, k_b, v_b = bf16_bits(q.reshape(Lq, H)), bf16_bits(k.reshape(Lk, H)), bf16_bits(v)
    o = torch.full((Lq, H), 0x7fc0, dtype=torch.int16, device="cuda")
    ws = torch.zeros(H * ((Lk + 63) // 64 * 64), dtype=torch.int16, device="cuda")
    binding.attention_bf16(dev(torch, q_b), dev(torch, k_b), dev(torch, v_b), o, Lq=Lq, Lk=Lk, heads=heads, ldq=H,
                           ldk=H, ldv=H, ldo=H, vt_ws=ws, flags=0)
    got = host_bf16(o)
    assert np.all(np.isfinite(got))
    rows = np.unique(np.concatenate([[0, 1, Lq - 2, Lq - 1], RNG.choice(Lq, 24, replace=False)]))
    for parity in (0, 1):
        r = rows[rows % 2 == parity]
        keys = ~huge if parity == 0 else np.ones(Lk, bool)
        ref = round_bf16(dit.attention(bits_to_f64(q_b)[r], bits_to_f64(k_b)[keys], bits_to_f64(v_b)[keys], heads, 128))
        assert rel_l2(got[r], ref) < 4e-3


def test_component_bits_do_not_depend_on_calls_in_flight():
    """Two calls wait behind other work on their streams; a third on a stream
    of its own gives the bits of a lone call (all of them share out their last
    round, attention and GEMM alike)."""
    import threading
    import time
    torch = torch_cuda()
    (q, k, v), args, _, _ = bounded_case(torch, 1000, 3000, 2, True)
    ws = [torch.zeros(256 * 3008, dtype=torch.int16, device="cuda") for _ in range(3)]
    M, N, K = 4300, 4104, 2112
    a, w, b = [dev(torch, make(s, 0.1)[0]) for s in ((M, K), (N, K), (N,))]
    big = torch.randn(8192, 8192, device="cuda").bfloat16()

    def attention(i, out, stream):
        binding.attention_bf16(q, k, v, out, vt_ws=ws[i], stream=stream, **args)

    def gemm(i, out, stream):
        binding.gemm_bf16(a, w, b, out, M=M, N=N, K=K, stream=stream)
    streams = [torch.cuda.Stream() for _ in range(3)]
    for call, shape in ((attention, (1000, 256)), (gemm, (M, N))):
        alone, *outs = [torch.zeros(shape, dtype=torch.int16, device="cuda") for _ in range(4)]
        torch.cuda.synchronize()
        call(2, alone, streams[2])
        for s in streams[:2]:
            with torch.cuda.stream(s):
                for _ in range(100):
                    big @ big
        ts = [threading.Thread(target=call, args=(i, outs[i], streams[i])) for i in range(2)]
        [t.start() for t in ts]
        time.sleep(0.03)
        call(2, outs[2], streams[2])
        [t.join() for t in ts]
        for o in outs:
            assert torch.equal(o, alone)


def strided(torch, bits, ld, fill=0x7fc0):
    """Rows of `bits` in a wider buffer whose other columns hold NaN."""
    b = np.full((bits.shape[0], ld), fill, np.uint16)
    b[:, :bits.shape[1]] = bits
    return dev(torch, b)


@pytest.mark.parametrize("M,N,K", [
    (33, 392, 40), (70, 520, 200), (28, 1160, 3072),   # small kernel: K off its steps, ragged tiles, whole K shared out
    (100, 17000, 448),                                 # 32 x 128 tiles
    (600, 1928, 1024), (4300, 4104, 2112),             # 128 x 128 tiles; ring, shared last round
])
@pytest.mark.parametrize("norm", [False, True])
def test_gemm_strided_forms(M, N, K, norm):
    """Row strides wider than the rows on every operand, a column gap, GELU
    from a column inside a tile and the norm on the first heads: the output's
    columns, and none beside them, in every kernel that takes such a call."""
    torch = torch_cuda()
    a_b, a = make((M, K))
    w_b, w = make((N, K), 0.05)
    b_b, b = make((N,), 0.1)
    gelu_from, gap, ldc = 260, 12, N + 12 + 4
    out = torch.full((M, ldc), 0x7fc0, dtype=torch.int16, device="cuda")
    binding.gemm_bf16(strided(torch, a_b, K + 8), strided(torch, w_b, K + 16), dev(torch, b_b), out, M=M, N=N, K=K,
                      lda=K + 8, ldw=K + 16, ldc=ldc, rms_cols=256 if norm else 0, gelu_from=gelu_from,
                      gap_at=gelu_from, gap=gap)
    rows = np.unique(np.concatenate([[0, M - 1], RNG.choice(M, min(M, 80), replace=False)]))
    y = a[rows] @ w.T + b
    if norm:
        y[:, :256] = dit.rms_heads(y[:, :256], 2, 128)
    y[:, gelu_from:] = dit.gelu_tanh(y[:, gelu_from:])
    got = host_bf16(out)
    assert np.all(np.isnan(got[:, gelu_from:gelu_from + gap])) and np.all(np.isnan(got[:, N + gap:]))
    assert_bf16_close(np.concatenate([got[rows, :gelu_from], got[rows, gelu_from + gap:N + gap]], axis=1), round_bf16(y))


@pytest.mark.parametrize("bounded", [True, False])
@pytest.mark.parametrize("Lq,Lk,heads", [(40, 300, 2), (300, 3000, 2), (9000, 130, 8)])
def test_attention_strided_forms(Lq, Lk, heads, bounded):
    """The same for attention (small kernel; list kernel with and without a
    shared last round), v at an odd stride."""
    torch = torch_cuda()
    H = heads * 128

    def mk(n, norm):
        x = RNG.standard_normal((n, H)) * 2.0
        b = bf16_bits(dit.rms_heads(x, heads, 128) if norm else x)
        return b, bits_to_f64(b)
    (q_b, q), (k_b, k), (v_b, v) = mk(Lq, bounded), mk(Lk, bounded), mk(Lk, False)
    o = torch.full((Lq, H + 4), 0x7fc0, dtype=torch.int16, device="cuda")
    ws = torch.zeros(H * ((Lk + 63) // 64 * 64), dtype=torch.int16, device="cuda")
    binding.attention_bf16(strided(torch, q_b, H + 8), strided(torch, k_b, H + 16), strided(torch, v_b, H + 1), o, Lq=Lq,
                           Lk=Lk, heads=heads, ldq=H + 8, ldk=H + 16, ldv=H + 1, ldo=H + 4, vt_ws=ws,
                           flags=binding.ATTN_BOUNDED_LOGITS if bounded else 0)
    got = host_bf16(o)
    assert np.all(np.isnan(got[:, H:])) and np.all(np.isfinite(got[:, :H]))
    rows = np.unique(np.concatenate([[0, Lq - 1], RNG.choice(Lq, min(Lq, 40), replace=False)]))
    assert rel_l2(got[rows, :H], round_bf16(dit.attention(q[rows], k, v, heads, 128))) < 4e-3
