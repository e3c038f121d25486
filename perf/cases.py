"""Performance cases of the cached DiT sampler and of its component kernels.

Three kinds of call, all through the package's public entry points:

* ``sample``: one call of the sampler (``DitCache.sample``, or
  ``sample_batch`` for several prompts): the whole loop with its gate,
  computed and reused steps, on models of the workloads' widths and token
  counts with one block of each kind (a block's cost does not depend on how
  many follow it), and on the small parity workloads as they are.
* ``gemm``: one linear layer with its fused epilogue (``gemm_bf16``).
* ``attention``: one attention call (``attention_bf16`` or its
  allocation-free form), q, k and v being column ranges of one projection
  buffer as a block produces them.

``exact`` evaluates the same calls with plain torch operations in float64.
"""
import functools
import math

import numpy as np
import torch

from paper_2608_09231_amd import binding, synth

DEV = "cuda"
KEPT_BLOBS = 8  # host weight blobs kept: several states of one model share one


# ------------------------------------------------------------------- cases

def _sample(name, dtype, heads, head_dim, mlp, n_img, n_txt, T, B, *, double=0, single=0, cross=0, channels=64,
            ctx=4096, batch=1, pooled=True, shift=3.0, guidance=1.0, solver="euler", prompts=1, policy="gate",
            bias=-10.0):
    c = dict(kind="sample", dtype=dtype, double=double, single=single, cross=cross, heads=heads, head_dim=head_dim,
             mlp=mlp, channels=channels, ctx=ctx, n_img=n_img, n_txt=n_txt, batch=batch, pooled=pooled, T=T, B=B,
             shift=shift, guidance=guidance, solver=solver, prompts=prompts, policy=policy, bias=bias)
    return dict(c, name=name) if name else c


def _gemm(name, M, N, K, epilogue="store", rms=0):
    c = dict(kind="gemm", M=M, N=N, K=K, epilogue=epilogue, rms=rms)
    return dict(c, name=name) if name else c


def _attention(name, Lq, Lk, heads, bounded, noalloc=False):
    c = dict(kind="attention", Lq=Lq, Lk=Lk, heads=heads, bounded=bounded, noalloc=noalloc)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call a user makes: the f32 workload of 64 + 16 tokens, where
        # launches, the host's wait for the indicator sums and latency are the time.
        _sample("sample_tiny_f32", "f32", 4, 32, 512, 64, 16, 10, 5, single=2, channels=16, ctx=128, shift=1.0),
        # A small bf16 model with ragged token counts (200 + 40): short launches of the MFMA kernels.
        _sample("sample_small_bf16", "bf16", 2, 128, 1024, 200, 40, 8, 4, double=2, single=2, ctx=96),
        # FLUX.1-dev widths at 1024^2 (4096 + 512 tokens), the 28-step schedule at B = 10.
        _sample("sample_flux1024", "bf16", 24, 128, 12288, 4096, 512, 28, 10, double=1, single=1),
        # Qwen-Image widths: a guidance pair, both branches stacked into each launch.
        _sample("sample_qwen_pair", "bf16", 24, 128, 12288, 4096, 256, 20, 8, double=1, ctx=3584, batch=2,
                pooled=False, guidance=4.0),
        # Wan2.1-14B widths: 81 frames at 480 x 832 (32760 video tokens), UniPC.  The largest call.
        _sample("sample_wan14b", "bf16", 40, 128, 13824, 32760, 512, 8, 2, cross=1, pooled=False, shift=5.0,
                solver="unipc"),
        # Serving several prompts at once: four 512^2 images (1024 + 512 tokens) in lockstep.
        _sample("sample_four_prompts", "bf16", 24, 128, 12288, 1024, 512, 8, 3, double=1, single=1, prompts=4),
        # The QKV projection of a block at 1024^2, q and k RMS-normalised per head.
        _gemm("gemm_qkv_flux1024", 4608, 9216, 3072, rms=6144),
        # The video blocks' FFN input projection with GELU: the largest linear layer.
        _gemm("gemm_ffn_wan14b", 32760, 13824, 5120, epilogue="gelu"),
        # Few rows: the modulation vectors of 28 steps (17 chunks of 3072), bound by the weights' bytes.
        _gemm("gemm_mod_28rows", 28, 52224, 3072, epilogue="f32"),
        # The joint self-attention of a block at 1024^2.
        _attention("attn_joint_flux1024", 4608, 4608, 24, True),
        # The video blocks' cross-attention: many queries, 512 text keys.
        _attention("attn_cross_wan14b", 32760, 512, 40, True),
        # Attention without a bound on the logits, ragged, through the entry point that allocates nothing.
        _attention("attn_general_ragged", 2111, 2111, 16, False, noalloc=True),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v / step) * step)) if v >= step else max(lo, step)


def draw(rng):
    what = rng.random()
    if what < 0.35:
        # linear layers: 1 to 32760 rows, widths of the small and the large models; K mostly a
        # multiple of the 64-deep slice, as every layer width of the workloads is
        M = _log_int(rng, 1, 32760)
        N = _log_int(rng, 64, 21504, 8)
        K = _log_int(rng, 64, 15360, 64 if rng.random() < 0.75 else 8)
        epi = rng.choice(["store", "store", "gelu", "silu", "f32"])
        rms = 0
        if epi == "store" and N >= 384 and rng.random() < 0.5:
            N = N // 384 * 384
            rms = N // 384 * 256
        M = max(1, min(M, int(2.0e12 / (N * K))))
        return _gemm(None, M, N, K, epi, rms)
    if what < 0.65:
        # one image's joint tokens, or queries against a shorter or longer set of keys
        Lq = _log_int(rng, 1, 20000)
        Lk = Lq if rng.random() < 0.5 else _log_int(rng, 1, 20000)
        heads = rng.choice([1, 2, 3, 8, 16, 24, 40])
        most = 2.0e12 / (512 * heads)
        if Lq * Lk > most:
            s = math.sqrt(most / (Lq * Lk))
            Lq, Lk = int(Lq * s), int(Lk * s)
        noalloc = heads * 128 * ((Lk + 63) // 64 * 64) <= binding.NOALLOC_VT_MAX_ELEMS and rng.random() < 0.3
        return _attention(None, Lq, Lk, heads, rng.random() < 0.7, noalloc)
    T = rng.randint(3, 20)
    B = rng.randint(1, T)
    common = dict(policy=rng.choice(["gate", "gate", "static"]), bias=rng.choice([-10.0, 10.0]),
                  solver=rng.choice(["euler", "euler", "unipc"]), shift=rng.choice([1.0, 3.0, 5.0]),
                  prompts=rng.choice([1, 1, 1, 2, 3]))
    batch = rng.choice([1, 1, 2])
    guidance = 4.0 if batch == 2 else 1.0
    if rng.random() < 0.25:
        heads, hd = rng.choice([(4, 32), (3, 64), (2, 128), (6, 64)])
        return _sample(None, "f32", heads, hd, 4 * heads * hd, _log_int(rng, 16, 1024), _log_int(rng, 4, 128), T, B,
                       double=rng.randint(0, 2), single=rng.randint(1, 2), channels=16, ctx=8 * rng.randint(8, 24),
                       batch=batch, guidance=guidance, pooled=rng.random() < 0.5, **common)
    heads = rng.choice([2, 3, 4, 8, 16, 24])
    video = rng.random() < 0.3
    n_img, n_txt = _log_int(rng, 16, 4096), _log_int(rng, 4, 512)
    if rng.random() < 0.4:
        n_img, n_txt = max(32, n_img // 32 * 32), max(32, n_txt // 32 * 32)
    blocks = dict(cross=rng.randint(1, 2)) if video else dict(double=rng.randint(1, 2), single=rng.randint(0, 1))
    return _sample(None, "bf16", heads, 128, 128 * heads * (3 if video else 4), n_img, n_txt, min(T, 8), min(B, 3),
                   channels=rng.choice([64, 64, 64, 32]), ctx=8 * rng.randint(8, 256), batch=batch,
                   guidance=guidance, pooled=not video and rng.random() < 0.5, **blocks, **common)


# ------------------------------------------------------------------ inputs

def _rng(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _layout(c):
    """(name, shape) of the weight blob in the order of include/dit_cache.h."""
    H, F, C, X = c["heads"] * c["head_dim"], c["mlp"], c["channels"], c["ctx"]
    mod = 12 * H * c["double"] + 3 * H * c["single"] + (6 * H if c["cross"] else 0) + 2 * H
    out = []

    def linear(name, n, k):
        out.append((name + ".w", (n, k)))
        out.append((name + ".b", (n,)))

    linear("img_in", H, C)
    linear("txt_in", H, X)
    linear("time0", H, 256)
    linear("time2", H, H)
    if c["pooled"]:
        linear("pool0", H, X)
        linear("pool2", H, H)
    linear("mod", mod, H)
    for i in range(c["double"]):
        for s in ("img", "txt"):
            for name, n, k in (("qkv", 3 * H, H), ("o", H, H), ("up", F, H), ("down", H, F)):
                linear("double%d.%s.%s" % (i, s, name), n, k)
    for i in range(c["single"]):
        linear("single%d.l1" % i, 3 * H + F, H)
        linear("single%d.l2" % i, H, H + F)
    for i in range(c["cross"]):
        out.append(("cross%d.offset" % i, (6 * H,)))
        for name, n, k in (("qkv", 3 * H, H), ("o", H, H), ("xq", H, H), ("xkv", 2 * H, H), ("xo", H, H),
                           ("up", F, H), ("down", H, F)):
            linear("cross%d.%s" % (i, name), n, k)
    linear("final", C, H)
    return out


def _dt(c):
    return torch.bfloat16 if c.get("dtype", "bf16") == "bf16" else torch.float32


MODEL_KEYS = ("dtype", "double", "single", "cross", "heads", "head_dim", "mlp", "channels", "ctx", "pooled")


def _device_weights(c):
    """The model's weights on the GPU, N(0, 0.02^2), flat in blob order: one model whatever the inputs' seed."""
    n = sum(math.prod(s) for _, s in _layout(c))
    flat, g = torch.empty(n, dtype=_dt(c), device=DEV), _rng(20260)
    for lo in range(0, n, 1 << 26):
        part = flat[lo:lo + (1 << 26)]
        part.copy_(0.02 * torch.randn(part.numel(), generator=g, device=DEV))
    return flat


@functools.lru_cache(maxsize=KEPT_BLOBS)
def _host_blob(key):
    flat = _device_weights(dict(zip(MODEL_KEYS, key))).cpu()
    return flat.view(torch.int16).numpy().view(np.uint16) if flat.dtype == torch.bfloat16 else flat.numpy()


def _gate(c):
    """A gate of the workloads' shape (8-32-16-1, N(0, 0.3^2)) that votes clearly
    (its output bias), so that rounding does not move a decision."""
    blob = synth.make_gate_blob(seed=42)
    blob[-1] = c["bias"]
    return blob


def _sample_inputs(c, seed):
    g, S = _rng(seed), c["prompts"]
    x0 = torch.randn(S, c["n_img"], c["channels"], generator=g, device=DEV)
    text = torch.randn(S, c["batch"], c["n_txt"], c["ctx"], generator=g, device=DEV).to(_dt(c))
    return x0, text


def _gemm_inputs(c, seed):
    g = _rng(seed)
    A = torch.randn(c["M"], c["K"], generator=g, device=DEV).bfloat16()
    W = torch.empty(c["N"], c["K"], dtype=torch.bfloat16, device=DEV)
    for lo in range(0, c["N"], 8192):
        W[lo:lo + 8192] = 0.02 * torch.randn(W[lo:lo + 8192].shape, generator=g, device=DEV)
    b = (0.02 * torch.randn(c["N"], generator=g, device=DEV)).bfloat16()
    return A, W, b


def _attention_inputs(c, seed):
    """q [Lq, H] and k, v as they leave a projection: RMS-normalised q and k where the logits are bounded."""
    g, H = _rng(seed), c["heads"] * 128

    def heads(n, norm):
        x = torch.randn(n, H, generator=g, device=DEV)
        if norm:
            x = x.view(n, -1, 128)
            x = (x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6)).view(n, H)
        return x.bfloat16()

    q, k, v = heads(c["Lq"], c["bounded"]), heads(c["Lk"], c["bounded"]), heads(c["Lk"], False)
    return q, k, v


# --------------------------------------------------------------- the calls

def prepare(case, seed):
    c = case
    if c["kind"] == "sample":
        cfg = synth.ModelConfig(
            name="case", dtype=c["dtype"], n_double=c["double"], n_single=c["single"], n_cross=c["cross"],
            hidden=c["heads"] * c["head_dim"], heads=c["heads"], head_dim=c["head_dim"], mlp_hidden=c["mlp"],
            in_channels=c["channels"], ctx_dim=c["ctx"], n_img=c["n_img"], n_txt=c["n_txt"], batch=c["batch"],
            pooled_text=c["pooled"])
        handle = binding.DitCache(cfg, _host_blob(tuple(c[k] for k in MODEL_KEYS)))
        x0, text = _sample_inputs(c, seed)
        return dict(case=c, handle=handle, x0=x0, x=torch.empty_like(x0), text=text, gate=_gate(c))
    if c["kind"] == "gemm":
        A, W, b = _gemm_inputs(c, seed)
        out = torch.empty(c["M"], c["N"], dtype=torch.float32 if c["epilogue"] == "f32" else torch.bfloat16, device=DEV)
        return dict(case=c, A=A, W=W, b=b, out=out)
    q, k, v = _attention_inputs(c, seed)
    H, Lk = c["heads"] * 128, c["Lk"]
    kv = torch.cat([k, v], dim=1)  # one projection's output: k | v
    ws = None if c["noalloc"] else torch.empty(c["heads"] * 128 * ((Lk + 63) // 64 * 64), dtype=torch.bfloat16, device=DEV)
    return dict(case=c, q=q, k=kv[:, :H], v=kv[:, H:], out=torch.empty_like(q), ws=ws)


def run(state):
    c = state["case"]
    if c["kind"] == "sample":
        # the sampler works in place: each pass starts from the drawn latent
        state["x"].copy_(state["x0"])
        args = dict(shift=c["shift"], guidance=c["guidance"], policy=c["policy"], solver=c["solver"])
        if c["prompts"] == 1:
            scheds = [state["handle"].sample(state["x"][0], state["text"][0], state["gate"], c["T"], c["B"], **args)]
        else:
            scheds = state["handle"].sample_batch(state["x"], state["text"], state["gate"], c["T"], c["B"], **args)
        return {"latent": state["x"], "full": np.stack([s.full for s in scheds]),
                "sums": np.stack([s.sums for s in scheds]), "logit": np.stack([s.logit for s in scheds])}
    if c["kind"] == "gemm":
        flags = {"f32": binding.EPI_F32, "silu": binding.EPI_SILU}.get(c["epilogue"], binding.EPI_STORE)
        binding.gemm_bf16(state["A"], state["W"], state["b"], state["out"], M=c["M"], N=c["N"], K=c["K"], flags=flags,
                          rms_cols=c["rms"], gelu_from=0 if c["epilogue"] == "gelu" else None)
        return state["out"]
    H = c["heads"] * 128
    args = dict(Lq=c["Lq"], Lk=c["Lk"], heads=c["heads"], ldq=H, ldk=2 * H, ldv=2 * H, ldo=H,
                flags=binding.ATTN_BOUNDED_LOGITS if c["bounded"] else 0)
    if c["noalloc"]:
        binding.attention_bf16_noalloc(state["q"], state["k"], state["v"], state["out"], **args)
    else:
        binding.attention_bf16(state["q"], state["k"], state["v"], state["out"], vt_ws=state["ws"], **args)
    return state["out"]


# -------------------------------------------------------- work and tolerance

def work(case):
    c = case
    if c["kind"] == "gemm":
        out = 4 if c["epilogue"] == "f32" else 2
        return {"bytes": 2 * (c["M"] * c["K"] + c["N"] * c["K"] + c["N"]) + out * c["M"] * c["N"],
                "flops": 2 * c["M"] * c["N"] * c["K"]}
    if c["kind"] == "attention":
        H = c["heads"] * 128
        return {"bytes": 4 * (c["Lq"] + c["Lk"]) * H, "flops": 4 * c["Lq"] * c["Lk"] * H}
    H, F, N, Nt, C, T, B = c["heads"] * c["head_dim"], c["mlp"], c["n_img"], c["n_txt"], c["channels"], c["T"], c["B"]
    L, seqs, esz = N + Nt, c["batch"] * c["prompts"], 2 if c["dtype"] == "bf16" else 4
    rows = 2 * H * (4 * H + 2 * F)  # linear layers of one token and block: qkv, out and the MLP
    full = (c["double"] + c["single"]) * (L * rows + 4 * L * L * H)
    full += c["cross"] * (N * (rows + 4 * H * H) + 4 * N * N * H + 4 * N * Nt * H)
    weights = {n: math.prod(s) for n, s in _layout(c)}
    tables = seqs if c["pooled"] else 1
    once = 2 * seqs * Nt * (c["ctx"] * H + c["cross"] * 2 * H * H) + 2 * T * (256 * H + H * H)
    once += 2 * tables * T * weights["mod.w"]
    step = 2 * seqs * N * C * H  # the final projection; the patch embedding is one per prompt
    step += 2 * c["prompts"] * N * C * H
    # per step and prompt: m_t written, m_{t-1} and m_last read, each branch's residual read or written
    state = c["prompts"] * T * N * H * esz * (3 + c["batch"])
    return {"bytes": sum(weights.values()) * esz + state + seqs * Nt * c["ctx"] * esz + 8 * c["prompts"] * N * C,
            "flops": B * seqs * full + once + T * step}


def tolerance(case):
    """About four times the distance from ``exact`` that was measured: one bf16 rounding of each
    output (1.7e-3; 2.3e-3 where the probabilities are rounded too), 3e-7 to 7e-7 for f32 sums of
    a layer, 5.4e-3 for the latents of a bf16 guidance pair and 1.7e-7 for those of an f32 model."""
    if case["kind"] == "gemm":
        return {"rel": 3e-6} if case["epilogue"] == "f32" else {"rel": 7e-3}
    if case["kind"] == "attention":
        return {"rel": 1e-2}
    return {"rel": 1e-6} if case["dtype"] == "f32" else {"rel": 2e-2}


# ------------------------------------------------------- 64-bit evaluation

def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _silu(x):
    return x * torch.sigmoid(x)


def _rms(x, hd):
    h = x.view(x.shape[0], -1, hd)
    return (h * torch.rsqrt(h.square().mean(-1, keepdim=True) + 1e-6)).reshape(x.shape)


def _ln(x):
    x = x - x.mean(-1, keepdim=True)
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6)


def _softmax_attention(q, k, v, hd):
    out = torch.empty_like(q)
    rows = max(1, (1 << 29) // k.shape[0])
    for h in range(q.shape[1] // hd):
        s = slice(h * hd, (h + 1) * hd)
        kh, vh = k[:, s].T.contiguous(), v[:, s].contiguous()
        for lo in range(0, q.shape[0], rows):
            p = torch.softmax(q[lo:lo + rows, s] @ kh / math.sqrt(hd), dim=1)
            out[lo:lo + rows, s] = p @ vh
    return out


def _exact_gemm(c, seed):
    A, W, b = _gemm_inputs(c, seed)
    y = A.double() @ W.double().T + b.double()
    if c["rms"]:
        y[:, :c["rms"]] = _rms(y[:, :c["rms"]].contiguous(), 128)
    return {"gelu": _gelu, "silu": _silu}.get(c["epilogue"], lambda t: t)(y)


def _exact_gate(blob, f):
    u, p = np.asarray(f, np.float64), 6
    blob = blob.astype(np.float64)
    for n, k in ((32, 8), (16, 32), (1, 16)):
        u = blob[p:p + n * k].reshape(n, k) @ u + blob[p + n * k:p + n * k + n]
        p += n * k + n
        u = np.maximum(u, 0.0) if n > 1 else u
    return float(u[0])


def _stack(c, W, h, txt, mod):
    """Block stack on one sequence: image rows out."""
    H, hd = c["heads"] * c["head_dim"], c["head_dim"]

    def lin(x, n):
        return x @ W[n + ".w"].T + W[n + ".b"]

    def qkv(y):
        return _rms(y[:, :H].contiguous(), hd), _rms(y[:, H:2 * H].contiguous(), hd), y[:, 2 * H:3 * H]

    if c["cross"]:
        for i in range(c["cross"]):
            p = "cross%d." % i
            sh1, sc1, g1, sh2, sc2, g2 = (mod[:6 * H] + W[p + "offset"]).view(6, H)
            q, k, v = qkv(lin(_ln(h) * (1 + sc1) + sh1, p + "qkv"))
            h = h + g1 * lin(_softmax_attention(q, k, v, hd), p + "o")
            q, kv = _rms(lin(_ln(h), p + "xq"), hd), lin(txt, p + "xkv")
            h = h + lin(_softmax_attention(q, _rms(kv[:, :H].contiguous(), hd), kv[:, H:], hd), p + "xo")
            h = h + g2 * lin(_gelu(lin(_ln(h) * (1 + sc2) + sh2, p + "up")), p + "down")
        return h
    nt, off, s = txt.shape[0], 0, {"img": h, "txt": txt}
    for i in range(c["double"]):
        m = {"img": mod[off:off + 6 * H].view(6, H), "txt": mod[off + 6 * H:off + 12 * H].view(6, H)}
        off += 12 * H
        a = [qkv(lin(_ln(s[n]) * (1 + m[n][1]) + m[n][0], "double%d.%s.qkv" % (i, n))) for n in ("txt", "img")]
        o = _softmax_attention(*(torch.cat(t) for t in zip(*a)), hd)
        for n, part in (("txt", o[:nt]), ("img", o[nt:])):
            p = "double%d.%s." % (i, n)
            s[n] = s[n] + m[n][2] * lin(part, p + "o")
            s[n] = s[n] + m[n][5] * lin(_gelu(lin(_ln(s[n]) * (1 + m[n][4]) + m[n][3], p + "up")), p + "down")
    x = torch.cat([s["txt"], s["img"]])
    for i in range(c["single"]):
        sh, sc, g = mod[off:off + 3 * H].view(3, H)
        off += 3 * H
        y = lin(_ln(x) * (1 + sc) + sh, "single%d.l1" % i)
        o = _softmax_attention(*qkv(y), hd)
        x = x + g * lin(torch.cat([o, _gelu(y[:, 3 * H:])], 1), "single%d.l2" % i)
    return x[nt:]


def _unipc(sig, T):
    """Step rule x, m-history -> x of UniPC-2 with B(h) = e^h - 1 on x - sigma v."""
    def lam(s):
        return -math.inf if s >= 1 else math.inf if s <= 0 else math.log((1 - s) / s)

    def terms(s, t):
        h = lam(t) - lam(s)
        if math.isinf(h):
            return h, -1.0, 1.0, 1.0
        e = math.expm1(-h)
        p1 = -e / h - 1
        p2 = -p1 / h - 0.5
        return h, e, p1 / e, 2 * p2 / e

    def order(i):
        return min(2, i + 1, T - i)

    def back(p, s, h):
        return -math.inf if math.isinf(lam(p)) or math.isinf(h) else (lam(p) - lam(s)) / h

    hist, last = [], [None]

    def step(t, x, v):
        m = x - sig[t] * v
        if t:
            h, e, b1, b2 = terms(sig[t - 1], sig[t])
            ms, a = hist[-1], 1 - sig[t]
            y = sig[t] / sig[t - 1] * last[0] - a * e * ms
            r = back(sig[t - 2], sig[t - 1], h) if order(t - 1) == 2 else -math.inf
            if order(t - 1) == 1:
                x = y - a * e * 0.5 * (m - ms)
            elif math.isinf(r):
                x = y - a * e * b1 * (m - ms)
            else:
                r1 = (b1 - b2) / (1 - r)
                x = y - a * e * (r1 * (hist[-2] - ms) / r + (b1 - r1) * (m - ms))
        hist.append(m)
        last[0] = x
        h, e, _, _ = terms(sig[t], sig[t + 1])
        y = sig[t + 1] / sig[t] * x - (1 - sig[t + 1]) * e * m
        if order(t) == 2:
            r = back(sig[t - 1], sig[t], h)
            if not math.isinf(r):
                y = y - (1 - sig[t + 1]) * e * 0.5 * (hist[-2] - m) / r
        return y

    return step


def _exact_prompt(c, W, gate, x, text):
    H, T, B, nb = c["heads"] * c["head_dim"], c["T"], c["B"], c["batch"]
    sig = [c["shift"] * u / (1 + (c["shift"] - 1) * u) for u in (1 - i / T for i in range(T + 1))]

    def lin(v, n):
        return v @ W[n + ".w"].T + W[n + ".b"]

    f = torch.exp(-math.log(10000.0) * torch.arange(128, dtype=torch.float64, device=DEV) / 128)
    a = 1000.0 * torch.tensor(sig[:T], dtype=torch.float64, device=DEV)[:, None] * f
    tv = lin(_silu(lin(torch.cat([a.cos(), a.sin()], 1), "time0")), "time2")
    mods = []
    for b in range(nb):
        v = tv + lin(_silu(lin(text[b].mean(0, keepdim=True), "pool0")), "pool2") if c["pooled"] else tv
        mods.append(lin(_silu(v), "mod"))
    txt = [lin(text[b], "txt_in") for b in range(nb)]
    first = W["cross0.offset"][:2 * H] if c["cross"] else 0.0
    full, sums, logit = np.zeros(T, np.uint8), np.full((T, 4), np.nan), np.full(T, np.nan)
    static = {i * T // B for i in range(B)}
    rule = _unipc(sig, T) if c["solver"] == "unipc" else lambda t, x, v: x + (sig[t + 1] - sig[t]) * v
    cnt, at, acc, prev, comp, res = 0, 0, 0.0, None, None, [None] * nb
    for t in range(T):
        h = lin(x, "img_in")
        sh, sc = (mods[0][t, :2 * H] + first).view(2, H)
        m = _ln(h) * (1 + sc) + sh
        dec = 1
        if t:
            sums[t] = [float(s) for s in ((m - prev).abs().sum(), prev.abs().sum(), (m - comp).abs().sum(), comp.abs().sum())]
            dp, dl = sums[t][0] / sums[t][1], sums[t][2] / sums[t][3]
            acc += dp
            if c["policy"] == "gate":
                z = _exact_gate(gate, [B / T, (B - cnt) / B, (B - cnt) / (T - t), t - at, dl, dp, t / T, acc])
                logit[t] = z
                dec = 0 if cnt == B else 1 if B - cnt >= T - t else int(z > 0)
            else:
                dec = int(t in static)
        full[t], prev = dec, m
        v = []
        for b in range(nb):
            if dec:
                res[b] = _stack(c, W, h, txt[b], mods[b][t]) - h
            sf, cf = mods[b][t, -2 * H:].view(2, H)
            v.append(lin(_ln(h + res[b]) * (1 + cf) + sf, "final"))
        if dec:
            cnt, at, acc, comp = cnt + 1, t, 0.0, m
        x = rule(t, x, v[0] if nb == 1 else v[1] + c["guidance"] * (v[0] - v[1]))
    return x, full, sums, logit


def exact(case, seed):
    c = case
    if c["kind"] == "gemm":
        return _exact_gemm(c, seed)
    if c["kind"] == "attention":
        return _softmax_attention(*(t.double() for t in _attention_inputs(c, seed)), 128)
    flat, W, at = _device_weights(c), {}, 0
    for name, shape in _layout(c):
        n = math.prod(shape)
        W[name] = flat[at:at + n].view(shape).double()
        at += n
    x0, text = _sample_inputs(c, seed)
    got = [_exact_prompt(c, W, _gate(c), x0[j].double(), text[j].double()) for j in range(c["prompts"])]
    return {"latent": torch.stack([g[0] for g in got]), "full": np.stack([g[1] for g in got]),
            "sums": np.stack([g[2] for g in got]), "logit": np.stack([g[3] for g in got])}
