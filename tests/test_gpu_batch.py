"""Multi-prompt sampling (dit_cache_sample_batch): S samples in lockstep,
each with its own schedule, the computing ones' block stacks stacked into
shared launches.  Every sample is checked against the oracle run on that
sample alone (the problem is posed per prompt), under the same bar as the
single-sample parity tests, and against the library's own single-sample
path on the same inputs."""
import numpy as np
import pytest

from oracle import sample as oracle_sample
from paper_2608_09231_amd import binding, synth
from tests._gpu import check_logits, check_schedule_against_oracle, dev, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}
# stacked launches may pick other GEMM tiles than a lone sequence: same
# products, but e.g. the per-head RMS sum of squares in another order
SELF_TOL = {"f32": 1e-6, "bf16": 5e-3}

# Replay masks (T = 8, B = 4) whose per-step computing sets include all
# samples (t = 0), none (t = 6), a non-contiguous subset of three ({0, 1, 3},
# t = 1: gathered modulation vectors), an evenly spaced pair ({0, 2}, t = 5)
# and single samples.
MASKS = np.array([[1, 1, 0, 1, 0, 1, 0, 0],
                  [1, 1, 1, 0, 0, 0, 0, 1],
                  [1, 0, 1, 0, 1, 1, 0, 0],
                  [1, 1, 0, 0, 1, 0, 0, 1]], np.uint8)


def inputs(w, S):
    cfg = w.model
    weights, _, _, gate = synth.make_inputs(w)
    x0 = np.stack([synth.make_latent(cfg, w.seed + 101 * j) for j in range(S)])
    text = np.stack([synth.make_text(cfg, w.seed + 211 * j + 1) for j in range(S)])
    return weights, x0, text, gate


def run_batch(torch, h, w, x0, text, gate, T, B, **kw):
    lat = dev(torch, x0.astype(np.float32))
    txt = dev(torch, text)
    scheds = h.sample_batch(lat, txt, gate, T, B, shift=w.shift, guidance=w.guidance, **kw)
    torch.cuda.synchronize()
    return lat.cpu().numpy().astype(np.float64), scheds


def run_one(torch, h, w, x0, text, gate, T, B, **kw):
    lat = dev(torch, x0.astype(np.float32))
    txt = dev(torch, text)
    sched = h.sample(lat, txt, gate, T, B, shift=w.shift, guidance=w.guidance, **kw)
    torch.cuda.synchronize()
    return lat.cpu().numpy().astype(np.float64), sched


def check_batch(name, S, *, masks=None, solver="euler", T=None, B=None, gate=None):
    torch = torch_cuda()
    w = synth.workload(name)
    cfg = w.model
    T = T or w.T
    B = B or w.B
    weights, x0, text, wgate = inputs(w, S)
    gate = wgate if gate is None else gate
    h = binding.DitCache(cfg, weights.blob)
    try:
        xb, scheds = run_batch(torch, h, w, x0, text, gate, T, B, forced_masks=masks, solver=solver)
        singles = [run_one(torch, h, w, x0[j], text[j], gate, T, B, forced_mask=scheds[j].full, solver=solver)
                   for j in range(S)]
    finally:
        h.close()
    for j, s in enumerate(scheds):
        assert s.nfe == B and int(s.full.sum()) == B and s.full[0] == 1 and s.steps_done == T
        if masks is not None:
            np.testing.assert_array_equal(s.full, masks[j])
        ores = oracle_sample(cfg, weights.tensors, gate, x0[j], text[j], T, B, shift=w.shift,
                             guidance=w.guidance, forced_mask=s.full, solver=solver)
        if masks is None:
            check_schedule_against_oracle(s, ores)
        check_logits(s, ores, gate, 1e-5 if cfg.dtype == "f32" else None)
        err = rel_l2(xb[j], ores.x)
        assert err <= TOL[cfg.dtype], (j, err)
        xs, ss = singles[j]
        np.testing.assert_array_equal(ss.full, s.full)
        assert rel_l2(xb[j], xs) <= SELF_TOL[cfg.dtype], (j, rel_l2(xb[j], xs))
        np.testing.assert_allclose(s.features[1:, :4], ss.features[1:, :4], rtol=1e-12)
    return scheds


@pytest.mark.parametrize("name", ["tiny", "small_bf16", "small_seg_bf16", "small_cfg_bf16", "small_cross_bf16"])
def test_batch_replay_masks(name):
    check_batch(name, 4, masks=MASKS, T=8, B=4)


@pytest.mark.parametrize("name", ["small_bf16", "small_seg_bf16", "small_cfg_bf16"])
def test_batch_gated(name):
    check_batch(name, 3)


def test_batch_flip_gate():
    """A gate whose vote changes sign within a run: each prompt's lane paces
    its own budget, so the prompts' schedules are checked one by one."""
    from tests.test_gpu_sampler import FLIP, flip_gate
    case = FLIP["cases"]["small_bf16_833"]
    scheds = check_batch("small_bf16", 3, gate=flip_gate(case), T=case["T"], B=case["B"])
    print("flip-gate batch schedules", [s.full.tolist() for s in scheds])


def test_batch_unipc():
    check_batch("small_cfg_bf16", 3, solver="unipc")


def test_batch_sizes_on_one_handle():
    """Workspace grows with the batch and is reused by smaller ones: results
    do not depend on what the handle ran before."""
    torch = torch_cuda()
    w = synth.workload("small_seg_bf16")
    weights, x0, text, gate = inputs(w, 3)
    h = binding.DitCache(w.model, weights.blob)
    try:
        x1, s1 = run_one(torch, h, w, x0[0], text[0], gate, w.T, w.B)
        x3, s3 = run_batch(torch, h, w, x0, text, gate, w.T, w.B)
        fm = np.stack([s3[0].full, s3[1].full])
        x2, s2 = run_batch(torch, h, w, x0[:2], text[:2], gate, w.T, w.B, forced_masks=fm)
        x1b, s1b = run_one(torch, h, w, x0[0], text[0], gate, w.T, w.B)
    finally:
        h.close()
    np.testing.assert_array_equal(x1, x1b)
    np.testing.assert_array_equal(s1.full, s1b.full)
    for j in range(2):
        assert rel_l2(x2[j], x3[j]) <= SELF_TOL["bf16"]
        np.testing.assert_array_equal(s2[j].sums[1:2], s3[j].sums[1:2])


def test_shared_last_round_on_one_handle(monkeypatch):
    """The same where a lone prompt's widest layer (four tile rows of 91, 108
    tiles past the whole round in two shares of K) is shared out and nothing
    else of the model is."""
    torch = torch_cuda()
    cfg = synth.ModelConfig(name="case", dtype="bf16", n_double=0, n_single=1, n_cross=0, hidden=3328, heads=26,
                            head_dim=128, mlp_hidden=13312, in_channels=64, ctx_dim=96, n_img=720, n_txt=80)
    monkeypatch.setitem(synth.WORKLOADS, "case", synth.Workload("case", cfg, T=2, B=1, shift=3.0, guidance=1.0, seed=43))
    w = synth.workload("case")
    weights, x0, text, gate = inputs(w, 2)
    h = binding.DitCache(cfg, weights.blob)
    try:
        x1, s1 = run_one(torch, h, w, x0[0], text[0], gate, w.T, w.B)
        run_batch(torch, h, w, x0, text, gate, w.T, w.B)
        x1b, s1b = run_one(torch, h, w, x0[0], text[0], gate, w.T, w.B)
    finally:
        h.close()
    np.testing.assert_array_equal(x1, x1b)
    np.testing.assert_array_equal(s1.sums[1:], s1b.sums[1:])


def test_shared_last_round_of_a_pair(monkeypatch):
    """A guidance pair's gated layers in shares of K against the same pair in
    a call over two prompts, which runs whole tiles: the rows that the shares
    hold by themselves (a gate vector of the other branch there moves them by
    2e-2 in the first gated layer and 7e-2 in the second, from the oracle)."""
    from tests.test_gpu_sampler import SHARED_PAIR
    torch = torch_cuda()
    cfg = synth.ModelConfig(name="case", dtype="bf16", n_cross=0, head_dim=128, in_channels=64, ctx_dim=96, batch=2,
                            **SHARED_PAIR)
    monkeypatch.setitem(synth.WORKLOADS, "case", synth.Workload("case", cfg, T=2, B=1, shift=3.0, guidance=4.0, seed=37))
    w = synth.workload("case")
    weights, x0, text, gate = inputs(w, 2)
    h = binding.DitCache(cfg, weights.blob)
    try:
        x1, _ = run_one(torch, h, w, x0[0], text[0], gate, 2, 1)
        x2, _ = run_batch(torch, h, w, x0, text, gate, 2, 1)
    finally:
        h.close()
    assert not np.array_equal(x1, x2[0])
    print("pair, shared against whole:", rel_l2(x1, x2[0]), rel_l2(x1[-512:], x2[0][-512:]))
    assert rel_l2(x1[-512:], x2[0][-512:]) <= SELF_TOL["bf16"]
    assert rel_l2(x1, x2[0]) <= SELF_TOL["bf16"]


# Prompt 0 computes at t = 0 and t = 1; beside it at t = 1: all, two, one and none of the others.
NEIGHBOURS = [np.array([[1, 1, 0]] * (1 + k) + [[1, 0, 1]] * (3 - k), np.uint8) for k in (3, 2, 1, 0)]


@pytest.mark.parametrize("dims", [
    # small kernels' sizes, ragged rows and keys
    dict(heads=2, mlp_hidden=1024, n_img=200, n_txt=40, n_double=2, n_single=2),
    # 272 tiles of 256 x 256 and K = 5120 where four compute: a last round that one prompt would share out
    dict(heads=8, mlp_hidden=4096, n_img=4096, n_txt=256, n_double=0, n_single=1),
])
@pytest.mark.parametrize("pooled", [1, 0])
def test_batch_bits_do_not_depend_on_neighbours(monkeypatch, dims, pooled):
    """A prompt's latent and indicator sums are the same bits whatever the
    other prompts of the call decide at each step."""
    torch = torch_cuda()
    cfg = synth.ModelConfig(name="case", dtype="bf16", n_cross=0, hidden=128 * dims["heads"], head_dim=128,
                            in_channels=64, ctx_dim=96, batch=1, pooled_text=pooled, **dims)
    monkeypatch.setitem(synth.WORKLOADS, "case", synth.Workload("case", cfg, T=3, B=2, shift=3.0, guidance=1.0, seed=41))
    w = synth.workload("case")
    weights, x0, text, gate = inputs(w, 4)
    h = binding.DitCache(cfg, weights.blob)
    try:
        runs = [run_batch(torch, h, w, x0, text, gate, 3, 2, forced_masks=m) for m in NEIGHBOURS]
    finally:
        h.close()
    x, s = runs[0]
    for xn, sn in runs[1:]:
        np.testing.assert_array_equal(xn[0], x[0])
        np.testing.assert_array_equal(sn[0].sums[1:], s[0].sums[1:])


def test_batch_error_paths():
    torch = torch_cuda()
    w = synth.workload("small_bf16")
    weights, x0, text, gate = inputs(w, 2)
    h = binding.DitCache(w.model, weights.blob)
    try:
        lat = dev(torch, x0.astype(np.float32))
        txt = dev(torch, text)
        with pytest.raises(ValueError):
            h.sample_batch(lat, txt, gate, 8, 4, forced_masks=MASKS[:1])
        bad = MASKS[:2].copy()
        bad[1, 0] = 0
        with pytest.raises(binding.DitError) as e:
            h.sample_batch(lat, txt, gate, 8, 4, forced_masks=bad)
        assert e.value.status == binding.DIT_EINVAL
        lat[1, 5, 3] = float("nan")
        with pytest.raises(binding.DitError) as e:
            h.sample_batch(lat, txt, gate, 8, 4)
        assert e.value.status == binding.DIT_ENONFINITE
        assert "sample 1" in str(e.value)
        assert all(s.steps_done == 1 for s in e.value.schedule)
    finally:
        h.close()
