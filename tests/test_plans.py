"""The size rules on the host (no GPU): the shapes that the GPU tests of the
shared last rounds and of the small attention kernel use do reach them."""
import random

import pytest

from tests import _plans
from tests.test_gpu_kernels import LAST_ROUND_ATTENTION, LAST_ROUND_GEMMS, SMALL_ATTENTION
from tests.test_gpu_sampler import SHARED_PAIR, STRADDLING_PAIR


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _plans.build(str(tmp_path_factory.mktemp("plans")))


@pytest.mark.parametrize("M,N,K,flags", LAST_ROUND_GEMMS)
def test_last_round_gemms_are_shared(lib, M, N, K, flags):
    kw = dict(rms=2048, gelu_from=3072, gap_at=3072, gap=512) if flags == 0 else {}
    assert _plans.gemm_shares(lib, [(M, N, K)], flags, **kw)
    assert not _plans.gemm_shares(lib, [(M, N, K)], flags, one_chain=1, **kw)


@pytest.mark.parametrize("Lq,Lk,heads,full,straddles", LAST_ROUND_ATTENTION)
def test_last_round_attention_is_shared(lib, Lq, Lk, heads, full, straddles):
    assert not lib.attention_small(Lq, Lk, heads, 1)
    p = _plans.AttentionPlan(Lq, Lk, heads)
    assert p.full == full
    if straddles is None:   # a last round of whole items
        assert p.rem and not p.shares and not lib.attention_shares(Lq, Lk, heads, 1)
    else:
        assert lib.attention_shares(Lq, Lk, heads, 1) and p.shares and bool(p.straddling) == straddles


@pytest.mark.parametrize("Lq,Lk,heads", SMALL_ATTENTION)
def test_small_attention_is_taken(lib, Lq, Lk, heads):
    assert lib.attention_small(Lq, Lk, heads, 1)


def test_attention_plan_matches_the_library(lib):
    rng = random.Random(5)
    seen = {True: 0, False: 0}
    for _ in range(4000):
        Lq, Lk = int(2 ** rng.uniform(0, 15)), int(2 ** rng.uniform(0, 15))
        heads, nseq = rng.randint(1, 48), rng.choice([1, 1, 2, 3, 8])
        got = bool(lib.attention_shares(Lq, Lk, heads, nseq))
        assert got == _plans.AttentionPlan(Lq, Lk, heads, nseq).shares, (Lq, Lk, heads, nseq)
        seen[got] += 1
    assert min(seen.values()) > 400


def test_sampler_cases_reach_the_shared_rounds(lib):
    H, F, N, Nt = (SHARED_PAIR[k] for k in ("hidden", "mlp_hidden", "n_img", "n_txt"))
    for K in (H, F):   # both branches' image rows and text rows, a gate vector per branch
        assert _plans.gemm_shares(lib, [(2 * N, H, K), (2 * Nt, H, K)], flags=2, gseg=2)
    L, heads, Nt = STRADDLING_PAIR["n_img"] + STRADDLING_PAIR["n_txt"], STRADDLING_PAIR["heads"], STRADDLING_PAIR["n_txt"]
    assert Nt % _plans.KT and not lib.attention_small(L, L, heads, 2) and lib.attention_shares(L, L, heads, 2)


def test_one_chain_never_shares(lib):
    """Stacked launches of several prompts: no shape of theirs is shared."""
    rng = random.Random(6)
    shared = 0
    for _ in range(3000):
        M, N, K = rng.randint(1, 20000), 8 * rng.randint(8, 3000), 64 * rng.randint(1, 240)
        M = min(M, int(2e9 / K))
        assert not _plans.gemm_shares(lib, [(M, N, K)], one_chain=1)
        shared += _plans.gemm_shares(lib, [(M, N, K)])
    assert shared > 100
