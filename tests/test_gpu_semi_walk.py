"""The semi-Markov walks over the segment potentials: every lane layout at its edge sizes, inputs
outside the linear range (walked again in float64 logarithms), sequences without any allowed
segmentation, and the lengths where the Viterbi walk hands over to the expanded chain.  Against
the float64 oracle, and against the expanded chain (TS_PATH=tree)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say
from paper_2002_00876_amd import binding, workloads as W

pytestmark = pytest.mark.gpu


def _call(sp, lens):
    tsp = torch.from_numpy(np.ascontiguousarray(sp)).cuda()
    tl = torch.from_numpy(np.ascontiguousarray(lens)).cuda()
    z = binding.semi_logpartition(tsp, tl)
    z2, m = binding.semi_marginals(tsp, tl)
    path, seglen, score = binding.semi_viterbi(tsp, tl)
    return [x.cpu().numpy() for x in (z, z2, m, path, seglen, score)]


def _check(sp, lens, tag, against_chain=None):
    # float32 results of float32 inputs: log Z and score to 1e-5 of max(|value|, 1), marginals
    # to 1e-5, as everywhere; paths exactly
    say(f"semi walk {tag}: {sp.shape}")
    z, z2, m, path, seglen, score = _call(sp, lens)
    if against_chain is None:
        zo, mo = oracle.semi_marginals(sp, lens)
        po, go, so = oracle.semi_viterbi(sp, lens)
    else:
        against_chain.setenv("TS_PATH", "tree")
        zo, _, mo, po, go, so = _call(sp, lens)
        against_chain.delenv("TS_PATH")
    ok = np.isfinite(zo)
    for got in (z, z2):
        assert np.array_equal(np.isfinite(got), ok)
        np.testing.assert_allclose(got[ok], zo[ok], rtol=1e-5, atol=1e-5)
    # (without any allowed segmentation the marginals have no reference)
    assert np.abs(m[ok] - mo[ok]).max(initial=0.0) <= 1e-5
    fin = np.isfinite(so)
    assert np.array_equal(np.isfinite(score), fin)
    np.testing.assert_allclose(score[fin], so[fin], rtol=1e-5, atol=1e-5)
    keep = slice(None) if against_chain else fin
    assert np.array_equal(path[keep], po[keep]) and np.array_equal(seglen[keep], go[keep])


def _ragged(seed, B, N, K, C, kind="normal"):
    sp, _ = W.semi_case(seed, B, N, K, C, kind=kind)
    return sp, np.array([N, N - 1, 2, 1, max(N // 2, 1), max(N - 2, 1)][:B], np.int32)


@pytest.mark.parametrize("K,C", [(40, 1), (64, 1), (65, 1), (256, 1), (17, 2), (4, 9), (4, 16),
                                 (16, 16), (2, 17), (2, 32), (3, 32), (8, 32), (2, 33), (3, 63),
                                 (4, 64), (3, 65), (2, 127), (2, 128)])
@pytest.mark.parametrize("kind", ["normal", "int"])
def test_layouts(K, C, kind):
    sp, lens = _ragged(50 + K * C, 6, 14, K, C, kind)
    _check(sp, lens, f"layout K={K} C={C} {kind}")


@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 7, 8, 9, 10])
def test_short(N):
    sp, lens = _ragged(400 + N, 6, N, 5, 9)
    _check(sp, lens, f"N={N}")


@pytest.mark.parametrize("K,C", [(5, 20), (2, 90)])
def test_outside_the_linear_range(K, C):
    rng = np.random.default_rng(500 + C)
    sp, lens = _ragged(500 + C, 5, 16, K, C)
    sp[0] *= 30                                    # large scores
    sp[1] -= 40                                    # a common offset
    sp[4][rng.random(sp[4].shape) < 0.3] = -1e4    # soft masks
    _check(sp, lens, "wide")


@pytest.mark.parametrize("K,C", [(5, 20), (5, 8)])
def test_forbidden_entries(K, C, monkeypatch):
    rng = np.random.default_rng(600 + C)
    sp, lens = _ragged(600 + C, 5, 18, K, C)
    sp[rng.random(sp.shape) < 0.5] = -np.inf
    sp[0, 7:12] = -np.inf                           # no segmentation at all
    sp[1, :, :, :, 1:] = -np.inf                    # label 0 only
    _check(sp, lens, "forbidden")
    _check(sp, lens, "forbidden, against the chain", monkeypatch)


@pytest.mark.parametrize("N", [80, 81, 82])
def test_longest_viterbi_walk(N):
    # 80 steps of 256 states are the most backpointers kept in LDS
    sp, _ = W.semi_case(700 + N, 24, N, 8, 32)
    _check(sp, np.arange(N, N - 24, -1).astype(np.int32), f"N={N}")


@pytest.mark.parametrize("K,C,N", [(9, 20, 300), (10, 20, 300), (12, 20, 200), (64, 1, 400)])
def test_long_segments(K, C, N):
    # the expanded chain with and without recursions before the tree
    sp, _ = W.semi_case(900 + K, 2, N, K, C)
    _check(sp, np.array([N, N - 41], np.int32), f"long segments K={K}")
