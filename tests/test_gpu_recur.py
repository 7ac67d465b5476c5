"""Parity of the chunked vector recursions (several chunks per sequence) with the float64
oracle: every lane layout at its edge label counts, chains that forget their start quickly,
slowly, or never (the sequences that the tree has to compute), ties, -inf structure and
ragged lengths."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_all, check_logz, say
from paper_2002_00876_amd import binding, workloads as W

pytestmark = pytest.mark.gpu

# every layout: rows of 16-byte loads (C a multiple of 4) and of single entries, at the largest
# and smallest label counts of each
LABELS = [2, 7, 20, 31, 32, 33, 36, 63, 64, 65, 68, 95, 96, 97, 100, 127, 128, 129, 132, 191, 192,
          193, 196, 255, 256]


@pytest.mark.parametrize("C", LABELS)
def test_layouts(C):
    N = 390 if C > 32 else 700
    pot, lens = W.random_case(31000 + C, 4, N, C, sigma=1.0,
                              lengths=[N, N - 1, N // 2 + 1, 2])
    check_all(pot, lens, f"layout C={C}")


@pytest.mark.parametrize("C", [36, 50, 100, 101, 200])
def test_integer_ties(C):
    pot, lens = W.random_case(32000 + C, 3, 400, C, kind="int", int_range=1,
                              lengths=[400, 257, 130])
    check_all(pot, lens, f"ties C={C}")


def _check_viterbi(pot, lens, tag):
    say(f"viterbi {tag}: {pot.shape}")
    tl = torch.from_numpy(lens).cuda()
    path, score = binding.viterbi(torch.from_numpy(pot).cuda(), tl)
    po, so = oracle.viterbi(pot, lens)
    assert np.array_equal(path.cpu().numpy(), po)
    check_logz(score.cpu().numpy(), so, "score")


# The masks leave the best path alone, so that path and score are those of the other entries,
# which add exactly in float64; -FLT_MAX sums stay finite there.
MASKS = [-1e9, -1e12, -1e20, -1e30, float(np.finfo(np.float32).min)]


@pytest.mark.parametrize("mask", MASKS)
@pytest.mark.parametrize("C,N", [(12, 900), (24, 900), (36, 400), (40, 331), (75, 400), (101, 400),
                                 (128, 600), (131, 300), (256, 300)])
def test_large_masks(C, N, mask):
    rng = np.random.default_rng(38000 + C)
    pot = rng.standard_normal((4, N - 1, C, C)).astype(np.float32)
    pot[0, :, :, 0] = mask                                       # one label, every edge
    pot[1, ::3, :, C - 1] = mask                                 # one label, some edges
    pot[2][rng.random(pot[2].shape) < 0.2] = mask                # random entries
    pot[3, :, :, 0], pot[3, :, 1, :] = mask, 2 * mask if mask > -1e38 else mask
    _check_viterbi(pot, np.array([N, N - 1, N, N - 3], np.int32), f"mask {mask:g}")


@pytest.mark.parametrize("mask", MASKS[1:])
@pytest.mark.parametrize("C,N", [(24, 900), (75, 400), (128, 600), (129, 1000), (256, 300)])
def test_masks_on_every_path(C, N, mask):
    # one edge (in a middle chunk, in the last) masked whole: past it float64 holds the scores to
    # the mask's last bit only, and decisions are those of sums from the sequence's start
    pot = np.random.default_rng(38500 + C).integers(-4, 5, (3, N - 1, C, C)).astype(np.float32)
    mask = np.float32(-2.0 ** round(np.log2(-mask))) if mask > -1e38 else np.float32(mask)
    pot[0, N // 2] = mask
    pot[1, N - 3] = mask
    _check_viterbi(pot, np.array([N, N, N - 20], np.int32), f"masked edge {mask:g}")


@pytest.mark.parametrize("mask", [-1e9, -1e20, -1e30])
def test_large_masks_semi_markov(mask):
    # long enough for the expanded chain
    sp, lens = W.semi_case(38800, 3, 500, 4, 12)
    sp[0, :, :, :, 0] = mask
    sp[1, ::2, 1, 3, :] = mask
    assert 499 * 4 * 12 > 20480
    tl = torch.from_numpy(lens).cuda()
    path, seglen, score = binding.semi_viterbi(torch.from_numpy(sp).cuda(), tl)
    po, go, so = oracle.semi_viterbi(sp, lens)
    assert np.array_equal(path.cpu().numpy(), po) and np.array_equal(seglen.cpu().numpy(), go)
    check_logz(score.cpu().numpy(), so, "score")


def _sticky(seed, B, N, C, stay):
    # labels keep themselves with a bonus: the chain remembers its start for long
    rng = np.random.default_rng(seed)
    pot = rng.standard_normal((B, N - 1, C, C)).astype(np.float32)
    pot += np.float32(stay) * np.eye(C, dtype=np.float32)
    return pot, np.array([N, N - 70, 1][:B], np.int32)


@pytest.mark.parametrize("C,stay", [(40, 6.0), (40, 12.0), (101, 8.0), (128, 14.0), (200, 9.0)])
def test_slow_mixing(C, stay):
    pot, lens = _sticky(33000 + C, 3, 500, C, stay)
    check_all(pot, lens, f"sticky C={C} stay={stay}")


@pytest.mark.parametrize("C", [40, 70, 128])
def test_never_mixing(C):
    # two label sets without transitions between them: the walks never agree
    rng = np.random.default_rng(34000 + C)
    pot = rng.standard_normal((3, 330, C, C)).astype(np.float32)
    pot[1:, :, :C // 2, C // 2:] = -np.inf
    pot[1:, :, C // 2:, :C // 2] = -np.inf
    check_all(pot, np.array([331, 331, 200], np.int32), f"two components C={C}")


@pytest.mark.parametrize("C", [48, 65, 256])
def test_left_to_right_structure(C):
    # label i reaches labels i .. i + 3 only
    rng = np.random.default_rng(35000 + C)
    pot = rng.standard_normal((2, 300, C, C)).astype(np.float32)
    i, j = np.indices((C, C))
    pot[:, :, (j < i) | (j > i + 3)] = -np.inf
    check_all(pot, np.array([301, 150], np.int32), f"left to right C={C}")


@pytest.mark.parametrize("C", [36, 129])
def test_no_finite_path_in_a_later_chunk(C):
    rng = np.random.default_rng(36000 + C)
    pot = rng.standard_normal((3, 400, C, C)).astype(np.float32)
    pot[1, 190] = -np.inf                       # sequence 1 is cut in two
    pot[2, 250, :, 1:] = -np.inf                # sequence 2 passes through label 0
    check_all(pot, np.array([401, 401, 401], np.int32), f"cut C={C}")


@pytest.mark.parametrize("C", [33, 64, 100, 130, 256])
def test_outside_the_linear_range(C):
    # sequences that leave the log-semiring walks' range beside one that does not: a large
    # potential in the middle of a chunk, masks of -1e4, entries far below their vector's largest
    pot, lens = W.random_case(37000 + C, 4, 200, C, lengths=[200, 200, 150, 200])
    pot[0, 101, 0, C - 1] = 40.0
    pot[1, :, :, 0] = -1e4
    pot[2, 50:60, :, 1:2] -= 23.0
    check_all(pot, lens, f"range C={C}")


@pytest.mark.parametrize("C", [33, 40, 63, 64])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 12, 17, 65, 100, 140, 200])
def test_short_chains_at_the_chunk_kernels(C, N):
    # on both sides of the line up to which the chunk kernels compute alone
    pot, lens = W.random_case(39900 + C + N, 3, N, C, lengths=[N, max(1, N // 2), 1])
    pot[0, N // 2 - 1, 0, 1:] = -np.inf
    check_all(pot, lens, f"short C={C} N={N}")


@pytest.mark.parametrize("C,N", [(129, 600), (160, 1000), (200, 600), (256, 300), (256, 600)])
def test_some_walks_left_after_the_rounds(C, N):
    # short chunks (32 edges for Viterbi, 16 for the marginals): some do not meet in two rounds and are
    # walked in order before the tree is asked, at the first edges, later ones and the last
    pot, lens = W.random_case(39800 + C + N, 2, N, C, lengths=[N, N - 77])
    check_all(pot, lens, f"walked in order C={C} N={N}")


@pytest.mark.parametrize("C", [9, 24, 36, 64, 75, 100, 130, 256])
def test_range_left_by_a_second_walk(C):
    # two label sets without transitions between them, one falling behind by e^-0.3 per edge: every
    # chunk's first walk stays within the linear range, the walks from true starts leave it
    N = 700 if C < 100 else 400
    rng = np.random.default_rng(40000 + C)
    pot = rng.standard_normal((4, N - 1, C, C)).astype(np.float32)
    h = C // 2
    pot[1:, :, :h, h:] = -np.inf
    pot[1:, :, h:, :h] = -np.inf
    pot[1:3, :, h:, h:] -= np.float32(0.3)
    check_all(pot, np.array([N, N, N - 9, N], np.int32), f"falling behind C={C}")


def _normalised(seed, B, N, C):
    rng = np.random.default_rng(seed)
    p = rng.standard_normal((B, N - 1, C, C))
    return (p - np.log(np.exp(p).sum(3, keepdims=True))).astype(np.float32)


@pytest.mark.parametrize("B,N,C", [(1, 16384, 8), (1, 65536, 8), (1, 16384, 33), (1, 65536, 33),
                                   (4, 8192, 20), (1, 8192, 100), (2, 4096, 200), (1100, 2600, 3)])
def test_row_normalised_potentials(B, N, C):
    # log Z is near log C however many edges and chunks there are, so that an error per edge or
    # per chunk shows (the last case has one chunk per sequence)
    p = _normalised(39000 + C, B, N, C)
    lens = np.array([N - 7 * (b % 5) for b in range(B)], np.int32)
    ref = oracle.logpartition(p, lens)
    labels = np.random.default_rng(1).integers(0, C, (B, N)).astype(np.int32)
    tp, tl = torch.from_numpy(p).cuda(), torch.from_numpy(lens).cuda()
    z = binding.logpartition(tp, tl).cpu().numpy()
    lp = binding.log_density(tp, torch.from_numpy(labels).cuda(), tl).cpu().numpy()
    say(f"normalised B={B} N={N} C={C}: log Z off by {np.abs(z - ref).max():.1e}")
    check_logz(z, ref)
    check_logz(lp, oracle.log_density(p, labels, lens), "log density")
    if N * C * C <= 1 << 24:
        z2, _ = binding.marginals(tp, tl)
        check_logz(z2.cpu().numpy(), ref, "logZ (marginals call)")


def test_refined_log_z_replays_in_a_graph():
    # the last chunk to end adds the others up: every replay counts them anew
    p = torch.from_numpy(_normalised(39700, 2, 4000, 8)).cuda()
    lens = torch.tensor([4000, 3100], device="cuda", dtype=torch.int32)
    z = torch.empty(2, device="cuda")
    ws = torch.empty(binding.workspace_bytes(binding.OP_LOGPARTITION, 2, 4000, 8), device="cuda",
                     dtype=torch.uint8)
    want = binding.logpartition(p, lens, out=z, ws=ws).clone()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        binding.logpartition(p, lens, out=z, ws=ws)
    torch.cuda.synchronize()
    for _ in range(4):
        z.fill_(-7)
        binding.viterbi(p, lens)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, want)


def test_chunk_scales_have_no_bias():
    # before log Z is refined: 900 edges in one chunk (among many copies) and in 14 (alone)
    for C in (8, 33):
        p = torch.from_numpy(_normalised(39500 + C, 1, 901, C)).cuda()
        z, _ = binding.marginals(p)
        many, _ = binding.marginals(p.expand(1024, -1, -1, -1).contiguous())
        # a rounding per edge at random, 2^-26 per chunk, and the results' own rounding
        assert abs(z.item() - many[0].item()) <= 2.0 ** -24 * 30 + 14 * 2.0 ** -26 + 2.0 ** -22


def test_more_edges_than_a_launch_has_threads_for():
    # one label, 68.8 million edges: one workgroup of 64 threads per edge would pass 2^32 threads
    B, N = 8400, 8193
    g = torch.Generator(device="cuda")
    g.manual_seed(41000)
    pot = torch.randn(B, N - 1, 1, 1, generator=g, device="cuda")
    lens = torch.randint(1, N + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    z, m = binding.marginals(pot, lens)
    on = torch.arange(N - 1, device="cuda")[None] < (lens - 1)[:, None]
    # each marginal is 1 = a E b / (a' b) with a' = a E: two products, a division, the exponent's power
    # of two and a' rounded to float32, 5 * 2^-24; padding is exactly 0
    assert (m[:, :, 0, 0] - on.float()).abs().max().item() <= 5 * 2.0 ** -24
    assert not m[:, :, 0, 0][~on].any()
    ref = torch.where(on, pot[:, :, 0, 0].double(), 0.0).sum(1)
    assert ((z - ref).abs() / ref.abs().clamp(min=1)).max().item() <= 1e-5


def test_noalloc_without_the_recursions_buffers():
    # too large for the scratch array with the recursions' buffers, small enough without: the
    # chunk kernels take it, to the accuracy of the marginals either way (float32 storage of
    # values in [0, 1] over messages of both paths: 2e-6)
    B, N, C = 900, 1000, 9
    assert binding.workspace_bytes(binding.OP_MARGINALS, B, N, C) > binding.noalloc_scratch_bytes()
    torch.manual_seed(3)
    pot = torch.randn(B, N - 1, C, C, device="cuda")
    lens = torch.randint(1, N + 1, (B,), device="cuda", dtype=torch.int32)
    z1, m1 = binding.marginals(pot, lens)
    z2, m2 = binding.marginals_noalloc(pot, lens)
    assert torch.allclose(z1, z2, rtol=1e-6, atol=1e-6)
    assert (m1 - m2).abs().max().item() <= 2e-6
