"""Parity of the single-launch kernels' walks with the float64 oracle: every lane layout
(C padded to 8, 16, 20, 24 or 32) at its edge label counts, lengths on both sides of the one
where log Z and Viterbi go over to the tree, and inputs that leave the walks' range."""
import numpy as np
import pytest

from gpu_util import check_all
from paper_2002_00876_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [1, 2, 7, 8, 9, 16, 17, 20, 21, 24, 25, 32])
def test_layouts(C):
    N = 12 if C > 24 else 24
    pot, lens = W.random_case(41000 + C, 5, N, C, sigma=1.5, lengths=[N, N - 1, 3, 2, 1])
    check_all(pot, lens, f"walk C={C}")


@pytest.mark.parametrize("C,N", [(8, 80), (8, 81), (8, 82), (5, 120), (3, 150)])
def test_walk_and_tree_lengths(C, N):
    pot, lens = W.random_case(42000 + N, 4, N, C, sigma=1.0, lengths=[N, N - 1, min(N, 81), 40])
    check_all(pot, lens, f"C={C} N={N}")
    pot, lens = W.random_case(43000 + N, 4, N, C, kind="int", int_range=1, lengths=[N, N - 1, min(N, 82), 40])
    check_all(pot, lens, f"ties C={C} N={N}")


@pytest.mark.parametrize("C", [4, 13, 20, 32])
def test_outside_the_range(C):
    # a batch in which some sequences leave the range: one large potential, masks of -1e4, an
    # entry far below its vector's largest, and one ordinary sequence
    pot, lens = W.random_case(44000 + C, 5, 12, C, lengths=[12, 12, 12, 9, 12])
    pot[0, 5, 0, C - 1] = 30.0
    pot[1, :, :, 0] = -1e4
    pot[2, 3:7, :, 1:2] -= 20.0
    pot[3, 2, : C // 2] = -np.inf
    check_all(pot, lens, f"range C={C}")


@pytest.mark.parametrize("C", [1, 2, 4])
def test_viterbi_walk_and_tree_lengths_of_few_labels(C):
    # 56 / 57, 64 / 65 and 76 / 77 edges, where Viterbi of up to 4 labels changes between them
    lens = [57, 58, 65, 66, 77, 78, 79, 1]
    for kind, kw in (("normal", {}), ("int", dict(int_range=1))):
        pot, ln = W.random_case(45000 + C, 8, 79, C, kind=kind, lengths=lens, **kw)
        check_all(pot, ln, f"few labels C={C} {kind}")
