"""GPU placement against the CPU oracle where the greedy's step can go wrong:
ties everywhere, NaN and infinite scores beside full ranks, every butterfly
width, chunk edges, and counts staged whole, by columns and by pieces."""
import numpy as np
import pytest

from tests.test_gpu_place import _check, _gpu_place, moe  # noqa: F401  (moe: the module fixture)
from oracle import oracle

pytestmark = pytest.mark.gpu


def _inputs(L, S, E, G, seed, hi=1000):
    rng = np.random.default_rng(seed)
    A = rng.integers(0, hi, (L, S, E)).astype(np.int64)
    D = rng.integers(0, 3, (S, G)).astype(np.float64)
    x0 = rng.integers(-1, G, (L, E)).astype(np.int32)
    return A, D, x0, np.full(G, -(-E // G), np.int32)


@pytest.mark.parametrize("G", [1, 2, 3, 7, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("hi", [1, 3, 1000])
def test_widths_and_ties(moe, G, hi):  # noqa: F811
    """hi = 1: no counts at all, every score ties; 3: many ties."""
    _check(moe, *_inputs(2, 5, 2 * G + 1, G, G + hi, hi), what=f"G {G} hi {hi}")


@pytest.mark.parametrize("S,E,G", [
    (8, 33, 8), (8, 512, 8),        # staged whole, one expert past a chunk; the largest staged
    (64, 31, 64), (64, 241, 64),    # columns, one expert per wave
    (100, 700, 5), (300, 64, 3),    # batches cut to fit a wave's piece
    (1000, 40, 4), (4096, 9, 1),    # columns longer than a piece
    (1, 1024, 64), (17, 1024, 33),
])
def test_chunks_and_staging(moe, S, E, G):  # noqa: F811
    _check(moe, *_inputs(2, S, E, G, S + E + G), what=f"{S} {E} {G}")


@pytest.mark.parametrize("S,E,G", [
    (3, 33, 2), (8, 512, 8), (1, 70, 64),   # staged whole: four waves per layer
    (100, 48, 3), (64, 70, 64), (300, 64, 5), (1100, 9, 3),   # columns and pieces: eight
])
def test_more_layers_than_cus(moe, S, E, G):  # noqa: F811
    _check(moe, *_inputs(260, S, E, G, S + E + G), what=f"{S} {E} {G}")


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("G", [2, 5, 8, 20])
def test_bad_scores_beside_full_ranks(moe, G, bad):  # noqa: F811
    """Ranks fill up while the others' migration costs are NaN or infinite:
    the choice is still an open rank, by the tie rules."""
    E = 3 * G
    A, D, x0, _ = _inputs(2, 4, E, G, 7)
    x0[:] = np.arange(E) % G
    cap = np.full(G, 5, np.int32)
    cap[0] = 1
    rng = np.random.default_rng(G)
    M = rng.uniform(0, 50, (2, E, G))
    M[:, :, 1:] = bad
    M[1, ::2, G // 2] = 1.0
    x, _, _ = _gpu_place(moe, A, D, x0, cap, M=M)
    ref, _ = oracle.place_greedy(A, D, x0, cap, M=M)
    np.testing.assert_array_equal(x, ref)
