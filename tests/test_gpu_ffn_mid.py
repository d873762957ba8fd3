"""GPU parity of the mid-sized grouped GEMM (more rows per expert than a
decode step, fewer than fill 256-row tiles) against the CPU oracle, every row,
and of the 256-row tiles at shapes that stay on them."""
import numpy as np
import pytest

from tests.test_gpu_ffn import _case, _run_ffn, moe  # noqa: F401  (moe: the module fixture)

pytestmark = pytest.mark.gpu

# rows per expert at the edges of 32-row MFMA tiles, of the narrow items (64
# rows), of 128-row chunks and of the equal split of larger groups into chunks
EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 193, 255, 256, 257, 300]
TILE_EDGES = [1, 127, 128, 129, 255, 256, 257, 511, 512, 513, 65]


def _sized(moe, sizes, H, I, n_sh=0, I_sh=0):
    T = sum(sizes)
    cfg, wl, _ = _case(T, H, len(sizes), 1, I, len(sizes), n_sh, I_sh)
    idx = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)[np.random.default_rng(3).permutation(T)]
    assert _run_ffn(moe, cfg, wl, idx.reshape(T, 1)) == T


@pytest.mark.parametrize("H,I,n_sh,I_sh", [
    (64, 64, 0, 0),         # one stage, one column block; few wide items (128 weight rows each)
    (136, 200, 0, 0),       # ragged K and N
    (264, 1160, 0, 0),      # gate/up with many wide items (256 weight rows each), ragged
    (2312, 72, 0, 0),       # down likewise
    (264, 72, 2, 1160),     # shared rows in the launch, K stacked over two experts, many wide items
    (136, 200, 2, 40),      # ... few, segments shorter than a stage
    (8, 8, 1, 8),           # a single 16-byte piece of K
])
def test_mid_chunk_edges(moe, H, I, n_sh, I_sh):  # noqa: F811
    _sized(moe, EDGES, H, I, n_sh, I_sh)


@pytest.mark.parametrize("sizes", [[66] * 3, [0, 70, 0, 0], [40] * 70, [1] * 100 + [200], [64, 65] * 40])
def test_mid_group_mixes(moe, sizes):  # noqa: F811
    """Only wide groups, one group with rows, only narrow groups in more than
    one 64-group pass, one hot group, and both kinds taking turns."""
    _sized(moe, sizes, 136, 200)


@pytest.mark.parametrize("H,I", [
    (136, 1544),            # gate/up: 286 tiles, past the few-tiles rule; wide tails
    (5000, 136),            # gate/up on long K (half tails), down with 440 tiles
])
def test_tile_boundaries_on_the_tiled_kernel(moe, H, I):  # noqa: F811
    _sized(moe, TILE_EDGES, H, I)


@pytest.mark.parametrize("sizes", [[64], [33, 31], [1, 31, 32], [0, 50, 2], [3] * 20, [1]])
@pytest.mark.parametrize("H,I,n_sh,I_sh", [
    (136, 200, 0, 0),       # few items: K in two halves
    (8, 8, 1, 8),           # ... one half empty
    (264, 520, 0, 0),       # with 20 groups: K whole for gate/up
    (4104, 72, 2, 40),      # long K with a ragged second half; shared rows, a stacked K
])
def test_decode_batches(moe, sizes, H, I, n_sh, I_sh):  # noqa: F811
    _sized(moe, sizes, H, I, n_sh, I_sh)


def test_last_round_in_halves(moe):  # noqa: F811
    """Gate/up on long K: 280 tiles, the 24 past the first 256 (whole tiles of
    256 and 129 rows, and tail tiles, which have no second half) as halves."""
    _sized(moe, [385] * 14 + [300, 128, 257, 385], 4104, 1016)


def test_only_round_of_long_k(moe):  # noqa: F811
    """Gate/up on long K, 200 tail tiles on 256 CUs: more than run in halves,
    dealt to the XCDs in equal shares."""
    _sized(moe, [41] * 20, 4104, 1160)


@pytest.mark.parametrize("sizes", [[1] * 256, [0] * 255 + [5], [0] * 256 + [70], [2] * 257 + [66, 0], [65] + [0] * 320 + [3],
                                   [0] * 1023 + [3], [1] * 40 + [0] * 943 + [130] + [1] * 40])
def test_many_groups(moe, sizes):  # noqa: F811
    """The group of an item, at and past 256 groups (one batch of offsets)."""
    _sized(moe, sizes, 72, 136)
