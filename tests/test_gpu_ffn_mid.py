"""GPU parity of the mid-sized grouped GEMM (decode batches and more rows per
expert, fewer than fill 256-row tiles) against the CPU oracle, every row, and of
the 256-row tiles at the shapes that the launch rules leave them."""
import numpy as np
import pytest

from tests.gpu_util import MID, TILED, ffn_plan
from tests.test_gpu_ffn import _case, _run_ffn, moe  # noqa: F401  (moe: the module fixture)

pytestmark = pytest.mark.gpu

# rows per expert at the edges of 32-row MFMA tiles, of the narrow items (64
# rows), of 128-row chunks and of the equal split of larger groups into chunks
EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 193, 255, 256, 257, 300]
TILE_EDGES = [1, 127, 128, 129, 255, 256, 257, 511, 512, 513, 65]


def _sized(moe, sizes, H, I, n_sh=0, I_sh=0, kernels=None):
    """Groups of these rows; kernels: those that (gate/up, down) are to take."""
    T = sum(sizes)
    cfg, wl, _ = _case(T, H, len(sizes), 1, I, len(sizes), n_sh, I_sh)
    if kernels is not None:
        plan = ffn_plan(moe, moe.dims_of(cfg), False)
        assert tuple((p["kernel"], p["tail"]) if p["kernel"] == TILED else p["kernel"] for p in plan) == kernels
    idx = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)[np.random.default_rng(3).permutation(T)]
    assert _run_ffn(moe, cfg, wl, idx.reshape(T, 1)) == T


@pytest.mark.parametrize("H,I,n_sh,I_sh", [
    (64, 64, 0, 0),         # one stage, one column block; few wide items (128 weight rows each)
    (136, 200, 0, 0),       # ragged K and N
    (264, 1160, 0, 0),      # ten column blocks of gate/up, ragged
    (2312, 72, 0, 0),       # gate/up on long K; down on wide tail tiles
    (264, 72, 2, 1160),     # gate/up with shared rows in the launch; down on whole tiles
    (136, 200, 2, 40),      # shared rows in both, K stacked over two experts, segments shorter than a stage
    (8, 8, 1, 8),           # a single 16-byte piece of K
])
def test_mid_chunk_edges(moe, H, I, n_sh, I_sh):  # noqa: F811
    _sized(moe, EDGES, H, I, n_sh, I_sh)


# 22 chunks of more than 64 rows in EDGES, 19 of the shared rows: 256 items of
# 256 weight rows or more
@pytest.mark.parametrize("sizes,H,I,n_sh,I_sh", [
    (EDGES, 264, 1544, 0, 0),               # gate/up, 13 column blocks
    (EDGES + [0] * 40, 2840, 72, 0, 0),     # down, 12
    (EDGES, 1544, 264, 2, 40),              # down, 7, with K stacked over two shared experts
])
def test_mid_many_wide_items(moe, sizes, H, I, n_sh, I_sh):  # noqa: F811
    _sized(moe, sizes, H, I, n_sh, I_sh, kernels=(MID, MID))


@pytest.mark.parametrize("sizes", [[66] * 3, [0, 70, 0, 0], [40] * 70, [1] * 100 + [200], [64, 65] * 40])
def test_mid_group_mixes(moe, sizes):  # noqa: F811
    """Only wide groups, one group with rows, only narrow groups in more than
    one 64-group pass, one hot group, and both kinds taking turns."""
    _sized(moe, sizes, 136, 200)


@pytest.mark.parametrize("H,I,kernels", [
    (136, 1544, (MID, MID)),                # gate/up: 143 tiles of a mean group, few enough for the mid-sized kernel
    (5000, 136, ((TILED, 2), (TILED, 1))),  # gate/up on long K: half tails; down: wide tails, an even number of column tiles
    (1016, 1288, ((TILED, 1), MID)),        # gate/up: wide tails, an odd number of column tiles
])
def test_tile_boundaries_on_the_tiled_kernel(moe, H, I, kernels):  # noqa: F811
    _sized(moe, TILE_EDGES, H, I, kernels=kernels)


def test_tiles_of_more_than_256_groups(moe):  # noqa: F811
    """16 prefix entries per lane, whole tiles, gate/up and down."""
    _sized(moe, [130] * 246 + TILE_EDGES, 1008, 136, kernels=((TILED, 0), (TILED, 0)))


@pytest.mark.parametrize("T", [1000, 2900])
def test_shared_gate_up_alone_in_blocked_order(moe, T):  # noqa: F811
    """64 column tiles of shared gate/up fill whole rounds of 256 CUs with 4 and
    with 12 m-tiles: a launch of their own, m-tiles in blocks of 8 and a
    remainder of 4."""
    cfg, wl, idx = _case(T, 1008, 8, 2, 64, 8, 1, 8192)
    p = ffn_plan(moe, moe.dims_of(cfg), False)[0]
    assert (p["kernel"], p["merged"], p["sh_kernel"]) == (TILED, 0, TILED)
    _run_ffn(moe, cfg, wl, idx)


@pytest.mark.parametrize("I_sh,merged", [(1024, 0), (960, 1)])
def test_shared_gate_up_with_or_without_the_routed_tiles(moe, I_sh, merged):  # noqa: F811
    """256 shared tiles on launches of their own; 240 in the routed launch, whose
    tail tiles are then half ones."""
    cfg, wl, idx = _case(4096, 1008, 16, 2, 128, 16, 2, I_sh)
    p = ffn_plan(moe, moe.dims_of(cfg), False)[0]
    assert (p["kernel"], p["merged"], p["tail"]) == (TILED, merged, 2 if merged else 1)
    _run_ffn(moe, cfg, wl, idx)


@pytest.mark.parametrize("sizes", [[64], [33, 31], [1, 31, 32], [0, 50, 2], [3] * 20, [1]])
@pytest.mark.parametrize("H,I,n_sh,I_sh", [
    (136, 200, 0, 0),       # few items: K in two halves (with 20 groups, or one row: the decode kernel)
    (8, 8, 1, 8),           # ... one half empty
    (264, 520, 0, 0),       # with 20 groups: K whole for gate/up, down on the decode kernel
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
