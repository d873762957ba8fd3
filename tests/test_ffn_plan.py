"""Which kernel each expert GEMM takes and how it is launched: host-side rules,
checked without a GPU (where the rules ask, 256 compute units)."""
import pytest

from paper_2606_15177_amd import workloads as W
from tests.gpu_util import DECODE, MID, TILED, ffn_plan


@pytest.fixture(scope="module")
def moe():
    from paper_2606_15177_amd import moe
    return moe


def _plan(moe, T, H, E, k, I, E_local=None, n_shared=0, I_shared=0, rows_indexed=True):
    return ffn_plan(moe, moe.dims(T, H, E, k, I, 2, E_local or E, n_shared, I_shared), rows_indexed)


@pytest.mark.parametrize("name,T,up,down", [
    ("decode_mixtral", 64, DECODE, MID), ("decode_mixtral", 2000, TILED, TILED),
    ("prefill_qwen3_30b_a3b", 1, MID, MID), ("prefill_qwen3_30b_a3b", 256, MID, MID),
    ("prefill_qwen3_30b_a3b", 8192, TILED, TILED),
    ("prefill_dsv2_lite", 1021, MID, MID), ("prefill_dsv2_lite", 4096, TILED, TILED),
    ("ep_share_dsv3", 512, MID, MID), ("ep_share_dsv3", 16384, TILED, TILED),
])
def test_kernels_of_the_workloads(moe, name, T, up, down):
    p = ffn_plan(moe, moe.dims_of(W.CONFIGS[name], T=T), True)
    assert [q["kernel"] for q in p] == [up, down]


@pytest.mark.parametrize("dims,gemm,tiles", [
    # the shared experts' tiles first (600 tokens: 3 m-tiles), then at most 7 routed m-tiles; gate/up, 4 column tiles
    (dict(T=600, H=4096, E=4, k=1, I=512, n_shared=1, I_shared=512), 0, (3 + 7) * 4),
    # down with whole tiles (shared rows), past the mid-sized kernel's mean: 4 + 3 + 8 m-tiles, one column tile
    (dict(T=900, H=256, E=4, k=2, I=1024, n_shared=1, I_shared=1024), 1, 4 + 8 + 4),
    # wide tail tiles: 32 + 10 m-tiles, 5 column tiles of 128
    (dict(T=8000, H=1024, E=10, k=1, I=640), 0, (32 + 10) * 5),
])
def test_tiled_grid_is_one_workgroup_per_tile(moe, dims, gemm, tiles):
    """The tiles are dealt to the XCDs by workgroup number: more workgroups
    than tiles would leave whole XCDs without any."""
    p = _plan(moe, **dims)[gemm]
    assert p["kernel"] == TILED and (p["tail"] != 2 or p["merged"])
    assert p["blocks"] == -(-min(tiles, 256) // 8) * 8


def test_tiled_grid_two_workgroups_per_tile_for_halves(moe):
    """Long K alone: the last round may run in half tiles, two workgroups each."""
    p = _plan(moe, T=300, H=4096, E=3, k=1, I=512)[0]     # (2 + 3) x 4 tiles
    assert (p["kernel"], p["tail"], p["merged"], p["blocks"]) == (TILED, 2, 0, 40)


@pytest.mark.parametrize("dims,up,down", [
    # tiles of more than half a round, or of several: gate/up on them
    (dict(T=824, H=1560, E=36, k=7, I=1496, E_local=31, n_shared=1, I_shared=1024), TILED, MID),
    (dict(T=3143, H=2688, E=48, k=2, I=1400), TILED, TILED),
    (dict(T=2211, H=2048, E=128, k=8, I=768), MID, TILED),    # (past the second round, a mean of 138)
    # ... of at most half a round, of few rows, of a short K
    (dict(T=600, H=2048, E=8, k=2, I=512), MID, MID),
    (dict(T=400, H=2688, E=48, k=2, I=3200), MID, MID),
    (dict(T=3143, H=896, E=48, k=2, I=3200), MID, TILED),
    # small decode batches of short K; gate/up of many items over hit experts
    (dict(T=1, H=1280, E=8, k=3, I=448), MID, DECODE),
    (dict(T=1, H=640, E=8, k=3, I=448), DECODE, DECODE),
    (dict(T=1, H=640, E=8, k=3, I=448, n_shared=1, I_shared=448), MID, MID),
    (dict(T=64, H=640, E=8, k=3, I=448), MID, MID),
    (dict(T=24, H=4096, E=8, k=2, I=2816), DECODE, MID),
    (dict(T=8, H=2048, E=16, k=2, I=5632), MID, MID),        # a third of the experts not hit
    (dict(T=24, H=8192, E=16, k=2, I=2816), MID, MID),
])
def test_kernels_by_rule(moe, dims, up, down):
    assert [q["kernel"] for q in _plan(moe, **dims)] == [up, down]


def test_long_k_split_by_items(moe):
    """Gate/up of 8 hit experts on K 4096: 176 items run whole, few in halves."""
    assert _plan(moe, T=64, H=4096, E=8, k=2, I=1408)[0]["split_k"] == 0
    assert _plan(moe, T=64, H=4096, E=8, k=2, I=704)[0]["split_k"] == 1
    assert _plan(moe, T=24, H=5120, E=96, k=8, I=640, E_local=24)[0]["split_k"] == 1   # not mostly hit


def test_mid_launch_fits_one_grid_dimension(moe):
    """1024 experts of 2^21 output columns make more items than one grid
    dimension holds threads for (2^32 - 1): the decode kernel's grid has two."""
    d = moe.dims(64, 2 ** 21, 1024, 32, 8, 2, 1024)
    assert moe.validate(d, moe.ENTRY_EXPERT_FFN, 1 << 62) == moe.MOE_OK
    assert ffn_plan(moe, d, False)[1]["kernel"] == DECODE
    p = _plan(moe, T=64, H=2 ** 20, E=1024, k=32, I=8, rows_indexed=False)[1]
    assert p["kernel"] == MID and p["blocks"] * 256 < 2 ** 32
