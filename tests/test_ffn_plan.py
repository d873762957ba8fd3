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
