"""GPU parity of the decode kernel of the expert GEMMs against the CPU oracle
(every row), at the shapes that the launch rules send to it: small launches of
short K, gate/up of many items on long K, and output columns past the 32-bit
tile offsets of the other kernels."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DECODE, MID, ffn_plan
from tests.test_gpu_ffn import _case, _run_ffn, moe  # noqa: F401  (moe: the module fixture)

pytestmark = pytest.mark.gpu


def _pairs(moe, sizes, T, k, H, I, kernels):  # noqa: F811
    """T tokens of k pairs each, sizes[e] of the pairs on expert e (the same
    expert twice for one token where need be)."""
    assert sum(sizes) == T * k
    cfg, wl, _ = _case(T, H, len(sizes), k, I, len(sizes))
    assert tuple(p["kernel"] for p in ffn_plan(moe, moe.dims_of(cfg), False)) == kernels
    idx = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)[np.random.default_rng(T).permutation(T * k)]
    assert _run_ffn(moe, cfg, wl, idx.reshape(T, k)) == T * k


# rows per expert: one; at and past the 32-row chunks; at and past one pass of
# 64 rows; all of them on one expert (two passes); and none
SIZES = [[2] + [0] * 15, [1, 31, 32, 0] + [0] * 12, [33, 3, 0, 28] + [0] * 12, [63, 65] + [0] * 14, [0] * 15 + [128],
         [8] * 16]


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("H,I", [
    (136, 200),             # ragged K and N of both projections
    (1024, 72),             # the longest K of the rule, sixteen steps of 64
    (8, 8),                 # one 16-byte piece of K, three of four K parts empty
    (72, 1016),             # down on long K, gate/up on two steps
])
def test_small_launches(moe, sizes, H, I):  # noqa: F811
    n = 16 * -(-I // 32)
    _pairs(moe, sizes, sum(sizes) // 2, 2, H, I, (DECODE if n <= 256 else MID, DECODE))


@pytest.mark.parametrize("sizes", [[12, 12, 12, 12], [1, 32, 33, 0], [64, 0, 63, 1], [128, 0, 0, 0]])
def test_many_items_on_long_k(moe, sizes):  # noqa: F811
    """Gate/up of 4 experts, 157 column blocks each, ragged K and N."""
    _pairs(moe, sizes, sum(sizes) // 2, 2, 4104, 5000, (DECODE, MID))


@pytest.mark.parametrize("T", [5, 33])
def test_columns_past_32_bit_tile_offsets(moe, T):  # noqa: F811
    """H of 4178000: a 256-row tile of outputs spans 2^31 bytes, so all four
    GEMMs (routed and shared ones, those with static rows, the shared down
    projection with K stacked over two experts) take the decode kernel.
    Reference: the same layer in float64."""
    H, I, n_sh, I_sh = 4178000, 8, 2, 8
    d = moe.dims(T, H, 1, 1, I, 1, 1, n_sh, I_sh)
    for p in ffn_plan(moe, d, False):
        assert (p["kernel"], p["merged"], p["sh_kernel"]) == (DECODE, 0, DECODE)
    g = torch.Generator(device="cuda").manual_seed(T)

    def normal(shape, std):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)

    x = normal((T, H), 1.0)
    w = {"w_gate": normal((1, I, H), H ** -0.5), "w_up": normal((1, I, H), H ** -0.5), "w_down": normal((1, H, I), 0.3),
         "sh_gate": normal((n_sh, I_sh, H), H ** -0.5), "sh_up": normal((n_sh, I_sh, H), H ** -0.5),
         "sh_down": normal((n_sh, H, I_sh), 0.3)}
    y, ysh = torch.zeros_like(x), torch.zeros_like(x)
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    moe.expert_ffn(d, x, offsets, w, x, y, ysh, moe.workspace(d, moe.ENTRY_EXPERT_FFN))
    xd = x.double()

    def ref(gate, up, down):
        h = torch.nn.functional.silu(xd @ gate.double().T) * (xd @ up.double().T)
        return h @ down.double().T

    refs = [(y, ref(w["w_gate"][0], w["w_up"][0], w["w_down"][0])),
            (ysh, sum(ref(w["sh_gate"][q], w["sh_up"][q], w["sh_down"][q]) for q in range(n_sh)))]
    for got, want in refs:
        # h and y are rounded to bf16 (2^-9 each), the terms of up to 16 products add up
        assert (got.double() - want).abs().max() <= 2e-2 * want.abs().max()
