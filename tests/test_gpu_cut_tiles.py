"""Key tiles whose dK/dV work is cut into chunks over several workgroups (few tiles, or many query heads per KV
head): chunk boundaries, ragged tiles and both workgroup shapes, against the oracle at the bar of the other tests."""
import numpy as np
import pytest
import torch

from paper_2407_09105_amd import binding, workloads as wl
from tests.gpu_util import assert_close, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,hq,hkv,d,dtype,hint", [
    ([[640]], 4, 1, 128, "bf16", 0),                       # ten blocks, G = 4: last tiles have one trip per head
    ([[513, 1, 257]], 16, 1, 64, "f16", 0),                # MQA, a chunk begins inside a block's heads
    ([[383], [383], [383]], 9, 1, 128, "bf16", 0),         # rows that start off the 64-token grid, G = 9
    ([[1600]], 5, 1, 128, "bf16", binding.HINT_LONG_EXAMPLES),   # the 128-key shape, cut
    ([[1600]], 5, 1, 128, "bf16", binding.HINT_SHORT_EXAMPLES),
    ([[1100, 1030]], 4, 2, 96, "bf16", 0),                 # the device picks the 128-key shape
    ([[700, 31]], 6, 1, 256, "f16", 0),                    # two 128-column halves
    ([[1700]], 1, 1, 80, "bf16", 0),                       # no grouped heads: blocks in ascending order
    ([[30] * 40], 16, 1, 64, "bf16", 0),                   # cut or not by a short tile's trips
])
def test_cut_tiles(lengths, hq, hkv, d, dtype, hint):
    w = wl.make_custom(lengths, hq, hkv, d, dtype, seed=71)
    print(f"case: {lengths if len(lengths[0]) < 5 else 'many'} {hq}/{hkv} d={d} {dtype} hint={hint}", flush=True)
    got = run_gpu(w, grad_dtype=torch.float32, nan_fill=True, hint=hint)
    assert_close(got, run_oracle(w), dtype)
    again = run_gpu(w, grad_dtype=torch.float32, nan_fill=True, hint=hint)
    for key in ("dQ", "dK", "dV"):
        assert np.array_equal(got[key], again[key]), key   # the chunks are added in a fixed order
