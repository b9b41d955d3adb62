"""Key tiles whose dK/dV work is cut into chunks over several workgroups (few tiles, or many query heads per KV
head): chunk boundaries, ragged tiles and both workgroup shapes, against the oracle at the bar of the other tests."""
import numpy as np
import pytest
import torch

from paper_2407_09105_amd import binding, workloads as wl
from tests.gpu_util import DEV, assert_close, run_gpu, run_oracle, to_dev
from tests.test_gpu_guards import _guarded

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
    ([[500]], 4, 1, 128, "bf16", 0),                       # four chunks at most: first chunks move on from tile to tile
    ([[100] * 20], 6, 1, 64, "f16", 0),                    # two chunks at most
    ([[55] * 40], 8, 2, 64, "bf16", 0),                    # a row that could be cut, examples that are not
    ([[900, 50], [475, 475]], 16, 2, 96, "bf16", 0),       # rows off the 64-token grid, off the schedule tile
])
def test_cut_tiles(lengths, hq, hkv, d, dtype, hint):
    w = wl.make_custom(lengths, hq, hkv, d, dtype, seed=71)
    print(f"case: {lengths if len(lengths[0]) < 5 else 'many'} {hq}/{hkv} d={d} {dtype} hint={hint}", flush=True)
    got = run_gpu(w, grad_dtype=torch.float32, nan_fill=True, hint=hint)
    assert_close(got, run_oracle(w), dtype)
    again = run_gpu(w, grad_dtype=torch.float32, nan_fill=True, hint=hint)
    for key in ("dQ", "dK", "dV"):
        assert np.array_equal(got[key], again[key]), key   # the chunks are added in a fixed order


@pytest.mark.parametrize("lengths,hq,hkv,d,dtype", [
    ([[640]], 4, 1, 128, "bf16"),
    ([[640]], 4, 1, 64, "f32"),
    ([[33] * 70 + [1500] + [33] * 80], 21, 7, 96, "bf16"),   # only chunks of long key tiles have a place
])
@pytest.mark.parametrize("room", [0, 1, 3 << 20])   # bytes behind D: none, too little for a chunk, for some chunks only
def test_workspace_of_any_size(lengths, hq, hkv, d, dtype, room):
    w = wl.make_custom(lengths, hq, hkv, d, dtype, seed=72)
    N = w.q.shape[0]
    q, k, v, do = (to_dev(a, dtype) for a in (w.q, w.k, w.v, w.do))
    seg = binding.pack_to_cu_seqlens(torch.from_numpy(w.position_ids).to(DEV))
    o, lse = binding.varlen_attn_fwd(q, k, v, seg)
    (ws,), check = _guarded([(((N * hq * 4 + 255) // 256 * 64 + (room + 3) // 4,), torch.float32)])
    dq, dk, dv = binding.varlen_attn_bwd(do, q, k, v, o, lse, seg, grad_dtype=torch.float32, workspace=ws)
    check()
    ref = run_oracle(w)
    f = lambda t: t.float().cpu().numpy().astype(np.float64)
    assert_close({"O": f(o), "LSE": f(lse), "dQ": f(dq), "dK": f(dk), "dV": f(dv)}, ref, dtype)


@pytest.mark.parametrize("lengths,hq,hkv,d,dtype", [   # too many tiles to cut all of them finely, G > 1
    ([[1800] + [20] * 125] * 2, 20, 4, 128, "bf16"),
    ([[40] * 55 + [2100]], 16, 8, 128, "f16"),
    ([[33] * 70 + [1500] + [33] * 80], 21, 7, 96, "bf16"),
])
def test_long_chains_among_many_tiles(lengths, hq, hkv, d, dtype):
    w = wl.make_custom(lengths, hq, hkv, d, dtype, seed=73)
    print(f"case: {hq}/{hkv} d={d} {dtype}", flush=True)
    got = run_gpu(w, grad_dtype=torch.float32, nan_fill=True)
    assert_close(got, run_oracle(w), dtype)
    again = run_gpu(w, grad_dtype=torch.float32, nan_fill=True)
    for key in ("dQ", "dK", "dV"):
        assert np.array_equal(got[key], again[key]), key
