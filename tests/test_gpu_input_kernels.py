"""Boundary scan, collator and rotary embedding at the sizes where their launch rules and remainders lie."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2407_09105_amd import workloads as wl
from tests.gpu_util import assert_seg_equal
from tests.test_gpu_collate import _compare
from tests.test_gpu_pack import _check_orders, _gpu_pack
from tests.test_gpu_rope import _rel_l2, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,T,maxlen", [
    (8193, 1, 1),          # a tile per token
    (1, 10240, 10240),     # whole chunks of 2048 tokens, one example
    (33, 257, 257),        # tiles of one token
    (5, 4099, 700),        # rows that straddle chunks, tiles that straddle chunks
    (9, 1000003, 5000),    # more chunks than a workgroup folds into its own carries
])
def test_pack(R, T, maxlen):
    rng = np.random.default_rng(R + T)
    pos = np.empty((R, T), dtype=np.int64)
    for r in range(R):
        starts = np.unique(np.concatenate([[0], rng.integers(0, T, size=max(1, 2 * T // maxlen))]))
        pos[r] = np.arange(T) - np.repeat(starts, np.diff(np.concatenate([starts, [T]])))
    got = _gpu_pack(pos)
    assert_seg_equal(got, oracle.pack(pos))
    if R * T < 100000:
        _check_orders(got, pos)


@pytest.mark.parametrize("R,T,maxlen", [   # one launch: each size of workgroup, full and one token over, few and many tiles
    (1, 1, 1), (1, 2048, 90), (1, 2049, 700), (1, 4096, 4096), (1, 4097, 90), (1, 8192, 700), (256, 1, 1), (256, 8, 3), (255, 9, 4),
    (3, 513, 200), (2, 2048, 2048), (17, 241, 100), (256, 32, 9)])
def test_pack_in_one_launch(R, T, maxlen):
    test_pack(R, T, maxlen)


@pytest.mark.parametrize("n", [1, 255, 2047, 2048, 2049])  # up to 2048 examples run in one launch
@pytest.mark.parametrize("cut", [0, 5, -7])
def test_collate(n, cut):
    rng = np.random.default_rng(n)
    lengths = rng.integers(0, 9, size=n).astype(np.int32)
    lengths[0] = 8
    ids = rng.integers(0, 1000, size=(n, 8))
    total = int(np.minimum(lengths, 8).sum())
    _compare(ids, lengths, 0 if cut == 5 else total - cut, pad_id=3)


@pytest.mark.parametrize("n_out", [1024 * 256, 1024 * 256 + 1])  # the last of 2048 examples in one launch, the first in two
def test_collate_many_tokens(n_out):
    rng = np.random.default_rng(n_out)
    lengths = rng.integers(100, 160, size=2048).astype(np.int32)
    ids = rng.integers(0, 1000, size=(2048, 160))
    assert int(lengths.sum()) > n_out
    _compare(ids, lengths, n_out, pad_id=3)


@pytest.mark.parametrize("shape", [(4099, 1, 16), (1027, 7, 128), (3, 200, 128), (700, 5, 80), (259, 3, 6), (2, 130, 256), (5, 700, 96), (1, 2100, 10),
                                   (11000, 1, 96), (66000, 1, 2), (21845, 1, 48)])   # one head, an item a thread
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("inplace", [False, True])
def test_rope(shape, dtype, inplace):
    rng = np.random.default_rng(sum(shape))
    x = wl.round_to_bf16(rng.standard_normal(shape).astype(np.float32))
    pos = rng.integers(0, 20000, size=shape[0])
    got, ref = _run(x, pos, dtype, inplace=inplace), oracle.rope(x, pos)
    # bf16 results: half an ulp (2^-9) of rounding; fp32: a few roundings of 6e-8
    assert _rel_l2(got, ref) <= (1e-6 if dtype == torch.float32 else 3e-3)
    assert np.all(np.abs(got - ref) <= (4e-6 if dtype == torch.float32 else 2.0 ** -8 * np.abs(ref) + 4e-6))
