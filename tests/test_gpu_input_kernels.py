"""Rotary embedding at the sizes where their launch rules and remainders lie."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2407_09105_amd import workloads as wl
from tests.test_gpu_rope import _rel_l2, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4099, 1, 16), (1027, 7, 128), (3, 200, 128), (700, 5, 80), (259, 3, 6), (2, 130, 256)])
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
