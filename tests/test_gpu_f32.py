"""The kernels in fp32 arithmetic at the edges of their tiles: 16-token tiles, 32-token blocks over four waves,
head dims at the ends of each unrolling, dK/dV shared by several workgroups per tile, unaligned tensors."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2407_09105_amd import binding, workloads as wl
from tests.gpu_util import DEV, assert_close, rel_l2, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,hq,hkv,d,dtype", [
    ([[1]], 1, 1, 1, "f32"),                       # one token, one column
    ([[15]], 2, 1, 16, "f32"),                        # one short of a tile
    ([[17, 31, 33]], 4, 4, 17, "f32"),             # element-wise loads, one past the smallest unrolling
    ([[129, 3, 128], [260]], 6, 2, 32, "f32"),     # five blocks over four waves
    ([[700, 41]], 8, 1, 64, "f32"),                # 8 heads on one KV head: dK/dV in parts
    ([[300, 45]], 4, 2, 100, "f32"),               # padded to 128
    ([[90, 70]], 2, 1, 132, "f32"),                # padded to 256
    ([[90, 70]], 4, 1, 20, "bf16"),                # 16-bit head dims that are not a multiple of 8
    ([[333]], 4, 1, 129, "f16"),
])
def test_f32_kernels(lengths, hq, hkv, d, dtype):
    w = wl.make_custom(lengths, hq, hkv, d, dtype, seed=91)
    print(f"case: {lengths} {hq}/{hkv} d={d} {dtype}", flush=True)
    assert_close(run_gpu(w, grad_dtype=torch.float32, nan_fill=True), run_oracle(w), dtype)


def test_unaligned_fp32_tensors():
    # tensors that start 4 bytes off a 16-byte boundary take the element-wise loads and stores
    w = wl.make_custom([[70, 33]], 2, 2, 64, "f32", seed=92)

    def shifted(a):
        t = torch.empty(a.size + 1, device=DEV)[1:].view(a.shape)
        return t.copy_(torch.from_numpy(a))

    q, k, v, do = (shifted(a) for a in (w.q, w.k, w.v, w.do))
    seg = binding.pack_to_cu_seqlens(torch.from_numpy(w.position_ids).to(DEV))
    o, lse = binding.varlen_attn_fwd(q, k, v, seg, out=shifted(np.zeros_like(w.q)))
    dq, dk, dv = binding.varlen_attn_bwd(do, q, k, v, o, lse, seg, dq=shifted(np.zeros_like(w.q)))
    cu = oracle.pack(w.position_ids)["cu_seqlens"]
    for got, ref in zip((o, dq, dk, dv), (oracle.fwd(w.q, w.k, w.v, cu)[0], *oracle.bwd(w.do, w.q, w.k, w.v, cu))):
        assert rel_l2(got.cpu().numpy(), ref) <= 1e-5   # fp32 sums of at most 70 products: 70 x 2^-24 = 4e-6, with room


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("lengths,t,hq,hkv,d,dtype", [
    ([[9, 20, 11]], 15, 4, 2, 64, "f32"),          # three examples in the blocks of one tile
    ([[70, 45, 30], [145]], 95, 2, 2, 16, "f32"),
    ([[37, 150, 9]], 100, 8, 1, 128, "f32"),       # columns loaded where they are used; dK/dV in parts
    ([[37, 50, 9]], 60, 2, 1, 200, "f32"),
    ([[21, 40, 30]], 44, 4, 1, 20, "bf16"),        # element-wise loads
    ([[21, 340, 23]], 44, 32, 32, 64, "f32"),      # the dK/dV form for many tiles
])
def test_not_finite_tokens_stay_in_their_example(lengths, t, hq, hkv, d, dtype, value):
    # one token of an example is not finite in one tensor: what does not depend on it is as if it were
    w = wl.make_custom(lengths, hq, hkv, d, dtype, seed=93)
    ref = run_oracle(w)
    cu = ref["seg"]["cu_seqlens"]
    a, b = int(cu[np.searchsorted(cu, t, "right") - 1]), int(cu[np.searchsorted(cu, t, "right")])
    own, later, earlier, whole, none = range(t, t + 1), range(t, b), range(a, t + 1), range(a, b), range(0)
    reach = {"q": {"O": own, "LSE": own, "dQ": own, "dK": earlier, "dV": earlier},
             "k": {"O": later, "LSE": later, "dQ": later, "dK": whole, "dV": whole},
             "v": {"O": later, "LSE": none, "dQ": later, "dK": whole, "dV": none},
             "do": {"O": none, "LSE": none, "dQ": own, "dK": earlier, "dV": earlier}}
    for tensor, rows in reach.items():
        bad = wl.make_custom(lengths, hq, hkv, d, dtype, seed=93)
        getattr(bad, tensor)[t] = value
        got = run_gpu(bad, grad_dtype=torch.float32, nan_fill=True)
        for key, r in rows.items():
            view = (lambda x: x[:, list(r)]) if key == "LSE" else (lambda x: x[list(r)])
            if np.isnan(value):
                assert np.isnan(view(got[key])).all(), (tensor, key)   # and what depends on it shows it
            if key == "LSE":
                got[key][:, list(r)] = ref[key][:, list(r)]
            else:
                got[key][list(r)] = ref[key][list(r)]
        print(f"case: {tensor}[{t}] = {value}", flush=True)
        assert_close(got, ref, dtype)


@pytest.mark.parametrize("hq,hkv,d,n", [(4, 2, 16, 300), (8, 1, 32, 700), (4, 2, 64, 700), (2, 1, 128, 500), (2, 1, 256, 300)])
def test_large_scores(hq, hkv, d, n):
    # Scores of about 100.  Every score carries the rounding of its sum: of d products, whose absolute sum is A, in chains of
    # d / 8 and three levels of pairs; of d products in pairs alone it would be log2 d levels.  A rounding is 2^-24 at most,
    # 2^-24 / sqrt(3) in the mean, of a partial sum that grows to A / sqrt(d): what remains of a chain of d / 8 at random is
    # below 2^-24 A.  The LSE adds its own store's rounding.  One chain of all d products misses it at each of these d.
    w = wl.make_custom([[n]], hq, hkv, d, "f32", seed=94)
    w.q *= 30.0
    got, ref = run_gpu(w, grad_dtype=torch.float32), run_oracle(w)
    a = np.einsum("ihc,ihc->hi", np.abs(w.q).astype(np.float64), np.abs(np.repeat(w.k, hq // hkv, axis=1)).astype(np.float64)) / d ** 0.5
    bound = 2.0 ** -24 * np.sqrt((a ** 2).mean())
    err = np.sqrt(((got["LSE"] - ref["LSE"]) ** 2).mean())
    print(f"   LSE rms error {err:.2e}, bound {bound:.2e}", {k: f"{rel_l2(got[k], ref[k]):.2e}" for k in ("O", "dQ", "dK", "dV")}, flush=True)
    assert err <= bound
    # probabilities carry the error of the exponent, score - LSE: twice the bound, and dQ, dK sum differences of them
    for key in ("O", "dQ", "dK", "dV"):
        assert rel_l2(got[key], ref[key]) <= 2 * bound, key


@pytest.mark.parametrize("lengths,hq,hkv,d", [   # parts of a dK/dV tile (their number: test_parts_of_fp32_tiles)
    ([[676, 300, 24]], 8, 2, 64),    # 4
    ([[160, 1]], 20, 1, 64),         # 15, a last tile of one token
    ([[640, 17], [600, 57]], 4, 4, 16),   # 1: no query heads share a KV head
    ([[300]], 6, 3, 36),             # 2, a head_dim between the unrolled ones
    # workgroups, from 768 on two per CU (head_dim up to 32: 2048; from four query heads per KV head on twice as many):
    ([[367, 1]], 32, 32, 64),        # 736
    ([[300, 68]] + [[368]], 33, 33, 60),   # 1518: two rows whose tiles meet
    ([[400, 368]], 128, 32, 36),     # 1536, four query heads per KV head
    ([[700, 67]], 128, 32, 64),      # 1536, the last tile one short
    ([[1000, 24]], 32, 32, 20),      # 2048
])
def test_parts_of_shared_tiles(lengths, hq, hkv, d):
    w = wl.make_custom(lengths, hq, hkv, d, "f32", seed=83)
    got = run_gpu(w, grad_dtype=torch.float32, nan_fill=True)
    assert_close(got, run_oracle(w), "f32")
    again = run_gpu(w, grad_dtype=torch.float32, nan_fill=True)
    for key in ("dQ", "dK", "dV"):
        assert np.array_equal(got[key], again[key]), key   # the parts are added in a fixed order
