"""GPU parity of the K-split GEMM (small output tiles whose wavefronts split K)
at the shapes where it can go wrong: each of its tiles, ragged M and N
(remainders of 16-token and of 16-channel blocks), K that is not a multiple of
256 (a last stage of 128 k, row starts off the 128-byte lines) and K with
fewer stages than wavefronts.  The labels are the dispatch's choice at 256
compute units; test_gemm_rules.py checks that every tile is among them.

Bar: accumulators and fp16 outputs bit for bit against the oracle's exact GEMM
and pinned epilogue, for canonical weights, the 8-bit activation order and the
zero-point correction.  All arithmetic up to the epilogue is integer, so there
is no tolerance.
"""

import numpy as np
import pytest

import workloads
from oracle.range_quant import weight_sums_ref, zero_point_acc_ref
from paritylib import assert_acc, oracle_acc, oracle_y, safe_w_scales

torch = pytest.importorskip("torch")
dptq = pytest.importorskip("paper_2606_12487_amd")

pytestmark = pytest.mark.gpu

CASES = [
    # (M, K, N, bits).  At most 16 tokens: one or two blocks of 16 channels on eight
    # or four wavefronts.
    (13, 2176, 4128, 8), (9, 2432, 272, 4),                    # 1 x 8
    (16, 384, 10256, 4), (11, 896, 10256, 8),                  # 2 x 4
    (5, 640, 4624, 8), (9, 2176, 16400, 8), (3, 640, 4624, 4), (7, 384, 16400, 4),   # 2 x 8
    # The kernel that streams the weights into registers, at its K; one and two blocks.
    (1, 128, 16, 4), (13, 384, 272, 8), (3, 384, 3088, 4), (16, 128, 32768, 4), (16, 384, 16416, 8),
    # The tiles of larger batches, as TI x TJ x wavefronts.
    (17, 128, 16, 4), (18, 384, 48, 8), (17, 128, 2064, 4), (17, 128, 6160, 4),  # 1 x 1 x 8
    (31, 640, 2064, 8), (17, 2432, 2448, 4),                # 1 x 2 x 8
    (18, 384, 7088, 4), (18, 384, 6416, 8),                 # 2 x 2 x 8
    (33, 1920, 4240, 4), (33, 1920, 4240, 8),               # 2 x 3 x 8
    (50, 2944, 4112, 4),                                    # 2 x 4 x 8
    (33, 2688, 8560, 4), (37, 896, 8496, 8),                # 4 x 3 x 8
    (33, 640, 6160, 4), (63, 384, 6160, 4), (129, 384, 4112, 4), (300, 128, 3088, 4),  # 2 x 2 x 4
    (161, 896, 6160, 4), (97, 384, 11024, 4), (18, 1152, 8608, 4),
    (33, 896, 9072, 4),                                     # 2 x 3 x 4
    (47, 896, 4112, 8), (33, 384, 6160, 8), (129, 384, 4112, 8), (97, 384, 11024, 8),  # 2 x 4 x 4
    (161, 896, 8208, 8), (52, 1152, 12304, 4), (33, 1152, 4256, 8),
    (512, 1408, 3728, 4), (50, 2432, 8224, 8), (299, 1408, 6416, 4), (49, 2176, 10288, 8),  # 4 x 4 x 4
    (163, 2176, 8272, 8), (146, 6272, 8448, 4), (149, 6272, 8496, 4),  # 8 x 4 x 4
    (97, 1920, 12960, 8), (97, 1920, 12848, 8),             # 4 x 8 x 4
    (99, 4992, 12416, 4), (98, 4992, 12432, 4),
    (17, 640, 11024, 8), (300, 128, 3088, 8), (129, 1408, 11024, 8), (20, 256, 8800, 8),  # 4 x 2 x 4
    (17, 1152, 8704, 8),
    (161, 2432, 6160, 8), (65, 1408, 12480, 8),             # 4 x 6 x 4
]


def _d(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _h(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("M,K,N,bits", CASES)
def test_ksplit_matches_oracle(M, K, N, bits):
    rng = np.random.default_rng([M, K, N, bits])
    a = workloads.random_code_bytes(rng, M, K, bits)
    w = workloads.random_weight_bytes(rng, N, K)
    a_s = workloads.random_scales(rng, M, 1e-3, 1.0)
    w_s = safe_w_scales(rng, N, K, a_s, bits)
    ad, wd, asd, wsd = _d(a), _d(w), _d(a_s), _d(w_s)
    acc = oracle_acc(a, bits, w)
    what = f"{M}x{K}x{N} A{bits}"
    assert_acc(_h(dptq.qlinear_acc(ad, bits, wd)), acc, what)
    y_ref = oracle_y(acc, a_s, w_s).view(np.uint16)
    assert np.array_equal(_h(dptq.qlinear(ad, asd, bits, wd, wsd)).view(np.uint16), y_ref), what
    if bits == 8:
        y = dptq.qlinear_a8(ad, asd, dptq.pack_w4_a8(wd), wsd)
        assert np.array_equal(_h(y).view(np.uint16), y_ref), what + " 8-bit order"
    zeros = rng.integers(0, 2 ** bits, size=M).astype(np.int32)
    sums = weight_sums_ref(w)
    z_ref = oracle_y(zero_point_acc_ref(acc, zeros, bits, sums), a_s, w_s * np.float32(0.25))
    y = dptq.qlinear_range(ad, asd, _d(zeros), bits, wd, _d(w_s * np.float32(0.25)), _d(sums.astype(np.int32)))
    assert np.array_equal(_h(y).view(np.uint16), z_ref.view(np.uint16)), what + " zero points"
