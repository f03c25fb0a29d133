"""GPU parity of the FP6 GEMM's K-split kernel: one shape per instantiated tile
at which the dispatch picks it (ragged rows and channels, fewer k blocks than
wavefronts, partial last tiles), and the neighbouring shapes of the 192 x 256
kernel.  Accumulators and outputs bit for bit against the CPU oracle."""

import numpy as np
import pytest

import workloads
from oracle import qlinear_acc_ref
from paritylib import assert_acc, oracle_y, safe_w_scales

torch = pytest.importorskip("torch")
dptq = pytest.importorskip("paper_2606_12487_amd")

pytestmark = pytest.mark.gpu

CASES = [
    # (M, N, K)              blocks of 32 (n x m), wavefronts, stages each
    (10, 32, 128),         # 1 x 1, 8, 2: seven wavefronts without a k block
    (33, 1040, 1152),      # 1 x 1, 8, 2: N % 32 == 16, 9 k blocks
    (34, 5344, 128),       # 1 x 2, 8, 2
    (68, 9744, 128),       # 2 x 2, 4, 1: several workgroups a compute unit
    (1023, 2320, 1152),    # the same, ragged
    (8, 9680, 128),        # 2 x 2, 4, 2
    (99, 5328, 1920),      # the same, 15 k blocks
    (68, 8336, 384),       # 2 x 3, 4, 2
    (500, 2064, 2176),     # the same, 17 k blocks
    (98, 8464, 1920),      # 2 x 4, 4, 2
    (258, 10016, 1408),    # 4 x 3, 4, 1
    (331, 8416, 2048),     # 4 x 4, 4, 1: the sum takes several passes
    (517, 10928, 384),     # the 192 x 256 kernel at its fewest stages
    # its clamped variant: one and two stages, too few rows, too few channels
    (777, 11024, 128), (1029, 6160, 256), (217, 28688, 384), (65569, 160, 128),
]


@pytest.mark.parametrize("M,N,K", CASES)
def test_fp6_ksplit_tiles(M, N, K):
    rng = np.random.default_rng([M, N, K])
    a = workloads.random_weight_bytes(rng, M, K)
    w = workloads.random_weight_bytes(rng, N, K)
    a_s = workloads.random_scales(rng, M, 1e-3, 1.0)
    w_s = safe_w_scales(rng, N, K, a_s, 4)
    d = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (a, w, a_s, w_s)]
    a6, w6 = dptq.pack_fp6(d[0]), dptq.pack_fp6(d[1])
    acc_ref = qlinear_acc_ref(a, 4, w)
    assert_acc(dptq.qlinear_fp6_acc(a6, w6, M, K, N).cpu().numpy(), acc_ref, f"{M}x{N}x{K} acc")
    y = dptq.qlinear_fp6(a6, d[2], w6, d[3], M, K, N).cpu().numpy()
    bad = np.nonzero(y.view(np.uint16) != oracle_y(acc_ref, a_s, w_s).view(np.uint16))
    assert bad[0].size == 0, f"{bad[0].size} outputs differ, first at {bad[0][0]},{bad[1][0]}"


@pytest.mark.parametrize("off", [1, 2, 3])
def test_fp6_ksplit_scales_off_16_bytes(off):
    # The entry point takes scales that start at any multiple of 4 bytes.
    M, N, K = 500, 2064, 256
    rng = np.random.default_rng(off)
    a = workloads.random_weight_bytes(rng, M, K)
    w = workloads.random_weight_bytes(rng, N, K)
    a6, w6 = (dptq.pack_fp6(torch.from_numpy(v).cuda()) for v in (a, w))
    a_s = workloads.random_scales(rng, M, 1e-3, 1.0)
    w_s = safe_w_scales(rng, N, K, a_s, 4)
    ad, wd = (torch.from_numpy(np.concatenate([np.full(off, np.nan, np.float32), v])).cuda()[off:] for v in (a_s, w_s))
    y = dptq.qlinear_fp6(a6, ad, w6, wd, M, K, N).cpu().numpy()
    ref = oracle_y(qlinear_acc_ref(a, 4, w), a_s, w_s)
    assert np.array_equal(y.view(np.uint16), ref.view(np.uint16))


def test_fp6_rows_beyond_4_gib():
    # 32-row blocks whose byte offset is past 2^32 (3072 bytes each), on a shape
    # of the 192 x 256 kernel's clamped variant; the last rows against the int8 GEMM.
    M, N, K = (2 ** 32 // 3072 + 8) * 32, 16, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    a = torch.randint(0, 256, (M, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    a_s = torch.rand((M,), generator=g, device="cuda")
    w_s = torch.rand((N,), generator=g, device="cuda") * 1e-3
    y = dptq.qlinear_fp6(dptq.pack_fp6(a), a_s, dptq.pack_fp6(w), w_s, M, K, N)
    for rows in (slice(0, 512), slice(M - 512, M)):
        ref = dptq.qlinear(a[rows], a_s[rows], 4, w, w_s)
        assert torch.equal(y[rows].view(torch.int16), ref.view(torch.int16)), rows
