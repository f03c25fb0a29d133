"""GPU parity of rotate + quantize for rows of one 28 * 2^j block (j = 9, 10),
whose 28-point stage runs on the fp32 matrix cores: codes (4 and 8 bits and the
FP6 layout), scales and randomized signs bit for bit against the CPU oracle, on
both sides of the row counts from which that kernel is taken, with rows that
stress the order and rounding of the sums (wide ranges, zeros, fp16 subnormals,
the largest values)."""

import numpy as np
import pytest

from oracle import rotate_quant_ref
from paritylib import fp6_layout_ref

torch = pytest.importorskip("torch")
dptq = pytest.importorskip("paper_2606_12487_amd")

pytestmark = pytest.mark.gpu


def _rows(M, K, seed):
    rng = np.random.default_rng([M, K, seed])
    x = rng.standard_t(3, (M, K)).astype(np.float32)
    x[0] *= np.exp2(rng.integers(-14, 12, K)).astype(np.float32)   # wide range within a row
    if M > 4:
        x[1] = 0
        x[2] *= np.float32(2.0 ** -22)                             # fp16 subnormals
        x[3] = rng.choice([-65504.0, 65504.0], K)                  # the largest sums
        x[4] = 0
        x[4, K - 1] = 1
    return x.clip(-65504, 65504).astype(np.float16)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("K", [28 * 512, 28 * 1024])
@pytest.mark.parametrize("M", [7, 65, 256, 257])
def test_rq28_matches_oracle(M, K, bits):
    x = _rows(M, K, bits)
    c_ref, s_ref = rotate_quant_ref(x, K, bits)
    xd = torch.from_numpy(x).cuda()
    c, s = dptq.rotate_quant(xd, K, bits)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(c.cpu().numpy().view(np.uint8), np.asarray(c_ref).view(np.uint8))
    if bits == 4:
        a6, s6 = dptq.rotate_quant_fp6(xd, K)
        assert np.array_equal(s6.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
        assert np.array_equal(a6.cpu().numpy(), fp6_layout_ref(np.asarray(c_ref).view(np.uint8), K))


@pytest.mark.parametrize("M,K", [(65, 28 * 512), (257, 28 * 1024)])
def test_rq28_signs(M, K):
    x = _rows(M, K, 3)
    signs = np.random.default_rng(K).integers(0, 256, K // 8).astype(np.uint8)
    neg = np.unpackbits(signs, bitorder="little").astype(bool)
    c_ref, s_ref = rotate_quant_ref(np.where(neg, -x, x), K, 8)
    c, s = dptq.rotate_quant(torch.from_numpy(x).cuda(), K, 8, signs=torch.from_numpy(signs).cuda())
    assert np.array_equal(s.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(c.cpu().numpy().view(np.uint8), np.asarray(c_ref).view(np.uint8))
