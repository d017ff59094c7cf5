"""GPU: the row quantizer over every (row maximum, element) pair of bf16 significands, and beside
zeros of both signs, subnormals, infinities and NaN.

A row's scale follows from its maximum, so the 128 significands of the maximum with every bf16
value of the 20 binades below it (smaller elements have code 0) are all the quotients there are
at one exponent; codes and scales against the oracle bit for bit.
"""

import numpy as np
import pytest
import torch

from oracle import e4m3, quant

pytestmark = pytest.mark.gpu


def _quantize(bits):
    from paper_2602_10718_amd import snapmla as sm
    x = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)
    codes = torch.empty(bits.shape, dtype=torch.uint8, device="cuda")
    scale = torch.empty(len(bits), dtype=torch.float32, device="cuda")
    sm.snapmla_quantize_rows(x, codes, scale)
    return codes.cpu().numpy(), scale.cpu().numpy()


@pytest.mark.parametrize("exponent", [25, 88, 95, 127, 254])     # 95: scales at the floor 2^-40 and just above
def test_every_quotient(exponent):
    rows = []
    for top in range(exponent << 7, (exponent + 1) << 7):
        x = np.arange(max(0, top - (20 << 7)), top + 1)
        x = np.concatenate([x, x | 0x8000])
        x = np.concatenate([x, np.zeros(-len(x) % 511, x.dtype)]).reshape(-1, 511)
        rows.append(np.concatenate([np.full((len(x), 1), top), x], 1))
    bits = np.concatenate(rows).astype(np.uint16)
    codes, scale = _quantize(bits)
    c_ref, s_ref = quant.quantize_rows(bits)
    assert np.array_equal(scale.view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(codes, c_ref)


def test_zeros_infinities_and_nan():
    bits = np.zeros((6, 512), np.uint16)
    bits[:] = np.arange(512) % 510 * 64          # finite values of every exponent
    bits[:, 1::2] |= 0x8000
    bits[0] = 0
    bits[0, ::2] = 0x8000                        # only zeros
    bits[1, 7] = 0x7F80                          # an infinite maximum: finite elements 0, infinities NaN
    bits[2, 9], bits[2, 10] = 0xFF80, 0x7FC0
    bits[3, 11], bits[3, 12] = 0x7FC0, 0xFFC1    # NaN elements do not count towards the maximum
    bits[4] = np.where(np.arange(512) % 3 == 0, 0x0001, 0x8001)      # the smallest subnormals
    bits[5] = 0x7FC0
    codes, scale = _quantize(bits)
    x = quant.bf16_to_f32(bits)
    with np.errstate(all="ignore"):
        top = np.fmax.reduce(np.abs(x), axis=1, initial=np.float32(0))
        s_ref = np.maximum(top / np.float32(448), quant.EPS).astype(np.float32)
        y = (x / s_ref[:, None]).astype(np.float32)
    y = np.where(np.isnan(y), np.float32(-448), y)           # the clamp turns a NaN into its lower end
    assert np.array_equal(scale.view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(codes, e4m3.encode(y))
