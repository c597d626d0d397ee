"""Parity of the size- and alignment-dependent kernel variants at the edges of their ranges:
the wide quantiser against the oracle at ties."""
import numpy as np
import pytest
import torch

import oracle
import synthetic
from paper_2607_21604_amd import akvs
from tests.gpu_util import DEV, f64, to_dev

pytestmark = pytest.mark.gpu


def _near_ties(rows, hd, bits, seed):
    """fp32 values on and beside the quantiser's rounding boundaries of their group."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, hd)).astype(np.float32)
    if bits == 8:
        scale = np.float32(0.25)
        pos = oracle.e4m3_value(np.arange(0x7F))
        mid = ((pos[:-1] + pos[1:]) / 2).astype(np.float32)
        v = scale * rng.choice(mid, size=(rows, hd)) * rng.choice([-1, 1], size=(rows, hd))
        v[:, ::64] = 448 * scale
    else:
        top = 2 ** bits - 1
        scale, zero = np.float32(0.3125), np.float32(-1.5)
        v = zero + scale * (rng.integers(0, top, size=(rows, hd)) + np.float32(0.5))
        v[:, ::64], v[:, 1::64] = zero, zero + top * scale
    v = v.astype(np.float32)
    step = rng.integers(-1, 2, size=v.shape)
    step[:, ::64] = step[:, 1::64] = 0
    v = np.where(step == 0, v, np.nextafter(v, np.where(step > 0, np.inf, -np.inf),
                                            dtype=np.float32))
    x[::2] = v[::2]
    return x


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("rows,hd", [(1, 64), (33, 192), (127, 128), (257, 64)])
def test_quantise_codes_at_ties(bits, rows, hd):
    """Bit-exact codes and metadata at the rounding boundaries, for block remainders, fp32 and
    bf16 inputs, and operands that miss the wide kernel's alignment."""
    x32 = torch.from_numpy(_near_ties(rows, hd, bits, 7 * rows + bits))
    for x in (x32, x32.to(torch.bfloat16)):
        if bits == 8:
            codes, meta = oracle.quantize_e4m3_g64(f64(x))
        else:
            codes, meta = oracle.quantize_g64(f64(x), bits)
            codes = oracle.pack_codes(codes, bits)
        for shift in (0, 1):  # one element off: not 16-byte aligned
            buf = torch.zeros(rows * hd + shift, dtype=x.dtype, device=DEV)
            xd = buf[shift:].view(rows, hd)
            xd.copy_(x)
            c = torch.full((rows, hd * bits // 8), 0xA5, dtype=torch.uint8, device=DEV)
            mt = torch.empty((rows, hd // 64, 2), dtype=torch.float16, device=DEV)
            akvs.akvs_quantize_cache(xd, rows, hd, bits, c, mt)
            np.testing.assert_array_equal(c.cpu().numpy(), codes)
            np.testing.assert_array_equal(mt.cpu().numpy().view(np.uint16), meta.view(np.uint16))
