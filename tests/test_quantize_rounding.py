"""The quantizer's quotient: one product with the reciprocal of the scale and
Markstein's correction, instead of a division per weight."""
import numpy as np
import pytest

import oracle as O
from paper_2608_15383_amd.inputs import bf16_bits_to_f32

M = np.arange(128, 256) / 128.0   # the bf16 significands
EXPONENTS = range(15)             # below 2^-14 of the maximum every code is 0


def test_corrected_product_rounds_as_the_division():
    """All bf16 significands of a weight and of the group's maximum, over the
    exponents between them (both scale by powers of two); the fused operations
    in 64-bit significands, which hold their products exactly."""
    f, ld = np.float32, np.longdouble
    assert np.finfo(ld).nmant >= 63
    s = (M.astype(f) / f(7))[None, :]
    y = f(1) / s
    for e in EXPONENTS:
        w = (M * 2.0 ** -e).astype(f)[:, None]
        ok = w <= M.astype(f)[None, :]
        q = w * y
        r = (w.astype(ld) - q.astype(ld) * s.astype(ld)).astype(f)
        quot = (q.astype(ld) + r.astype(ld) * y.astype(ld)).astype(f)
        assert np.array_equal(np.rint(quot)[ok], np.rint(w / s)[ok]), e


@pytest.mark.gpu
def test_gpu_codes_over_all_significands():
    """Group (a, e): maximum M[a] and the weights M[j] * 2^-e below it, signs
    alternating; codes and scales equal the oracle's."""
    from paper_2608_15383_amd import api
    from paper_2608_15383_amd.inputs import LayerShape, f32_to_bf16_bits, make_layer
    from tests._gpu import dims_of, quantize
    from tests.test_gpu_parity import _check_codes
    shape = LayerShape(2048, 128, 1, 1)
    lay = make_layer(shape, 1, seed=1)
    g = np.zeros((2048, 128), np.float32)
    i = 0
    for e in EXPONENTS:
        for a in range(128):
            w = M * 2.0 ** -e
            w = np.where(w <= M[a], w, 0.0)
            w[-1 if w[-1] == 0 else 0] = M[a]
            g[i] = w * np.where(np.arange(128) % 2, -1, 1)
            i += 1
    lay.w_gate = f32_to_bf16_bits(g.reshape(1, 128, 2048))
    assert np.array_equal(bf16_bits_to_f32(lay.w_gate).reshape(2048, 128), g)
    dm = dims_of(shape)
    _check_codes(dm, lay, quantize(dm, lay), [0])
