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
    exponents between them (both scale by powers of two) and some past the last
    nonzero code: the quotient itself, so the rounded one too; the fused
    operations in 64-bit significands, which hold their products exactly."""
    f, ld = np.float32, np.longdouble
    assert np.finfo(ld).nmant >= 63
    s = (M.astype(f) / f(7))[None, :]
    y = f(1) / s
    for e in range(24):
        w = (M * 2.0 ** -e).astype(f)[:, None]
        ok = w <= M.astype(f)[None, :]
        q = w * y
        r = (w.astype(ld) - q.astype(ld) * s.astype(ld)).astype(f)
        quot = (q.astype(ld) + r.astype(ld) * y.astype(ld)).astype(f)
        assert np.array_equal(quot[ok], (w / s)[ok]), e


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


@pytest.mark.gpu
def test_gpu_codes_of_groups_without_a_scale():
    """A group whose scale is 0 (zeros, NaN, or a maximum below fp16's range)
    has code 0 throughout, a NaN beside a scale the lowest code; beside an
    infinite weight, which the call refuses, finite weights keep code 0."""
    import torch
    from paper_2608_15383_amd import api
    from paper_2608_15383_amd.inputs import LayerShape, f32_to_bf16_bits, make_layer
    from tests._gpu import dev, dims_of
    shape = LayerShape(256, 128, 1, 1)
    lay = make_layer(shape, 1, seed=2)
    dm = dims_of(shape)

    def codes(special):
        """Codes of gate row 0, group 0: dword lane 16q + n of a tile holds row
        n, inputs 32i + 8q + r at bits 4 (r / 2) + 16 (r % 2) of dword i."""
        w = bf16_bits_to_f32(lay.w_gate).reshape(1, 128, 256).copy()
        w[0, 0, :128] = special
        bank = torch.zeros(api.expert_record_bytes(dm), dtype=torch.uint8, device="cuda")
        err = False
        try:
            api.quantize_experts(dm, dev(f32_to_bf16_bits(w)), dev(lay.w_up), dev(lay.w_down), bank)
        except Exception:
            err = True
        torch.cuda.synchronize()
        dw = bank[:1024].cpu().numpy().view(np.uint32).reshape(64, 4)
        j = np.arange(128)
        i, q, r = j // 32, j % 32 // 8, j % 8
        return (dw[16 * q, i] >> (4 * (r // 2) + 16 * (r % 2))) & 15, err

    x = np.zeros(128, np.float32)
    for fill in (0.0, np.nan, 2.0 ** -30):
        x[:] = 0.0
        x[::3] = fill
        got, err = codes(x)
        assert (got == 8).all() and not err, fill
    x[:] = 1.0
    x[5] = np.nan
    got, err = codes(x)
    assert got[5] == 0 and (np.delete(got, 5) == 15).all() and not err
    x[5] = np.inf
    got, err = codes(x)
    assert got[5] == 0 and (np.delete(got, 5) == 8).all() and err
