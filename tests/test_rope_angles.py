"""The decoder's rotary angles over every position it allows: the fp64 cosine
and sine of csrc/decoder.hip (rope_cos_sin), and the rotated keys it appends."""
import math
from fractions import Fraction

import numpy as np
import pytest

MAX_POSITIONS, BASE = 8192, 10000.0


def _fma(a, b, c):
    """a * b + c with one rounding (a Fraction's float is correctly rounded)."""
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _cos_sin(x):
    """rope_cos_sin's operations in their order."""
    n = float(round(x * 0.63661977236758134308))
    r = _fma(-n, 1.5707963267948965580, x)
    r = _fma(-n, 6.1232339957367660359e-17, r)
    z = r * r
    ps = _fma(z, 1.0 / 355687428096000.0, -1.0 / 1307674368000.0)
    for k in (1.0 / 6227020800.0, -1.0 / 39916800.0, 1.0 / 362880.0, -1.0 / 5040.0, 1.0 / 120.0,
              -1.0 / 6.0):
        ps = _fma(z, ps, k)
    sn = _fma(r * z, ps, r)
    pc = _fma(z, 1.0 / 20922789888000.0, -1.0 / 87178291200.0)
    for k in (1.0 / 479001600.0, -1.0 / 3628800.0, 1.0 / 40320.0, -1.0 / 720.0, 1.0 / 24.0, -0.5,
              1.0):
        pc = _fma(z, pc, k)
    k = int(n) & 3
    a, b = (sn, pc) if k & 1 else (pc, sn)
    return (-a if k in (1, 2) else a), (-b if k >= 2 else b)


def test_cosine_and_sine_over_every_allowed_angle():
    """Angles p * base^(-2i/Dh) up to position 8191, and the points around
    multiples of pi/2, where the reduction cancels.  The C library's results are
    within an ulp of the exact value (1.1e-16); so is this evaluation: 4e-16."""
    rng = np.random.default_rng(1)
    xs = [0.0, 1.0, 8191.0, 8192.0]
    for _ in range(1500):
        dh = int(rng.choice([64, 128, 256]))
        i = int(rng.integers(0, dh // 2))
        xs.append(float(rng.integers(0, MAX_POSITIONS)) * BASE ** (-2.0 * i / dh))
    for n in [1, 2, 3, 4, 5, 1000, 5214, 5215] + list(rng.integers(0, 5215, 200)):
        h = float(n) * (math.pi / 2)
        xs += [h, math.nextafter(h, 0.0), h + 1e-9, h + math.pi / 4]
    for x in xs:
        c, s = _cos_sin(x)
        assert abs(c - math.cos(x)) <= 4e-16 and abs(s - math.sin(x)) <= 4e-16, x


@pytest.mark.gpu
@pytest.mark.parametrize("heads,head_dim", [(2, 64), (1, 128), (1, 256)])
def test_gpu_keys_hold_every_angle(heads, head_dim):
    """A decoder whose keys are (1, .., 1, 0, .., 0) before rotation appends the
    cosine and the sine of every angle as bf16: all positions through a prompt,
    some through steps on both sides of the step's own attention."""
    import torch
    from oracle import decoder_oracle as D
    from paper_2608_15383_amd.inputs import f32_to_bf16_bits
    from tests.test_gpu_decoder import GpuDecoder, _model
    d = heads * head_dim
    shape = D.DecoderShape(n_layers=1, d_model=d, n_heads=heads, head_dim=head_dim, vocab=4,
                           d_ff=128, n_experts=2, top_k=1, rms_eps=0.0)
    m = _model(shape, seed=3)
    ones = f32_to_bf16_bits(np.ones(d, np.float32))
    m["embed"] = np.broadcast_to(ones, (4, d)).copy()   # normalized: exactly 1
    m["attn_norm"] = [ones]
    w = np.zeros((3 * d, d), np.float32)
    half = head_dim // 2
    for h in range(heads):
        w[d + h * head_dim:d + h * head_dim + half, 0] = 1.0
    m["wqkv"] = [f32_to_bf16_bits(w)]
    p = np.arange(MAX_POSITIONS, dtype=np.float64)[:, None]
    ang = p * BASE ** (-2.0 * np.arange(half) / head_dim)
    want = f32_to_bf16_bits(np.concatenate([np.cos(ang), np.sin(ang)], axis=1).astype(np.float32))
    gpu = GpuDecoder(shape, m, 2, max_positions=MAX_POSITIONS, max_tokens=1024)

    def keys():
        return gpu.kv.cpu().numpy().view(np.uint16).reshape(2, MAX_POSITIONS, heads, head_dim)[0]

    try:
        for p0 in range(0, MAX_POSITIONS, 1024):
            gpu.run([0] * 1024, p0)
        got = keys()
        for h in range(heads):
            assert np.array_equal(got[:, h], want)
        gpu.kv.zero_()
        steps = [(0, 1), (5, 4), (511, 2), (1020, 4), (1535, 1), (4097, 3), (8188, 4)]
        for p0, t in steps:
            gpu.dec.set_step_keys(MAX_POSITIONS if p0 != 4097 else -1)
            gpu.run([0] * t, p0)
        got = keys()
        for p0, t in steps:
            for h in range(heads):
                assert np.array_equal(got[p0:p0 + t, h], want[p0:p0 + t]), p0
    finally:
        gpu.close()
