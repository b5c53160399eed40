"""GPU tests of the layer call's size-dependent routes: the router's slices of
d, the fused top-k and grouping, and the row sums that ride with the top-k."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
from paper_2608_15383_amd import api
from paper_2608_15383_amd.inputs import LayerShape, bf16_bits_to_f32, make_layer

from _gpu import Layer, assert_close_rel, dims_of

pytestmark = pytest.mark.gpu


def _y_ref(lay, r, k):
    """fp64 layer output of the oracle for the routing r."""
    experts = [O.quantize_expert(lay.f32("w_gate")[e], lay.f32("w_up")[e], lay.f32("w_down")[e])
               for e in range(lay.shape.n_experts)]
    return O.moe_forward(lay.f32("h"), experts, r)


# One, two and four slices of d and none (d not a multiple of 512); tokens on
# both sides of the fused top-k and grouping (64) and of the wide grouping
# (1024 pairs), with k dividing 64 or not; a partial token and expert tile.
@pytest.mark.parametrize("shape,tokens", [
    (LayerShape(512, 128, 6, 2), 5), (LayerShape(1024, 128, 17, 3), 16),
    (LayerShape(2048, 128, 64, 8), 17), (LayerShape(2048, 128, 200, 8), 64),
    (LayerShape(1024, 128, 64, 8), 65), (LayerShape(640, 128, 12, 3), 64),
    (LayerShape(640, 128, 12, 3), 343), (LayerShape(384, 128, 16, 8), 130),
    (LayerShape(2048, 128, 16, 8), 129)])
@pytest.mark.parametrize("given", [False, True])
def test_layer_routing_equals_the_oracle(shape, tokens, given):
    """Logits, ids, weights and grouping of a layer call on the MFMA path, and
    its output; the logits bit for bit (an fp64 sum rounds to the same fp32
    value whatever its slices at these magnitudes)."""
    lay = make_layer(shape, tokens, seed=31)
    layer = Layer(dims_of(shape), lay, tokens)
    layer.ws.fill_(0xA5)
    k, e = shape.top_k, shape.n_experts
    z = None
    if given:
        z = np.random.default_rng(3).standard_normal((tokens, e)).astype(np.float32)
    y = layer.forward(lay.h, logits=z, path=api.EMOE_PATH_MFMA)
    r = O.route(bf16_bits_to_f32(lay.h), bf16_bits_to_f32(lay.w_router), k, True, z)
    if not given:
        got = layer.ws_array("logits", tokens * e, np.float32).reshape(tokens, e)
        assert np.array_equal(got.view(np.uint32), r.logits.view(np.uint32))
    gr = O.group_by_expert(r.ids, e)
    assert np.array_equal(layer.ws_array("topk_ids", tokens * k, np.int32).reshape(tokens, k), r.ids)
    assert np.array_equal(layer.ws_array("counts", e, np.int32), gr.counts)
    assert np.array_equal(layer.ws_array("offsets", e + 1, np.int32), gr.offsets)
    assert np.array_equal(layer.ws_array("sorted_pairs", tokens * k, np.int32), gr.sorted_pairs)
    assert_close_rel(y, _y_ref(lay, r, k), f"{shape} T={tokens} given={given}")


# More row tiles than co-resident workgroups: 200 experts (four rounds of the
# lanes) with uneven rows, and one expert that takes every pair.
@pytest.mark.parametrize("shape,tokens,skew", [
    (LayerShape(512, 512, 200, 8), 3000, 1.2), (LayerShape(512, 512, 200, 8), 3001, 0.0),
    (LayerShape(512, 512, 65, 4), 8200, 0.4), (LayerShape(256, 256, 1, 1), 33000, 0.0),
    (LayerShape(256, 256, 2, 1), 33001, 3.0)])
def test_many_row_tiles_match_the_gemv_path(shape, tokens, skew):
    """Every row of the MFMA and mixed paths agrees with
    the GEMV path, which has no row tiles."""
    from paper_2608_15383_amd.inputs import zipf_gumbel_logits
    lay = make_layer(shape, tokens, seed=8)
    layer = Layer(dims_of(shape), lay, tokens)
    rng = np.random.default_rng(9)
    z = zipf_gumbel_logits(tokens, shape.n_experts, skew, rng.permutation(shape.n_experts), rng)
    ref = layer.forward(lay.h, logits=z, path=api.EMOE_PATH_GEMV)
    for path in (api.EMOE_PATH_MFMA, api.EMOE_PATH_MIXED):
        y = layer.forward(lay.h, logits=z, path=path)
        rms = np.sqrt((ref.astype(np.float64) ** 2).mean(axis=1))
        err = np.sqrt(((y - ref).astype(np.float64) ** 2).mean(axis=1))
        # bf16 pair outputs and sums in another order: about 2^-8 of a row.
        assert (err <= 2e-2 * rms).all(), (path, int(np.argmax(err / rms)), float((err / rms).max()))
