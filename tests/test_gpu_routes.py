"""GPU tests of the layer call's size-dependent routes: the router's slices of
d, the fused top-k and grouping, and the row sums that ride with the top-k."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as O
from paper_2608_15383_amd import api
from paper_2608_15383_amd.inputs import LayerShape, bf16_bits_to_f32, make_layer

from _gpu import Layer, assert_close_rel, dev, dims_of

pytestmark = pytest.mark.gpu


def _y_ref(lay, r, k):
    """fp64 layer output of the oracle for the routing r."""
    experts = [O.quantize_expert(lay.f32("w_gate")[e], lay.f32("w_up")[e], lay.f32("w_down")[e])
               for e in range(lay.shape.n_experts)]
    return O.moe_forward(lay.f32("h"), experts, r)


# One, two and four slices of d and none (d not a multiple of 512); tokens on
# both sides of the fused top-k and grouping (16, and 64 experts) and of the
# wide grouping (1024 pairs), with k dividing 64 or not; a partial token and
# expert tile.
@pytest.mark.parametrize("shape,tokens", [
    (LayerShape(512, 128, 6, 2), 5), (LayerShape(1024, 128, 17, 3), 16),
    (LayerShape(2048, 128, 64, 8), 17), (LayerShape(2048, 128, 200, 8), 64),
    (LayerShape(1024, 128, 64, 8), 65), (LayerShape(640, 128, 12, 3), 64),
    (LayerShape(640, 128, 12, 3), 343), (LayerShape(384, 128, 16, 8), 130),
    (LayerShape(2048, 128, 16, 8), 129), (LayerShape(1024, 128, 64, 8), 16),
    (LayerShape(1024, 128, 64, 64), 16), (LayerShape(640, 128, 64, 8), 17),
    (LayerShape(1024, 128, 65, 8), 16)])
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


@pytest.mark.parametrize("experts,tokens,launches", [
    (64, 5, 5), (64, 16, 5), (64, 17, 6), (64, 64, 6), (65, 16, 6), (200, 5, 6), (8, 16, 5), (8, 17, 6)])
def test_one_routing_launch_only_for_the_smallest_calls(experts, tokens, launches):
    """Above 16 tokens or 64 experts the top-k keeps its own launch: all tokens
    on one compute unit cost more there than the launch saved."""
    shape = LayerShape(512, 128, experts, 4)
    lay = make_layer(shape, tokens, seed=5)
    st = api.Stats()
    Layer(dims_of(shape), lay, tokens).forward(lay.h, stats=st)
    assert st.kernel_launches == launches  # router, routing (1 or 2), gate/up, down, combine


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


# Experts on both sides of the scans' blocks of 64; pairs on both sides of the
# one-workgroup grouping (1024) and of a pass over the chunk counts (64 chunks
# above 64 experts, 256 below); k = 5 takes the counts' own launch.
@pytest.mark.parametrize("experts", [64, 65, 128, 129, 192, 193, 256])
@pytest.mark.parametrize("tokens,k", [(1, 8), (4, 8), (128, 8), (129, 8), (207, 5), (512, 8),
                                      (513, 8), (2100, 8), (64, 17)])
def test_grouping_over_blocks_of_experts_equals_the_oracle(experts, tokens, k):
    """Every array of the grouping, in a layer call (up to 4 tokens also the
    fused launch) and in emoe_route; a third of the experts never chosen, so
    the active list has gaps in every block."""
    shape = LayerShape(128, 128, experts, k)
    lay = make_layer(shape, tokens, seed=17)
    layer = Layer(dims_of(shape), lay, tokens)
    rng = np.random.default_rng([experts, tokens])
    z = rng.standard_normal((tokens, experts)).astype(np.float32)
    z[:, ::3] -= 50
    pairs = tokens * k
    ids = O.topk_experts(z, k)
    gr = O.group_by_expert(ids, experts)
    tiles = np.concatenate([[0], np.cumsum((gr.counts + 63) // 64)]).astype(np.int32)
    pos = np.empty(pairs, np.int32)
    pos[gr.sorted_pairs] = np.arange(pairs, dtype=np.int32)
    want = dict(topk_ids=ids.reshape(-1), counts=gr.counts, offsets=gr.offsets,
                sorted_pairs=gr.sorted_pairs, active=gr.active, n_active=[len(gr.active)],
                tile_offsets=tiles, pair_pos=pos)
    for path in (api.EMOE_PATH_MFMA, api.EMOE_PATH_AUTO):
        layer.ws.fill_(0xA5)
        st = api.Stats()
        layer.forward(lay.h, logits=z, path=path, stats=st)
        fused = st.kernel_launches == 1   # writes no row tiles
        assert fused == (tokens <= 4 and path == api.EMOE_PATH_AUTO)
        for name, w in want.items():
            got = layer.ws_array(name, len(w), np.int32)
            assert (fused and name == "tile_offsets") or np.array_equal(got, np.asarray(w, np.int32)), name
    i32 = lambda n: torch.full((n,), -1, dtype=torch.int32, device="cuda:0")
    out = dict(topk_ids=i32(pairs), counts=i32(experts), offsets=i32(experts + 1),
               sorted_pairs=i32(pairs), active=i32(experts), n_active=i32(1))
    api.route(layer.dm, tokens, dev(lay.h), layer.wr, dev(z), True, None, out["topk_ids"],
              torch.empty(pairs, device="cuda:0"), out["counts"], out["offsets"],
              out["sorted_pairs"], out["active"], out["n_active"])
    for name, t in out.items():
        w = np.asarray(want[name], np.int32)
        assert np.array_equal(t.cpu().numpy()[:len(w)], w), name
