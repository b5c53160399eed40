"""GPU tests of the decode step (one to four tokens) over a given key/value
cache: every head size, cache lengths on both sides of a round of keys, and a
row too wide for the norm inside the QKV projection."""
import numpy as np
import pytest
import torch

from oracle import decoder_oracle as D
from paper_2608_15383_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits
from tests._gpu import dev
from tests.test_gpu_decoder import GpuDecoder, _check_logits, _model, _oracle_weights

pytestmark = pytest.mark.gpu


# A round of keys is 512 positions; 20 values per stripe are 640, 320 and 160.
@pytest.mark.parametrize("heads,head_dim,pos0,tokens", [
    (4, 64, 0, 4), (4, 64, 1025, 1), (4, 64, 127, 2), (2, 128, 0, 1), (2, 128, 1, 3),
    (2, 128, 63, 1), (2, 128, 318, 4), (2, 128, 513, 1), (1, 256, 31, 2), (1, 256, 159, 4),
    (17, 128, 70, 3), (1, 256, 513, 1), (1, 256, 510, 4), (2, 128, 1022, 3), (1, 256, 8185, 4)])
def test_step_over_a_given_cache_matches_the_oracle(heads, head_dim, pos0, tokens):
    """Two layers, so the second layer's norm takes the experts' output."""
    d = heads * head_dim
    shape = D.DecoderShape(n_layers=2, d_model=d, n_heads=heads, head_dim=head_dim, vocab=300,
                           d_ff=128, n_experts=4, top_k=2)
    m = _model(shape, seed=41)
    max_pos = pos0 + tokens + 3
    gpu = GpuDecoder(shape, m, 4, max_positions=max_pos, max_tokens=4)
    try:
        rng = np.random.default_rng(pos0 + tokens)
        past = f32_to_bf16_bits(rng.standard_normal((2, 2, pos0, d)).astype(np.float32))
        full = np.zeros((2, 2, max_pos, d), np.uint16)
        full[:, :, :pos0] = past
        gpu.kv.copy_(dev(full).view(torch.uint8).reshape(-1))
        kv = D.KVState()
        if pos0:
            rows = bf16_bits_to_f32(past).astype(np.float64).reshape(2, 2, pos0, heads, head_dim)
            kv.k = [rows[l, 0] for l in range(2)]
            kv.v = [rows[l, 1] for l in range(2)]
        seq = list(rng.integers(0, 300, tokens))
        got, _ = gpu.run(seq, pos0)
        _, ref, _ = D.decoder_forward(shape, _oracle_weights(shape, m), seq, kv)
        _check_logits(got, ref, f"H={heads} Dh={head_dim} pos0={pos0} T={tokens}")
        after = bf16_bits_to_f32(gpu.kv.cpu().numpy().view(np.uint16)).reshape(2, 2, max_pos, d)
        # The old positions and those past the call are untouched; the new ones
        # hold the rotated keys and the values (bf16: 2^-8 of the largest).
        assert np.array_equal(after[:, :, :pos0], bf16_bits_to_f32(past))
        assert not after[:, :, pos0 + tokens:].any()
        for l in range(2):
            for which, want in ((0, kv.k[l]), (1, kv.v[l])):
                w = want[pos0:].reshape(tokens, d)
                err = np.abs(after[l, which, pos0:pos0 + tokens] - w).max() / np.abs(w).max()
                assert err <= 2e-2, (l, which, err)
    finally:
        gpu.close()


# Both sides of the first 512 keys, of 20 values a stripe (640, 320, 160) and of
# the last position of the default rule (1536; 1024 above head size 64), head
# size 256 with its key row in several parts and more than one round, and the
# longest cache.
@pytest.mark.parametrize("heads,head_dim,pos0,tokens", [
    (2, 64, 0, 4), (2, 64, 637, 4), (2, 64, 1535, 1), (2, 64, 4001, 3), (1, 128, 0, 1),
    (1, 128, 509, 4), (2, 128, 1023, 1), (1, 128, 2099, 2), (1, 256, 158, 4), (1, 256, 510, 4),
    (1, 256, 513, 1), (1, 256, 1025, 2), (1, 256, 8188, 4)])
def test_step_attention_gives_the_bits_of_the_prompt_launches(heads, head_dim, pos0, tokens):
    """The one-launch rotation and attention of a step against the rotation
    and attention launches of prompts: logits, token and cache bit for bit."""
    d = heads * head_dim
    shape = D.DecoderShape(n_layers=2, d_model=d, n_heads=heads, head_dim=head_dim, vocab=300,
                           d_ff=128, n_experts=4, top_k=2)
    m = _model(shape, seed=43)
    max_pos = pos0 + tokens
    gpu = GpuDecoder(shape, m, 4, max_positions=max_pos, max_tokens=4)
    try:
        rng = np.random.default_rng(pos0 + tokens)
        past = np.zeros((2, 2, max_pos, d), np.uint16)
        past[:, :, :pos0] = f32_to_bf16_bits(rng.standard_normal((2, 2, pos0, d)).astype(np.float32))
        seq = list(rng.integers(0, 300, tokens))
        out = []
        for keys in (max_pos, max_pos - 1, -1):   # one launch, two, the rule's choice
            gpu.dec.set_step_keys(keys)
            gpu.kv.copy_(dev(past).view(torch.uint8).reshape(-1))
            gpu.logits.fill_(float("nan"))
            logits, tok = gpu.run(seq, pos0)
            out.append((logits.view(np.uint32), tok, gpu.kv.cpu().numpy().copy()))
        assert np.isfinite(out[0][0].view(np.float32)).all()
        for got in out[1:]:
            assert np.array_equal(got[0], out[0][0]) and got[1] == out[0][1]
            assert np.array_equal(got[2], out[0][2])
    finally:
        gpu.close()
