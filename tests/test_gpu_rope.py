"""Stored keys carry one rounding, whichever kernel projects and rotates them.

The embedding rows are one-hot, so the RMSNorm and the projection are exact in
fp32 and the rotation's inputs are known to the last bit; a stored key is then
the fp16 rounding of v1 cos - fp32(v2 sin) or v2 cos + fp32(v1 sin), rounded
once.  A second rounding (to fp32 on the way) changes about one value in 15000,
enough to show in each of these caches.
"""

import numpy as np
import pytest

from gpu_util import archer, dev_i32, make_ctx, say
from synth.gen import bf16_bits_to_f32, f32_to_bf16_bits, model_weights
from synth.workloads import ModelShape

pytestmark = pytest.mark.gpu


def _expected_k(W, m, tokens, gain):
    d, hd, half = m.d_model, m.head_dim, m.head_dim // 2
    P = len(tokens)
    wk = bf16_bits_to_f32(W["layers"][0]["w_qkv"])[m.n_heads * hd:(m.n_heads + m.n_kv_heads) * hd].astype(np.float64)
    act = np.sqrt(d) * gain.astype(np.float64)       # the normalised one-hot entry, exact in bf16
    i = np.asarray(tokens) % d
    v = (wk[:, i] * act[i]).T.reshape(P, m.n_kv_heads, hd)   # exact in fp32
    assert np.array_equal(v, v.astype(np.float32))
    ang = np.arange(P)[:, None] * m.rope_theta ** (-2.0 * np.arange(half) / hd)
    c = np.cos(ang).astype(np.float32).astype(np.float64)[:, None]
    s = np.sin(ang).astype(np.float32).astype(np.float64)[:, None]
    v1, v2 = v[..., :half], v[..., half:]
    s1, s2 = (v2 * s).astype(np.float32).astype(np.float64), (v1 * s).astype(np.float32).astype(np.float64)
    k = np.concatenate([v1 * c - s1, v2 * c + s2], -1).astype(np.float16)
    return k.transpose(1, 0, 2)


@pytest.mark.parametrize("d,hq,hkv,hd,B,P,G,tiles", [
    (1024, 3, 1, 64, 1, 4000, 64, "4064 rows staged 256x64, 8 slices"),
    (256, 4, 2, 64, 1, 3000, 64, "3064 rows 64x128, 4 slices"),
    (256, 4, 2, 64, 1, 4700, 64, "4764 rows 128x128, 4 folded slices"),
    (256, 8, 8, 128, 8, 100, 256, "2848 rows 64x192"),
    (256, 32, 32, 128, 8, 300, 256, "4448 rows 64x192"),
    (1024, 32, 32, 128, 16, 256, 256, "8192 rows wide 256x256"),
    (1024, 28, 4, 128, 16, 256, 256, "8192 rows wide 256x192"),   # tiles that straddle the key and value heads
    (1024, 42, 3, 64, 16, 256, 256, "8192 rows wide 256x192"),
    (1024, 36, 4, 64, 16, 256, 256, "8192 rows 128x256"),
    (1024, 10, 5, 128, 3, 1390, 72, "3072 rows wide 128x256, 8 folded slices; 1314 rows 64x128, 8 slices"),
])
def test_stored_keys_are_rounded_once(d, hq, hkv, hd, B, P, G, tiles):
    say(f"rope d={d} heads={hq}/{hkv}x{hd} B={B} P={P} G={G}")
    m = ModelShape(n_layers=1, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=128, vocab=1024, dtype="bf16",
                   init_std=0.05)
    a = archer()
    assert a.projection_tiles(m, (B, P, B * P, G), a.K_GEMM_QKV, B * (P + G)) == tiles
    W = model_weights(m, seed=21)
    emb = np.zeros((m.vocab, d), np.float32)
    emb[np.arange(m.vocab), np.arange(m.vocab) % d] = 2.0**20    # its square swamps the norm's epsilon
    W["tok_emb"] = f32_to_bf16_bits(emb)
    rng = np.random.default_rng(22)
    gain = bf16_bits_to_f32(f32_to_bf16_bits((1.0 + 0.2 * rng.standard_normal(d)).astype(np.float32)))
    W["layers"][0]["attn_norm"] = gain
    ctx = make_ctx(m, W, B, P, B * P, G)
    prompt = rng.integers(0, m.mask_id, B * P).astype(np.int32)
    ctx.refresh_prompt(dev_i32(prompt), [P] * B, dev_i32(np.full((B, G), m.mask_id)))
    for b in (0, B - 1):
        k = ctx.read_prompt_kv(0, b, P)[0].cpu().numpy()
        want = _expected_k(W, m, prompt[b * P:(b + 1) * P], gain)
        bad = int((k != want).sum())
        assert bad == 0, f"sequence {b}: {bad} of {k.size} keys differ"
