"""The tiles a projection takes depend on the rows of its pass; the bits do not.

In a context of one K slice (2048 or more response rows) every sequence's
cached step is computed twice: in the whole batch's pass and alone, in other
tiles.  Short prompts keep attention in one split in both, so the logits must be
the same bits; the last row tile of the batch is ragged.  The tables name the
tiles they are there for, and the library says which ones a launch takes
(archer_op_projection_tiles), so a case that no longer reaches its kernel fails.
Of the tiles of few rows the other GPU tests hold 128 x 128, 64 x 128 and 64 x 192
against the oracle.
"""

import numpy as np
import pytest
import torch

from gpu_util import archer, dev_i32, host, make_ctx, say, with_gains
from oracle import model as om
from synth.gen import model_weights
from synth.workloads import ModelShape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv,hd,F,fp16,B,G", [
    (128, 32, 32, 128, 12288, True, 15, 264),    # QKV 64 x 192 in many rounds; fp16 gate/up 256 x 256; 3960 rows
    (128, 32, 32, 128, 12288, False, 16, 256),   # QKV and two-term gate/up 64 x 192; whole tiles
    (192, 36, 4, 64, 6336, True, 15, 264),       # fp16 gate/up 256 x 192; QKV 256 x 256 of 64-dimension heads
    (64, 32, 16, 64, 6336, False, 10, 416),      # two k steps; O and down in the register-staged kernel; 4160 rows
    (4096, 2, 2, 64, 128, True, 16, 256),        # O and down 256 x 256
    (128, 28, 4, 128, 12288, True, 8, 256),      # Dream-like heads at 2048 rows
])
def test_batch_pass_equals_single_passes(d, hq, hkv, hd, F, fp16, B, G):
    say(f"tiles d={d} heads={hq}/{hkv}x{hd} F={F} fp16={fp16} rows={B * G}")
    m = ModelShape(n_layers=2, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=F, vocab=512, dtype="bf16",
                   gateup_fp16=fp16, init_std=0.05)
    ctx = make_ctx(m, with_gains(model_weights(m, seed=3), 4), B, 8, 8 * B, G)
    rng = np.random.default_rng(5)
    prompt = dev_i32(rng.integers(0, m.mask_id, 8 * B))
    g0 = rng.integers(0, m.mask_id, (B, G)).astype(np.int32)
    z_full = ctx.refresh_prompt(prompt, [8] * B, dev_i32(g0))
    g1 = dev_i32(np.where(rng.random((B, G)) < 0.3, m.mask_id, g0))
    z = ctx.step(g1)
    assert bool(torch.isfinite(z).all()) and bool(torch.isfinite(z_full).all())
    for b in (0, B // 2, B - 1):
        sel = [i == b for i in range(B)]
        alone = ctx.step(g1, seq_sel=sel, logits=torch.full_like(z, 7.0))
        assert bool((alone[b] == z[b]).all()), b
        assert bool((alone[(b + 1) % B] == 7.0).all())
        again = ctx.refresh_prompt(prompt, [8] * B, dev_i32(g0), seq_sel=sel, logits=torch.full_like(z, 7.0))
        assert bool((again[b] == z_full[b]).all()), b


ONE = dict(n_layers=1, d_model=128, n_heads=2, n_kv_heads=2, head_dim=64, d_ff=128, vocab=512, dtype="bf16",
           gateup_fp16=False, init_std=0.05)


@pytest.mark.parametrize("cls,batch,alone,B,G,model", [
    # QKV: tiles of whole heads, staged; tiles that straddle the value heads, stored by element
    ("QKV", "2088 rows wide 256x256", "232 rows 64x128", 9, 232, dict(n_heads=34, n_kv_heads=2, head_dim=128)),
    ("QKV", "3960 rows wide 256x192", "264 rows 64x128", 15, 264, dict(n_heads=42, n_kv_heads=3)),
    ("QKV", "2088 rows wide 256x192", "232 rows 64x128", 9, 232, dict(n_heads=28, n_kv_heads=4, head_dim=128)),
    ("QKV", "2088 rows 128x256", "232 rows 64x128", 9, 232, dict(n_heads=36, n_kv_heads=4)),
    ("QKV", "2088 rows 128x192", "232 rows 64x128", 9, 232, dict(n_heads=30, n_kv_heads=3)),
    ("GATEUP", "2088 rows wide 256x256", "232 rows 64x128", 9, 232, dict(d_ff=3072)),
    ("GATEUP", "3960 rows wide 256x192", "264 rows 64x128", 15, 264, dict(d_model=1024, d_ff=3072, init_std=0.02)),
    ("GATEUP", "3960 rows 128x256", "264 rows 64x128", 15, 264, dict(d_model=2048, d_ff=3072, init_std=0.02)),
    ("GATEUP", "2088 rows wide 256x256", "232 rows 128x128", 9, 232, dict(d_ff=2048, gateup_fp16=True)),
    ("GATEUP", "3960 rows wide 256x192", "264 rows 128x128", 15, 264, dict(d_ff=3072, gateup_fp16=True)),
    ("GATEUP", "2088 rows wide 256x256", "232 rows wide 128x192", 9, 232, dict(d_ff=9216, gateup_fp16=True)),
    ("DOWN", "3960 rows wide 256x256", "264 rows 64x128", 15, 264, dict(d_model=4096, init_std=0.02)),
    ("DOWN", "2088 rows 128x256", "232 rows 64x128", 9, 232, dict(d_model=2048, init_std=0.02)),
    ("HEAD", "2088 rows wide 256x256", "232 rows 64x128", 9, 232, dict(vocab=6144)),
    ("HEAD", "2088 rows 128x256", "232 rows 64x128", 9, 232, dict(vocab=2048)),
])
def test_tiles_of_a_batch_give_the_bits_of_single_passes(cls, batch, alone, B, G, model):
    m = ModelShape(**{**ONE, **model})
    a = archer()
    lim, k = (B, 8, 8 * B, G), getattr(a, "K_GEMM_" + cls)
    assert (a.projection_tiles(m, lim, k, B * G), a.projection_tiles(m, lim, k, G)) == (batch, alone)
    say(f"{cls} {batch} against {alone}")
    ctx = make_ctx(m, with_gains(model_weights(m, seed=13), 14), *lim)
    rng = np.random.default_rng(15)
    g0 = rng.integers(0, m.mask_id, (B, G)).astype(np.int32)
    ctx.refresh_prompt(dev_i32(rng.integers(0, m.mask_id, 8 * B)), [8] * B, dev_i32(g0))
    g1 = dev_i32(np.where(rng.random((B, G)) < 0.3, m.mask_id, g0))
    z = ctx.step(g1)
    x = ctx.read_rows(a.READ_RESIDUAL, B).view(B, G, -1)
    assert bool(torch.isfinite(z).all())
    for b in (0, B // 2, B - 1):
        zb = ctx.step(g1, seq_sel=[i == b for i in range(B)], logits=torch.full_like(z, 7.0))[b]
        assert bool((ctx.read_rows(a.READ_RESIDUAL, 1) == x[b]).all()) and bool((zb == z[b]).all()), b


FOLD = "4096 rows wide 128x256, {} folded slices; 290 rows "


@pytest.mark.parametrize("d,hq,hkv,hd,F,fp16,B,P,G,tiles", [
    # the slices of the first 4096 rows folded in wide tiles, a ragged rest
    (4096, 2, 2, 64, 128, True, 3, 1390, 72, dict(O=FOLD.format(2), DOWN=FOLD.format(2))),
    (1024, 8, 4, 128, 2048, True, 3, 1390, 72, dict(QKV=FOLD.format(8), GATEUP=FOLD.format(4))),
    # two-term gate/up; a query / key tile of QKV straddles the value heads
    (1024, 10, 5, 128, 2048, False, 3, 1390, 72, dict(QKV="3072 rows wide 128x256, 8 folded", GATEUP=FOLD.format(4))),
    # more rows than the partial buffer: 128 x 128 tiles that fold
    (4096, 2, 2, 64, 128, True, 4, 1500, 256, dict(O="7024 rows 128x128, 2 folded slices")),
    (1024, 8, 8, 64, 1024, False, 3, 1536, 256, dict(QKV="5376 rows 128x128, 8 folded slices")),
])
def test_split_k_refresh_does_not_depend_on_the_batch(d, hq, hkv, hd, F, fp16, B, P, G, tiles):
    """In a context that splits K, a sequence refreshed in a pass of several whole rounds of CUs and
    refreshed alone gets the same bits: logits, and the deepest layer's keys and values.  (Attention splits its
    keys in both passes: fewer than 192 query tiles of 256 rows.)"""
    say(f"split-K context, batch against alone d={d} heads={hq}/{hkv}x{hd} rows={B * (P + G)}")
    m = ModelShape(n_layers=2, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=F, vocab=256, dtype="bf16",
                   gateup_fp16=fp16, init_std=0.02)
    for cls, want in tiles.items():
        got = [archer().projection_tiles(m, (B, P, B * P, G), getattr(archer(), "K_GEMM_" + cls), n * (P + G)) for n in (B, 1)]
        assert want in got[0] and "folded" not in got[1], (cls, got)
    ctx = make_ctx(m, with_gains(model_weights(m, seed=8), 9), B, P, B * P, G)
    rng = np.random.default_rng(P)
    prompt = dev_i32(rng.integers(0, m.mask_id, B * P))
    g0 = dev_i32(np.where(rng.random((B, G)) < 0.5, m.mask_id, rng.integers(0, m.mask_id, (B, G))))
    z = ctx.refresh_prompt(prompt, [P] * B, g0).clone()
    kv = [ctx.read_prompt_kv(1, b, P) for b in range(B)]
    assert bool(torch.isfinite(z).all())
    for b in range(B):
        alone = ctx.refresh_prompt(prompt, [P] * B, g0, seq_sel=[i == b for i in range(B)], logits=torch.full_like(z, 7.0))
        k, v = ctx.read_prompt_kv(1, b, P)
        assert bool((k == kv[b][0]).all()) and bool((v == kv[b][1]).all()), b
        assert bool((alone[b] == z[b]).all()), b


@pytest.mark.parametrize("P,G", [(4100, 264), (3840, 256), (4090, 8)])
def test_large_pass_of_split_k_context_matches_oracle(P, G):
    """A context that splits K folds the slices of a large refresh's whole rounds in the tile and gives
    the rest's slices workgroups of their own (4364 rows: 4096 and a ragged 268; 4096 rows: no rest;
    4098 rows: a rest of two rows), as in its cached pass."""
    say(f"split-K context P={P} G={G}")
    m = ModelShape(n_layers=2, d_model=4096, n_heads=2, n_kv_heads=2, head_dim=64, d_ff=128, vocab=256, dtype="bf16",
                   init_std=0.02)
    W = with_gains(model_weights(m, seed=8), 9)
    ctx = make_ctx(m, W, 1, P, P, G)
    rng = np.random.default_rng(P)
    p = rng.integers(0, m.mask_id, P)
    g0 = np.full(G, m.mask_id)
    z = host(ctx.refresh_prompt(dev_i32(p), [P], dev_i32(g0[None])))[0]
    z_ref, cache, _ = om.full_forward(W, m, p, g0)
    err = np.max(np.abs(z - z_ref))
    g1 = np.where(rng.random(G) < 0.5, rng.integers(0, m.mask_id, G), g0)
    zc = host(ctx.step(dev_i32(g1[None])))[0]
    zc_ref, _ = om.cached_forward(W, m, g1, cache, P)
    errc = np.max(np.abs(zc - zc_ref))
    say(f"  max abs err full {err:.2e} cached {errc:.2e}")
    # logits of order 1; two-term operands and fp16 q, k, v (the two-layer full-width models stay below 4e-3)
    assert err < 8e-3 and errc < 8e-3


@pytest.mark.parametrize("G,B,d,hq,hkv,F,layers", [
    (64, 32, 128, 32, 32, 12288, 2),
    (72, 29, 128, 32, 32, 12288, 2),
    (120, 18, 128, 32, 32, 12288, 2),
    (256, 8, 4096, 64, 4, 128, 1),     # QKV 64 x 192, with a tile that straddles the value heads
])
def test_few_row_pass_equals_batch_pass(G, B, d, hq, hkv, F, layers):
    """Tiles of one sequence alone (64 x 128, at 256 rows 64 x 192 for QKV) give the bits of the batch's (64 x 192, and
    128 x 192 and 128 x 256 at 4096 columns); 72 and 120 rows leave a ragged last tile."""
    say(f"few rows G={G} B={B} d={d}")
    m = ModelShape(n_layers=layers, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=128, d_ff=F, vocab=512,
                   dtype="bf16", gateup_fp16=False, init_std=0.05 if d < 1024 else 0.02)
    ctx = make_ctx(m, with_gains(model_weights(m, seed=3), 4), B, 8, 8 * B, G)
    rng = np.random.default_rng(G)
    g0 = rng.integers(0, m.mask_id, (B, G)).astype(np.int32)
    ctx.refresh_prompt(dev_i32(rng.integers(0, m.mask_id, 8 * B)), [8] * B, dev_i32(g0))
    g1 = dev_i32(np.where(rng.random((B, G)) < 0.3, m.mask_id, g0))
    z = ctx.step(g1)
    assert bool(torch.isfinite(z).all())
    for b in (0, B - 1):
        alone = ctx.step(g1, seq_sel=[i == b for i in range(B)], logits=torch.full_like(z, 7.0))
        assert bool((alone[b] == z[b]).all()), b


@pytest.mark.parametrize("d,hq,hkv,hd,F,P,G", [
    (4096, 2, 2, 64, 512, 5, 64),      # O and down in slices of 64 x 128 tiles, one row tile
    (4096, 2, 2, 64, 512, 9, 72),      # a ragged second row tile
    (4096, 2, 2, 64, 512, 60, 128),    # two row tiles; the refresh in 128-row ones
    (3584, 28, 4, 128, 128, 7, 128),   # QKV in slices of 64 x 192 tiles
])
def test_few_row_split_k_pass_matches_oracle(d, hq, hkv, hd, F, P, G):
    say(f"few rows split K d={d} G={G}")
    m = ModelShape(n_layers=2, d_model=d, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=F, vocab=256, dtype="bf16",
                   init_std=0.02)
    W = with_gains(model_weights(m, seed=8), 9)
    ctx = make_ctx(m, W, 1, P, P, G)
    rng = np.random.default_rng(P)
    p = rng.integers(0, m.mask_id, P)
    g0 = np.full(G, m.mask_id)
    z = host(ctx.refresh_prompt(dev_i32(p), [P], dev_i32(g0[None])))[0]
    z_ref, cache, _ = om.full_forward(W, m, p, g0)
    g1 = np.where(rng.random(G) < 0.5, rng.integers(0, m.mask_id, G), g0)
    zc = host(ctx.step(dev_i32(g1[None])))[0]
    zc_ref, _ = om.cached_forward(W, m, g1, cache, P)
    err, errc = np.max(np.abs(z - z_ref)), np.max(np.abs(zc - zc_ref))
    say(f"  max abs err full {err:.2e} cached {errc:.2e}")
    # the bound of the larger passes above, with the same operands
    assert err < 8e-3 and errc < 8e-3


@pytest.mark.parametrize("V,B,G", [(4096, 16, 256), (4160, 11, 200), (8192, 17, 248)])
def test_head_tiles_equal_single_passes(V, B, G):
    """Logits of a batch's LM head (4096 columns 256 x 256 tiles; 4160 the register-staged kernel; 8192 columns
    128 x 256; the latter two with ragged last row tiles) against each sequence alone."""
    say(f"head V={V} rows={B * G}")
    m = ModelShape(n_layers=1, d_model=4096, n_heads=2, n_kv_heads=2, head_dim=64, d_ff=128, vocab=V, dtype="bf16",
                   init_std=0.02)
    ctx = make_ctx(m, with_gains(model_weights(m, seed=11), 12), B, 8, 8 * B, G)
    rng = np.random.default_rng(V)
    prompt = dev_i32(rng.integers(0, m.mask_id, 8 * B))
    g0 = dev_i32(np.where(rng.random((B, G)) < 0.5, m.mask_id, rng.integers(0, m.mask_id, (B, G))))
    z = ctx.refresh_prompt(prompt, [8] * B, g0).clone()
    assert bool(torch.isfinite(z).all())
    for b in (0, B - 1):
        alone = ctx.step(g0, seq_sel=[i == b for i in range(B)], logits=torch.full_like(z, 7.0))
        full = ctx.refresh_prompt(prompt, [8] * B, g0, seq_sel=[i == b for i in range(B)], logits=torch.full_like(z, 7.0))
        assert bool((full[b] == z[b]).all()), b
        assert float((alone[b] - z[b]).abs().max()) < 8e-3, b   # keys from the cache: attention sums in another order
        assert bool((alone[(b + 1) % B] == 7.0).all())
