"""Tables and destinations that are not aligned for vector loads and stores take the element path: the same bits."""

import numpy as np
import pytest
import torch

from gpu_util import archer, dev_i32, say
from synth.gen import model_weights
from synth.workloads import ModelShape

pytestmark = pytest.mark.gpu


def _shifted(t, elems):
    """The same contiguous tensor, `elems` elements into a buffer of its own."""
    buf = torch.empty(t.numel() + elems, dtype=t.dtype, device=t.device)
    v = buf[elems:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("dtype,hq,hkv,hd,P,G", [
    ("bf16", 4, 2, 64, [63, 65], 8),     # a tile short of one key, a tile and one key
    ("bf16", 2, 2, 128, [1, 130], 16),
    ("fp32", 4, 2, 64, [64, 7], 24),
    ("fp32", 2, 2, 128, [70, 1], 8),
])
def test_unaligned_table_and_cache_copies(dtype, hq, hkv, hd, P, G):
    say(f"alignment {dtype} heads={hq}/{hkv}x{hd} P={P} G={G}")
    a = archer()
    m = ModelShape(n_layers=2, d_model=192, n_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ff=256, vocab=256, dtype=dtype,
                   init_std=0.05)
    W = a.upload_weights(model_weights(m, seed=5), m.dtype)
    rng = np.random.default_rng(7)
    prompt = dev_i32(rng.integers(0, m.mask_id, sum(P)))
    g = dev_i32(rng.integers(0, m.mask_id, (2, G)))
    got = []
    for shift in (0, 1):
        Ws = dict(W, tok_emb=_shifted(W["tok_emb"], shift))
        ctx = a.Context(m, Ws, 2, max(P), sum(P), G)
        out = [ctx.refresh_prompt(prompt, P, g).clone(), ctx.step(g, seq_sel=[False, True]).clone()[1]]
        for layer in range(2):
            for b, p in enumerate(P):
                for what, t in zip((a.READ_PROMPT_K, a.READ_PROMPT_V), ctx.read_prompt_kv(layer, b, p)):
                    out.append(t)
                    u = _shifted(torch.zeros_like(t), 1)
                    a._check(a.lib.archer_read_state(ctx.h, what, layer, b, u.data_ptr(), u.numel() * u.element_size()))
                    assert torch.equal(u, t), (layer, b, what)
        got.append(out)
    torch.cuda.synchronize()
    for x, y in zip(*got):
        assert torch.equal(x, y)
    # the copies are the cache itself: prompt values of the first layer do not depend on the other sequence
    alone = a.Context(m, W, 1, max(P), max(P), G)
    for b in range(2):
        p0 = sum(P[:b])
        alone.refresh_prompt(prompt[p0:p0 + P[b]].contiguous(), [P[b]], g[b:b + 1].contiguous())
        k, v = alone.read_prompt_kv(0, 0, P[b])
        i = 2 + 2 * b
        assert torch.equal(k, got[0][i]) and torch.equal(v, got[0][i + 1])
