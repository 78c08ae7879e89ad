"""The matrix-unit LM head keeps every bit of the fp32 hidden state.  The first d
rows of the embedding are one-hot, so their logits are the hidden state itself:
a sequence gets the bits in a batch (three terms on the matrix units) that it
gets alone (fp32 dot products), at the edges of its groups of 16 and 32 sequences
and of its 64-row blocks.  The other rows are random: their logits'
error against float64, from that hidden state, is no larger than alone.  The layer's weights
are zeros and a sequence is one token, so the hidden state does not depend on the batch;
final gains and token rows of very different scale spread it."""
import ctypes

import numpy as np
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


class _Host:
    def __init__(self, layers, globals_):
        self.layers, self.globals = layers, globals_


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("d,B,extra", [(128, 16, 1500), (256, 16, 1500), (512, 3, 1503), (512, 16, 1409), (640, 17, 1410),
                                       (768, 33, 1472), (2048, 2, 1500), (2048, 17, 1500), (4096, 3, 1500),
                                       (4096, 33, 1500), (9216, 4, 1500)])
def test_lm_head_batch_keeps_the_hidden_state(kind, d, B, extra):
    import torch

    from paper_2503_17707_amd import binding as pb

    log("lm head precision", kind, d, B, extra)
    dt = torch.float16 if kind == "f16" else torch.bfloat16
    rng = np.random.default_rng(d + B)
    vocab = d + extra
    cfg = pb.Config(n_layers=1, d_model=d, n_heads=d // 64, d_ffn=64, vocab=vocab, max_pos=1, max_tokens=B, max_batch=B,
                    max_adapters=0, max_rank=0, dtype=pb.PB_F16 if kind == "f16" else pb.PB_BF16, ln_eps=1.0,
                    max_new_tokens=0, merge_shadow=0)
    L = pb.lib()
    layer, glob = pb.Pinned(L.pb_layer_bytes(ctypes.byref(cfg))), pb.Pinned(L.pb_globals_bytes(ctypes.byref(cfg)))
    layer.view(np.int16)[:] = 0
    glob.view(np.int16)[:] = 0

    def put(name, x):
        t = torch.from_numpy(np.ascontiguousarray(x)).to(dt)
        off, n = pb.globals_tensor(cfg, name)
        glob.view(np.int16)[off:off + n] = t.view(torch.int16).numpy().reshape(-1)
        return t.double().numpy()

    E = rng.normal(0.0, 0.5, (vocab, d)).astype(np.float32)
    E[:d] = np.eye(d)
    E[d:d + B] *= np.float32(10.0) ** rng.integers(-2, 2, (B, 1))  # the tokens' rows
    E64 = put("embed", E)
    put("lnf_g", 2.0 ** rng.uniform(-6, 0, d))
    put("lnf_b", rng.normal(0.0, 0.01, d))
    m = pb.Model(cfg)
    try:
        m.stream_layers(_Host([layer], glob))
        toks = np.arange(d, d + B, dtype=np.int32)[:, None]
        tok, batch = m.prefill(toks, [-1] * B)
        alone = np.concatenate([m.prefill(toks[b:b + 1], [-1])[1] for b in range(B)])
    finally:
        m.destroy()
        layer.free()
        glob.free()
    z = alone[:, :d]
    # elements this far below the row's largest keep fewer bits in f16 terms
    big = np.abs(z) >= np.abs(z).max(axis=1, keepdims=True) * 2.0 ** -22
    assert big.mean() > 0.99
    assert np.array_equal(batch[:, :d][big], z[big])
    # (not the tokens' own rows: one logit would outweigh the other errors)
    want = z.astype(np.float64) @ E64[d + B:].T
    size = np.linalg.norm(want, axis=1)
    e_batch, e_alone = (np.linalg.norm(x[:, d + B:] - want, axis=1) / size for x in (batch, alone))
    log("  error against float64: batch %.2e .. %.2e, alone %.2e .. %.2e" % (
        e_batch.min(), e_batch.max(), e_alone.min(), e_alone.max()))
    log("  ratio %.3f .. %.3f" % ((e_batch / e_alone).min(), (e_batch / e_alone).max()))
    # norms over 1500 errors scatter by a few per cent
    assert (e_batch <= 1.1 * e_alone).all()
    assert list(tok) == [int(np.argmax(r)) for r in batch]
