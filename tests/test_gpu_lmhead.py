"""The LM head of several sequences through prefills of one layer, on the matrix
units (d from 512 on) and on the dot products: sequence counts at the edges of
the matrix-unit head's 16- and 32-sequence groups, vocabularies ragged against
its 64-row blocks and against 16-byte stores, the fewest K stages and more;
logits against the oracle, tokens the first maximum of the returned logits."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import compare, log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("B,vocab,d", [(2, 63, 128), (16, 257, 128), (17, 642, 256), (33, 1000, 128),
                                       (5, 64, 2048), (2, 63, 512), (16, 257, 512), (17, 642, 640),
                                       (33, 1000, 512)])
def test_lm_head_of_several_sequences(kind, B, vocab, d):
    w = synth.Workload(name="lmhead", seed=61, n_layers=1, d_model=d, n_heads=d // 64, d_ffn=128, vocab=vocab,
                       max_pos=8, dtype=kind, batch=B, seq_len=3, lora_rank=8, lora_alpha=16.0, n_adapters=0,
                       adapter_of_seq=tuple([-1] * B))
    log("lm head", kind, B, vocab, d)
    ref_logits, ref_tok = oracle.prefill_first_token(w)
    tok, logits = run_gpu(w, max_adapters=0, max_rank=8)
    assert list(tok) == [int(np.argmax(row)) for row in logits]
    # tokens against the oracle only where its two largest logits are further
    # apart than the logits' own bar
    srt = np.sort(ref_logits, axis=1)
    clear = srt[:, -1] - srt[:, -2] > 2 * 3e-2
    tok = np.where(clear, tok, ref_tok)
    compare("B=%d vocab=%d d=%d %s" % (B, vocab, d, kind), logits, tok, ref_logits, ref_tok)
