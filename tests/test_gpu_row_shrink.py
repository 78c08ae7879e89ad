"""The LoRA shrink in blocks of its own (up to 64 rows), behind the first
LayerNorm, behind fc2's split-K reduce and of the attention rows (o), against
the oracle: both sides of the row limit, ranks that leave a partial group of
four, rows without an adapter, and a width whose last chunk is ragged."""
import pytest

import oracle
import synth
from gpu_common import compare, log, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("B,T,d,rank,seed", [(3, 3, 256, 6, 64), (4, 16, 256, 16, 61), (5, 13, 256, 6, 69),
                                             (4, 15, 2304, 5, 62)])
def test_row_shrink_of_few_rows(kind, B, T, d, rank, seed):
    log("row shrink", kind, B, T, d, rank)
    w = synth.Workload(name="rshrink", seed=seed, n_layers=2, d_model=d, n_heads=d // 64, d_ffn=2048, vocab=500,
                       max_pos=T, dtype=kind, batch=B, seq_len=T, lora_targets=("q", "k", "v", "o"), lora_rank=rank,
                       lora_alpha=2.0 * rank, n_adapters=2, adapter_of_seq=tuple((0, -1, 1)[b % 3] for b in range(B)))
    tok, logits = run_gpu(w)
    ref_logits, ref_tok = oracle.prefill_first_token(w)
    compare("row shrink", logits, tok, ref_logits, ref_tok)
