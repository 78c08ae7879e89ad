"""Adapter switches between adapters of different targets: the targets that
only the previous adapter changed go back to the unmerged weights, also when
the previous adapter's slot has been attached anew since its merge."""
import numpy as np
import pytest

import synth
from gpu_common import log

pytestmark = pytest.mark.gpu


def _bits(x):
    return np.asarray(x).view(np.uint32)


@pytest.mark.parametrize("d,kind", [(128, "bf16"), (2176, "f16")])  # one ragged column block; two
def test_switch_between_targets(d, kind):
    from paper_2503_17707_amd import binding as pb

    log("merge switch", d, kind)
    base = synth.Workload(name="mswitch", seed=36, n_layers=2, d_model=d, n_heads=d // 64, d_ffn=128, vocab=300,
                          max_pos=9, dtype=kind, batch=1, seq_len=9, lora_rank=5, lora_alpha=10.0, n_adapters=2)
    sets = {"qv": ("q", "v"), "ko": ("k", "o"), "q": ("q",)}
    hw, m = pb.setup(base.with_(lora_targets=("q", "v")), merge_shadow=True)
    hws = {n: pb.HostWeights(base.with_(lora_targets=t), m.cfg) for n, t in sets.items()}

    def attach(slot, name):
        h = hws[name]
        m.attach_lora(slot, h.loras.get(slot) or h.add_lora(slot), base.lora_rank, base.lora_alpha, h.lora_mask())

    def logits():
        return m.prefill(synth.tokens(base), [-1])[1]

    try:
        fresh = {}
        for slot, name in ((0, "qv"), (1, "ko"), (0, "q")):  # each onto freshly streamed weights
            attach(slot, name)
            m.stream_layers(hw)
            m.merge_lora(slot)
            fresh[name] = logits()
        m.stream_layers(hw)
        plain = logits()
        attach(0, "qv")
        m.merge_lora(0)
        attach(0, "q")  # slot 0 no longer says which targets were merged
        m.merge_lora(1)
        assert np.array_equal(_bits(logits()), _bits(fresh["ko"]))
        m.merge_lora(0)
        assert np.array_equal(_bits(logits()), _bits(fresh["q"]))
        m.unmerge_lora()
        assert np.array_equal(_bits(logits()), _bits(plain))
        assert not np.array_equal(_bits(fresh["ko"]), _bits(plain))
    finally:
        m.destroy()
        for h in [hw] + list(hws.values()):
            h.free()
