"""Merged weights bit for bit: W + s B A read back from the device arena against
the same sum on the CPU.  A and B lie on a coarse grid, so that B A is exact in
fp32 whatever the order of its sum, and W + s B A in float64; f16 weights are
then rounded once, bf16 weights to fp32 and from there to bf16.  Merged into
fresh weights (in place) and on a switch (from the shadow)."""
import ctypes

import numpy as np
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


class _Host:
    def __init__(self, layers, globals_):
        self.layers, self.globals = layers, globals_

    def free(self):
        for b in self.layers + [self.globals]:
            b.free()


def _bits(x, kind):
    import torch

    if kind == "f16":
        return x.astype(np.float16).view(np.int16)  # numpy rounds float64 to float16 once
    return torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16).view(torch.int16).numpy()


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("d,rank", [(1024, 5), (2176, 8)])
def test_merged_weights_bit_for_bit(kind, d, rank):
    import torch

    from paper_2503_17707_amd import binding as pb

    log("merge rounding", kind, d, rank)
    rng = np.random.default_rng(d + rank)
    dt = torch.float16 if kind == "f16" else torch.bfloat16
    cfg = pb.Config(n_layers=1, d_model=d, n_heads=d // 64, d_ffn=64, vocab=64, max_pos=2, max_tokens=2, max_batch=1,
                    max_adapters=2, max_rank=8, dtype=pb.PB_F16 if kind == "f16" else pb.PB_BF16, ln_eps=1e-5,
                    max_new_tokens=0, merge_shadow=1)
    L = pb.lib()
    nb = L.pb_layer_bytes(ctypes.byref(cfg))
    ng = L.pb_globals_bytes(ctypes.byref(cfg))
    layer, glob = pb.Pinned(nb), pb.Pinned(ng)
    layer.view(np.int16)[:] = 0
    glob.view(np.int16)[:] = 0
    w64 = {}
    for t in ("q", "k", "v", "o"):
        w = torch.from_numpy(rng.normal(0.0, 0.02, (d, d))).to(dt)
        w64[t] = w.double().numpy()
        off, n = pb.layer_tensor(cfg, "w" + t)
        layer.view(np.int16)[off:off + n] = w.view(torch.int16).numpy().reshape(-1)
    mask = 15
    blobs, prods = [], []
    for a in range(2):
        blob = pb.Pinned(L.pb_lora_layer_bytes(ctypes.byref(cfg), rank, mask))
        prod = {}
        for t in ("q", "k", "v", "o"):
            A, B = (rng.integers(-127, 128, s) / 128.0 for s in ((rank, d), (d, rank)))
            for which, x in (("A", A), ("B", B)):
                off, n = pb.lora_tensor(cfg, rank, mask, t, which)
                blob.view(np.int16)[off:off + n] = torch.from_numpy(x).to(dt).view(torch.int16).numpy().reshape(-1)
            prod[t] = B @ A  # exact: multiples of 2^-14 below 8
        blobs.append(blob)
        prods.append(prod)
    alpha = 0.3731  # a full 24-bit scale
    scale = np.float64(np.float32(alpha) / np.float32(rank))
    m = pb.Model(cfg)
    host = _Host([layer], glob)
    try:
        for a in range(2):
            m.attach_lora(a, [blobs[a]], rank, alpha, mask)
        m.stream_layers(host)
        start = m.base - m.arena.data_ptr() + ng
        for a in (0, 1):
            m.merge_lora(a)
            torch.cuda.synchronize()
            got = m.arena[start:start + nb].view(torch.int16).cpu().numpy()
            twice = 0
            for t in ("q", "k", "v", "o"):
                off, n = pb.layer_tensor(cfg, "w" + t)
                exact = w64[t] + scale * prods[a][t]
                want = _bits(exact, kind).reshape(-1)
                twice += int((want != _bits(exact.astype(np.float32).astype(np.float64), kind).reshape(-1)).sum())
                bad = np.flatnonzero(got[off:off + n] != want)
                assert bad.size == 0, "%s: %d of %d differ, columns mod 8 %s rows mod 8 %s" % (
                    t, bad.size, n, np.unique(bad % d % 8), np.unique(bad // d % 8))
            log("  adapter %d: %d elements tell one rounding from two" % (a, twice))
            assert kind == "bf16" or twice > 50
    finally:
        m.destroy()
        host.free()
        for b in blobs:
            b.free()
