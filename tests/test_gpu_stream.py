"""The wide-row streaming GEMM (3 to 64 token rows) against float64 products:
both row tiles at their edges, one block and many, K of one stage, of a ragged
last ring round and long enough to be split, both stage widths, with LoRA
columns (one 64-wide step pair and several) on some of the output groups."""
import numpy as np
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu

ULP = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("M", [3, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("N,K,K2", [(192, 128, 0), (192, 128, 64), (768, 640, 192), (768, 4096, 64),
                                    # unsplit: 512-byte rows, and 32-feature blocks
                                    (12288, 1280, 0), (6144, 1024, 64)])
@pytest.mark.parametrize("epi", [0, 2])
def test_stream_gemm(kind, M, N, K, K2, epi):
    import torch

    log("stream gemm", kind, M, N, K, K2, epi)
    from paper_2503_17707_amd import binding as pb

    dt = torch.float16 if kind == "f16" else torch.bfloat16
    code = {"bf16": 0, "f16": 1}[kind]
    g = torch.Generator(device="cuda").manual_seed(M * 7919 + N + K + K2)

    def draw(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)

    X, W, b = draw(M, K), draw(N, K, std=0.02), draw(N, std=0.02)
    ref = X.double() @ W.double().t() + b.double()
    terms = K + K2
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    lora = K2 > 0 and (N // 3) % 256 == 0
    if lora:
        group = N // 3
        Z, W2 = draw(M, 3 * K2), draw(N, K2, std=0.02)
        for q in (0, 2):  # the middle group takes no LoRA columns
            ref[:, q * group:(q + 1) * group] += (Z[:, q * K2:(q + 1) * K2].double()
                                                  @ W2[q * group:(q + 1) * group].double().t())
    # fp32 accumulation of `terms` products of magnitude ~0.02: error below
    # terms * 2^-24 of their sum of magnitudes (a bound far above what is seen)
    acc = terms * 2.0 ** -24 * 0.02 * 4 * np.sqrt(terms)
    if epi == 2:
        R0 = torch.randn((M, N), generator=g, device="cuda")
        out = R0.clone()
        kw = dict(R=out)
        ref = ref + R0.double()
        tol = acc + 2.0 ** -22 * ref.abs()
    else:
        out = torch.empty((M, N), dtype=dt, device="cuda")
        kw = dict(C=out, qscale=0.125, qcols=N // 3)
        ref[:, :N // 3] *= 0.125
        tol = acc + ULP[kind] * ref.abs()
    if lora:
        pb.op_gemm_lora(code, epi, X, W, b, Z, K2, W2, group, 0b101, workspace=ws, **kw)
    else:
        pb.op_gemm(code, epi, X, W, b, workspace=ws, **kw)
    torch.cuda.synchronize()
    err = (out.double() - ref).abs()
    assert bool((err <= tol).all()), "max err %.3e" % float(err.max())
