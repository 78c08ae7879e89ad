"""The 256 x 256 ping-pong GEMM at the lengths its two-stage schedule can get
wrong: one K tile, two, odd and even counts, base tiles followed by one to
three LoRA tiles (both parities), ragged rows, and split K; bit-identical over
repeated launches (a race would show as a difference) and within the float64
bound of the other GEMM tests."""
import numpy as np
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,K,K2", [(4100, 4096, 64, 0), (4096, 4096, 128, 0), (4096, 4096, 192, 0),
                                      (4000, 6144, 64, 64), (4000, 6144, 128, 64), (4000, 6144, 128, 128),
                                      (4000, 6144, 320, 192), (2000, 5120, 5120, 0), (1024, 4096, 8192, 0)])
def test_pingpong_gemm(kind, M, N, K, K2):
    import torch

    log("ping-pong gemm", kind, M, N, K, K2)
    from paper_2503_17707_amd import binding as pb

    dt = torch.float16 if kind == "f16" else torch.bfloat16
    code = {"bf16": 0, "f16": 1}[kind]
    g = torch.Generator(device="cuda").manual_seed(M + N + K + K2)

    def draw(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)

    X, W, b = draw(M, K), draw(N, K, std=0.02), draw(N, std=0.02)
    ref = X.double() @ W.double().t() + b.double()
    ws = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    R0 = torch.randn((M, N), generator=g, device="cuda")
    ref += R0.double()
    if K2:
        group = N // 3
        Z, W2 = draw(M, 3 * K2), draw(N, K2, std=0.02)
        for q in (0, 2):
            ref[:, q * group:(q + 1) * group] += (Z[:, q * K2:(q + 1) * K2].double()
                                                  @ W2[q * group:(q + 1) * group].double().t())
    outs = []
    for _ in range(4):
        R = R0.clone()
        if K2:
            pb.op_gemm_lora(code, 2, X, W, b, Z, K2, W2, group, 0b101, R=R, workspace=ws)
        else:
            pb.op_gemm(code, 2, X, W, b, R=R, workspace=ws)
        outs.append(R)
    torch.cuda.synchronize()
    for R in outs[1:]:
        assert torch.equal(R, outs[0])
    err = (outs[0].double() - ref).abs().max().item()
    tol = 1e-5 * ref.abs().max().item() + 2e-5 * np.sqrt(K + K2)
    assert err <= tol, "max err %.3e > %.3e" % (err, tol)
