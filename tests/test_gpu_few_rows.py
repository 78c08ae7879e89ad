"""Products of 3 to 8 rows, which the matrix units serve beside the GEMV: the
error of their fp32 sums against float64 is no larger than that of the same rows
one at a time (the GEMV's dot products), with and without a workspace, over K
from 128 to 20480, split and unsplit; a zero B leaves the base's bits."""
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("N,K", [(8192, 128), (2304, 768), (8192, 2048), (2048, 8192), (4096, 4096), (15360, 5120),
                                 (5120, 20480)])
def test_rounding_error_of_few_rows(kind, N, K):
    import torch

    from paper_2503_17707_amd import binding as pb

    log("few rows", kind, N, K)
    dt = torch.float16 if kind == "f16" else torch.bfloat16
    code = {"bf16": 0, "f16": 1}[kind]
    g = torch.Generator(device="cuda").manual_seed(N + K)
    X = torch.randn((8, K), generator=g, device="cuda").to(dt)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(dt)
    b = torch.zeros(N, dtype=dt, device="cuda")
    ref = X.double() @ W.double().t()
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")

    def error(M, workspace):
        worst = 0.0
        for m0 in range(0, 8 - M + 1, M):
            R = torch.zeros((M, N), dtype=torch.float32, device="cuda")
            pb.op_gemm(code, 2, X[m0:m0 + M], W, b, R=R, workspace=workspace)
            want = ref[m0:m0 + M]
            worst = max(worst, float((R.double() - want).norm() / want.norm()))
        return worst

    alone = error(1, ws)
    for M in (3, 4, 5, 8):
        for workspace in (ws, None):
            e = error(M, workspace)
            log("  %d rows%s: %.3e, alone %.3e" % (M, "" if workspace is not None else ", no workspace", e, alone))
            # alone is the worst of eight rows, a batch the worst of its groups: the
            # norms over N >= 2048 errors scatter by a few per cent
            assert e <= 1.05 * alone


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,K,K2", [(3, 12288, 2048, 64), (8, 6144, 1024, 192), (5, 3072, 8192, 128),
                                      (8, 768, 128, 64)])
def test_lora_columns_of_few_rows(kind, M, N, K, K2):
    import torch

    from paper_2503_17707_amd import binding as pb

    log("few rows with LoRA", kind, M, N, K, K2)
    dt = torch.float16 if kind == "f16" else torch.bfloat16
    code = {"bf16": 0, "f16": 1}[kind]
    g = torch.Generator(device="cuda").manual_seed(M + N + K + K2)

    def draw(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)

    X, W, b = draw(M, K), draw(N, K, std=0.02), draw(N, std=0.02)
    Z, W2 = draw(M, 3 * K2), draw(N, K2, std=0.02)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    group = N // 3
    ref = X.double() @ W.double().t() + b.double()
    for q in (0, 2):  # the middle group takes no LoRA columns
        ref[:, q * group:(q + 1) * group] += (Z[:, q * K2:(q + 1) * K2].double()
                                              @ W2[q * group:(q + 1) * group].double().t())
    for workspace in (ws, None):
        base, zero, out = (torch.zeros((M, N), dtype=torch.float32, device="cuda") for _ in range(3))
        pb.op_gemm(code, 2, X, W, b, R=base, workspace=workspace)
        pb.op_gemm_lora(code, 2, X, W, b, Z, K2, torch.zeros_like(W2), group, 0b101, R=zero, workspace=workspace)
        pb.op_gemm_lora(code, 2, X, W, b, Z, K2, W2, group, 0b101, R=out, workspace=workspace)
        assert torch.equal(base, zero)
        # sums of K2 more products and of bias and residual: a few roundings of 2^-24 above
        # the error of the base alone
        assert float((out.double() - ref).norm() / ref.norm()) < 2.5e-7
