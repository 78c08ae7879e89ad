"""Every block shape between the GEMV and the large tiles sums K in the ranges of
its plan and in their order: results bit for bit those of the 128 x 128 ring
kernel run over each range by itself (2049 rows of 128 features: no other shape
applies), the ranges' sums added in order and the epilogue's two additions made
by torch in fp32."""
import pytest

from gpu_common import log
from wide_cases import CASES, WORKSPACE

pytestmark = pytest.mark.gpu

ROWS = 2049  # above the rows that any other block shape serves


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,K,K2,plan", CASES)
def test_sums_in_the_planned_ranges(kind, M, N, K, K2, plan):
    import torch

    from paper_2503_17707_amd import binding as pb

    log("wide shape", kind, M, N, K, K2, plan)
    dt = torch.float16 if kind == "f16" else torch.bfloat16
    code = {"bf16": 0, "f16": 1}[kind]
    g = torch.Generator(device="cuda").manual_seed(M + N + K + K2)

    def draw(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)

    X, W, b = draw(M, K), draw(N, K, std=0.02), draw(N, std=0.02)
    R0 = torch.randn((M, N), generator=g, device="cuda")
    ws = torch.empty(WORKSPACE, dtype=torch.uint8, device="cuda")
    out = R0.clone()
    group = N // 3
    if K2:
        Z, W2 = draw(M, 3 * K2), draw(N, K2, std=0.02)  # the middle group takes no LoRA columns
        pb.op_gemm_lora(code, 2, X, W, b, Z, K2, W2, group, 0b101, R=out, workspace=ws)
    else:
        pb.op_gemm(code, 2, X, W, b, R=out, workspace=ws)

    step = int(plan.split()[5]) * 64
    starts = list(range(0, K, step))
    rows = torch.arange(ROWS, device="cuda") % M
    zero = torch.zeros(128, dtype=dt, device="cuda")
    Xr = [X[rows, k:k + step].contiguous() for k in starts]
    Zr = [Z[rows, q * K2:(q + 1) * K2].contiguous() for q in range(3)] if K2 else None
    total = torch.empty((M, N), dtype=torch.float32, device="cuda")
    part = torch.empty((ROWS, 128), dtype=torch.float32, device="cuda")
    for n in range(0, N, 128):
        for i, k in enumerate(starts):
            part.zero_()
            Wn = W[n:n + 128, k:k + step].contiguous()
            q = n // group if K2 else 1
            if i == len(starts) - 1 and q != 1:
                pb.op_gemm_lora(code, 2, Xr[i], Wn, zero, Zr[q], 0, W2[n:n + 128].contiguous(), 256, 1, R=part)
            else:
                pb.op_gemm(code, 2, Xr[i], Wn, zero, R=part)
            if i == 0:
                total[:, n:n + 128] = part[:M]
            else:
                total[:, n:n + 128] += part[:M]
    want = R0 + (total + b.float())
    torch.cuda.synchronize()
    bad = (out != want).nonzero()
    assert bad.shape[0] == 0, "%d of %d differ, first at %s" % (bad.shape[0], M * N, bad[0].tolist())
