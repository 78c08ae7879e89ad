"""Attention's choices by prompt length: prompts of up to 32, 64 and 128 tokens
and one past each, with few and many (sequence, head) pairs, both head sizes,
against float64."""
import pytest

from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,hd", [("f16", 64), ("bf16", 64), ("f16", 128)])
@pytest.mark.parametrize("B,T,H", [(40, 1, 16), (40, 31, 16), (3, 32, 2), (40, 33, 16), (40, 64, 16), (40, 65, 16),
                                   (3, 128, 2), (40, 128, 16), (20, 129, 32), (1, 1024, 32)])
def test_attention_by_length(kind, hd, B, T, H):
    import torch

    log("attention", kind, hd, B, T, H)
    from paper_2503_17707_amd import binding as pb

    dt = torch.float16 if kind == "f16" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + T)
    d = H * hd
    qkv = torch.randn((B * T, 3 * d), generator=g, device="cuda")
    qkv[:, :d] *= hd ** -0.5
    qkv = qkv.to(dt)
    out = torch.full((B * T, d), float("nan"), dtype=dt, device="cuda")
    pb.op_attention(1 if kind == "f16" else 0, qkv, out, B, T, H, hd)
    q, k, v = (qkv[:, i * d:(i + 1) * d].double().reshape(B, T, H, hd).transpose(1, 2).contiguous() for i in range(3))
    s = torch.matmul(q, k.transpose(2, 3).contiguous())
    s.masked_fill_(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    ref = torch.matmul(torch.softmax(s, -1), v).transpose(1, 2).reshape(B * T, d)
    # probabilities enter the products rounded to the storage type
    ulp = 2.0 ** -8 if kind == "bf16" else 2.0 ** -11
    err = (out.double() - ref).abs().max().item()
    assert err <= 4 * ulp * ref.abs().max().item() + 1e-3, "max err %.3e" % err
