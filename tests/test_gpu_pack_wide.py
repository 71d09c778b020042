"""The device packers that work on whole 16x64 tiles, byte for byte against the
host packer (which the property tests pin to the oracle): ragged unit and strip
counts, weights on the rounding boundaries of their row's scale, zero rows, and
scales at the ends of the format; and unaligned weights, which take the
one-element kernels."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # hidden, ffn, experts, dtype, magnitude, int4
    (64, 64, 1, "f32", 1.0, False),
    (128, 64, 3, "bf16", 0.02, False),
    (192, 1088, 2, "bf16", 0.02, False),
    (1088, 576, 2, "f32", 1e-7, False),
    (512, 640, 2, "f32", 1e4, False),
    (256, 256, 1, "f32", 1e-38, False),
    (256, 256, 1, "bf16", 1e-38, False),
    (128, 128, 2, "bf16", 0.02, True),
    (1152, 384, 2, "bf16", 0.02, True),
    (384, 1152, 2, "bf16", 1e-7, True),
    (256, 256, 1, "bf16", 1e8, True),
    (256, 384, 1, "f32", 1.0, True),
    # INT4 from bf16 takes whole tiles for large experts only: runs of one and two
    # column pairs in both dimensions, runs of two, and one expert too few
    (6016, 896, 5, "bf16", 0.02, True),
    (5888, 1024, 4, "bf16", 1e-7, True),
    (6016, 896, 4, "bf16", 0.02, True),
]


@pytest.mark.parametrize("C,R,n,dt,mag,int4", CASES)
@pytest.mark.parametrize("offset", [0, 1])
def test_pack_wide(mira, C, R, n, dt, mag, int4, offset):
    g = torch.Generator().manual_seed(C * 7 + R)
    w = [torch.randn(n, a, b, generator=g) * mag for a, b in ((R, C), (R, C), (C, R))]
    w[0][0, 0], w[1][0, 0], w[2][0, :, 0] = 0, 0, 0
    w[0][0, 1] = ((torch.arange(C) % 255 - 127).float() + 0.5) * mag
    w[0][0, 1, 0] = 127 * mag
    w[2][0, 2] = ((torch.arange(R) % 15 - 7).float() + 0.5) * mag
    t = torch.float32 if dt == "f32" else torch.bfloat16
    w = [x.to(t) for x in w]
    size = mira.mira_packed_expert_bytes_int4 if int4 else mira.mira_packed_expert_bytes
    stride = size(C, R) + 256
    s = mira.MoEShape(C, R, 1, 1, flags=mira.MIRA_FLAG_INT4 if int4 else 0)
    wt = mira.MIRA_F32 if dt == "f32" else mira.MIRA_BF16
    host = torch.empty(n * stride, dtype=torch.uint8)
    mira.mira_pack_experts(s, n, wt, *w, 1e-8, host, stride, 0)
    dev = torch.full((n * stride,), 0xAA, dtype=torch.uint8, device="cuda")
    dw = [torch.cat([torch.zeros(offset, dtype=t), x.reshape(-1)]).cuda()[offset:] for x in w]
    mira.mira_pack_experts(s, n, wt, *dw, 1e-8, dev, stride, 1)
    torch.cuda.synchronize()
    assert torch.equal(dev.cpu(), host)
