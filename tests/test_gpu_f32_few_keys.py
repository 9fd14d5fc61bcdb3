"""fp32 dense baseline on either side of the key counts up to which the operands stay fp32 (16 keys at 64
features, 64 at 128, 160 there under a mask), against softmax and products in 64 bits.  Bar: that of the
other fp32 tests (2-norm, 5e-6)."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu


# f_q, f_kv, h, w, d, causal chunk, frame offset
@pytest.mark.parametrize("size", [(1, 1, 4, 4, 64, 0, 0), (1, 1, 1, 17, 64, 0, 0), (3, 1, 8, 8, 128, 0, 0), (1, 1, 5, 13, 128, 0, 0),
                                  (2, 2, 5, 16, 128, 1, 0), (2, 2, 7, 23, 96, 1, 0), (1, 4, 5, 8, 96, 1, 3), (2, 2, 2, 4, 32, 1, 0),
                                  (2, 2, 3, 3, 64, 1, 0)], ids=str)
def test_against_64_bits(size):
    f_q, f_kv, h, w, d, chunk, off = size
    gen = torch.Generator(device="cuda:0").manual_seed(d + w)
    q, k, v = (torch.randn(2, 3, f * h * w, d, generator=gen, device="cuda:0") for f in (f_q, f_kv, f_kv))
    out = pkg.dense_attn_fwd(q, k, v, f_q=f_q, f_kv=f_kv, h=h, w=w, causal_chunk=chunk, q_frame_offset=off, scale=d ** -0.5)
    s = d ** -0.5 * torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous())
    if chunk > 0:
        at_q = (off + torch.arange(f_q * h * w, device="cuda:0") // (h * w)) // chunk
        at_k = torch.arange(f_kv * h * w, device="cuda:0") // (h * w) // chunk
        s = s.masked_fill(at_k[None] > at_q[:, None], float("-inf"))
    ref = torch.matmul(torch.softmax(s, -1), v.double())
    assert (out.double() - ref).norm() <= 5e-6 * ref.norm()
