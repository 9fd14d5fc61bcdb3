"""The bf16 dense baseline's workgroup shapes (256, 128 and 64 queries; the last two split the keys
between two waves; 64 features take the last two only, two workgroups to a compute unit), each at ragged query and key counts, under the chunk-causal mask with hidden
keys, with a query range whose key counts differ, and with rows that are not packed; against plain
torch in float64.  Bar: the probabilities and the output are rounded once each to 2^-9, which shows as
2.4e-3 (2-norm); four times that."""
import math

import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

CASES = {
    # name: (heads, d, f_q, f_kv, h, w, chunk, offset)
    "64-ragged": (1, 128, 1, 1, 7, 13, 0, 0),
    "64-one-key": (2, 64, 1, 1, 1, 1, 0, 0),
    "64-33-keys": (1, 128, 1, 1, 3, 11, 0, 0),
    "64-65-keys": (1, 64, 1, 1, 5, 13, 0, 0),
    "64-hidden": (1, 128, 2, 8, 9, 11, 2, 2),
    "64-steps": (2, 128, 6, 6, 7, 19, 2, 0),
    "128": (5, 128, 3, 3, 30, 52, 0, 0),
    "128-steps": (5, 64, 6, 6, 19, 41, 2, 0),
    "256": (7, 128, 3, 3, 30, 52, 0, 0),
    "256-hidden": (12, 128, 3, 5, 29, 53, 1, 1),
    "256-steps": (9, 128, 9, 9, 13, 41, 3, 0),
    "d64-second-round": (14, 64, 3, 3, 30, 52, 0, 0),
    "d64-steps": (9, 64, 9, 9, 13, 41, 3, 0),
    "d64-64-many": (20, 64, 1, 1, 30, 52, 0, 0),
}


def reference(q, k, v, hw, chunk, offset, scale):
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for h in range(q.shape[1]):
        s = scale * q[0, h].double() @ k[0, h].double().t().contiguous()
        if chunk:
            qc = (torch.arange(s.shape[0], device=q.device) // hw + offset) // chunk
            kc = (torch.arange(s.shape[1], device=q.device) // hw) // chunk
            s = s.masked_fill(kc[None, :] > qc[:, None], float("-inf"))
        out[0, h] = torch.softmax(s, -1) @ v[0, h].double()
    return out


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_dense(name, packed):
    heads, d, f_q, f_kv, h, w, chunk, offset = CASES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(len(name))

    def draw(n):
        x = torch.randn(1, heads, n, d, generator=gen, device="cuda:0").bfloat16()
        return x if packed else x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)   # tokens before heads

    q, k, v = draw(f_q * h * w), draw(f_kv * h * w), draw(f_kv * h * w)
    print(f"case {name} packed {packed}", flush=True)
    scale = 2.0 * d ** -0.5
    out = pkg.dense_attn_fwd(q, k, v, f_q=f_q, f_kv=f_kv, h=h, w=w, causal_chunk=chunk, q_frame_offset=offset,
                             scale=scale)
    ref = reference(q, k, v, h * w, chunk, offset, scale)
    err = ((out.double() - ref).norm() / ref.norm()).item()
    print(f"  rel {err:.2e}", flush=True)
    assert err <= 1e-2


def test_rising_logits_raise_the_reference():
    # keys in rising order of their logit: every step raises the softmax reference
    n, d = 60 * 11, 128
    q = torch.zeros(1, 1, n, d, device="cuda:0")
    q[..., 0] = 1.0
    k = torch.randn(1, 1, n, d, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(1))
    k[..., 0] = torch.arange(n, device="cuda:0") * 0.5
    v = torch.randn(1, 1, n, d, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(2))
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    out = pkg.dense_attn_fwd(q, k, v, f_q=1, f_kv=1, h=60, w=11, scale=1.0)
    ref = reference(q, k, v, n, 0, 0, 1.0)
    assert ((out.double() - ref).norm() / ref.norm()).item() <= 1e-2


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [1, 5, 12])
def test_sum_of_the_unrounded_probabilities(heads, d):
    # Two keys of probability 1 (one in either half of the first 64 keys) hold the values; every other key
    # has p = 0.50176, which bf16 rounds to 0.5.  The second product weighs the others' zeros with that, but
    # the denominator is a sum of fp32 numbers: a sum of the rounded ones would be 3.5e-3 short.  The
    # output's own rounding (1.1e-3 rms) averages out over the features to 1e-4.
    h, w, p = 90, 52, 0.5 * (1 + 0.9 * 2.0 ** -8)
    n = h * w
    q = torch.zeros(1, heads, n, d, device="cuda:0")
    q[..., 0] = 1.0
    k = torch.zeros_like(q)
    k[..., 0] = -1.0
    k[:, :, [0, 32]] = 0.0
    v = torch.zeros_like(q)
    value = 1.0 + torch.rand(1, heads, 1, d, generator=torch.Generator(device="cuda:0").manual_seed(heads), device="cuda:0")
    v[:, :, [0, 32]] = value
    out = pkg.dense_attn_fwd(q.bfloat16(), k.bfloat16(), v.bfloat16(), f_q=1, f_kv=1, h=h, w=w, scale=-math.log(p))
    exact = 2 * v.bfloat16()[:, :, :1].double() / (2 + (n - 2) * p)
    bias = (out.double() / exact - 1).mean().item()
    print(f"  mean relative error {bias:.1e}", flush=True)
    assert abs(bias) <= 8e-4
