"""Blocks of eleven and twelve tiles of rows at 128 features: whether one or two workgroups take a column's
rows depends on how many columns a call has, the results do not."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [161, 176, 177, 192])
def test_same_bits_for_any_number_of_heads(rows):
    w, d, heads = 8, 128, 56                 # 448 columns: whole; 2 or 112 heads: in parts
    gen = torch.Generator(device="cuda:0").manual_seed(rows)
    q, k, v = (torch.randn(1, heads, rows * w, d, generator=gen, device="cuda:0").bfloat16() for _ in range(3))

    def call(*x):
        return pkg.monarch_attn_fwd(*x, f_q=1, f_kv=1, h=rows, w=w, b1=rows, b2=w, tile=0, iters=2, scale=d ** -0.5)
    whole = call(q, k, v)
    assert torch.equal(call(*(x[:, :2].contiguous() for x in (q, k, v))), whole[:, :2])
    twice = call(*(torch.cat((x, x), 1) for x in (q, k, v)))
    assert torch.equal(twice[:, :heads], whole) and torch.equal(twice[:, heads:], whole)
