"""Stage L backward of resident key ranges at t < T: one launch, or two for 513 to 640 workgroups (of a compute unit's
two and a half) of five and six key tiles at 128 features.  A head's gradients are the same bits either way, and for any
number of heads in a call: 90 rows and 15 columns, 40 heads (600 workgroups, two launches), 2 and 48 (one)."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def one_head_group():
    pkg.binding.set_head_groups(1)
    yield
    pkg.binding.set_head_groups(0)


@pytest.mark.parametrize("rows,d,iters", [(90, 128, 2), (65, 128, 3), (80, 64, 2)])
@pytest.mark.parametrize("saved", [False, True])
def test_for_any_number_of_heads(rows, d, iters, saved):
    cols, heads = 15, 40
    gen = torch.Generator(device="cuda:0").manual_seed(rows)
    tensors = [torch.randn(1, heads, rows * cols, d, generator=gen, device="cuda:0").bfloat16() for _ in range(4)]
    kw = dict(f_q=1, f_kv=1, h=rows, w=cols, b1=rows, b2=cols, tile=0, iters=iters, scale=d ** -0.5)

    def grads(q, k, v, do):
        if not saved:
            return pkg.monarch_attn_bwd(q, k, v, do, **kw)
        _, workspace = pkg.monarch_attn_fwd_save(q, k, v, **kw)
        return pkg.monarch_attn_bwd_saved(q, k, v, do, workspace, **kw)
    whole = grads(*tensors)
    few = grads(*(x[:, :2].contiguous() for x in tensors))
    more = grads(*(torch.cat((x, x[:, :8]), 1) for x in tensors))
    for name, w, f, m in zip(("dQ", "dK", "dV"), whole, few, more):
        assert torch.equal(f, w[:, :2]), name
        assert torch.equal(m[:, :heads], w) and torch.equal(m[:, heads:], w[:, :8]), name
