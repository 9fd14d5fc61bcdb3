"""Values at the ends of their range: what a call returns there is what the plain formula gives."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

INF = float("inf")


def tensors(seed, n_q, n_kv, d, dtype=torch.float32, heads=2):
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    return [torch.randn(1, heads, n, d, generator=gen, device="cuda:0").to(dtype) for n in (n_q, n_kv, n_kv)]


def softmax_rows(q, k, v, scale, hidden=None):
    """softmax(scale q k^T) v in float64, weights of exactly zero ignoring what they weigh."""
    s = scale * torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous())
    if hidden is not None:
        s = s.masked_fill(hidden, -INF)
    p = torch.softmax(s, -1)
    finite = torch.where(v.isfinite(), v, torch.zeros_like(v)).double()
    out = torch.matmul(p, finite)
    inf = torch.matmul((p > 0).double(), v.isinf().double() * v.double().sign().nan_to_num())
    return torch.where(inf != 0, inf * INF, out)


# key counts with 10, 1 and 15 rows in the last chunk of 16
@pytest.mark.parametrize("rows,cols", [(9, 10), (11, 3), (7, 13)])
@pytest.mark.parametrize("d", [64, 128, 38])
def test_fp32_infinite_last_value_row(rows, cols, d):
    q, k, v = tensors(rows, rows * cols, rows * cols, d)
    v[:, :, -1] = INF
    v[:, :, -1, 1] = -INF
    out = pkg.dense_attn_fwd(q, k, v, f_q=1, f_kv=1, h=rows, w=cols, scale=d ** -0.5)
    assert torch.equal(out.double(), softmax_rows(q, k, v, d ** -0.5))
    # blocks (rows, cols): the last value row reaches the last key row of every column's stage L
    out = pkg.monarch_attn_fwd(q, k, v, f_q=1, f_kv=1, h=rows, w=cols, b1=rows, b2=cols, tile=0, iters=2, scale=d ** -0.5)
    expect = torch.full_like(out, INF)
    expect[..., 1] = -INF
    assert torch.equal(out, expect)
