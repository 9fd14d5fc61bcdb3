"""Streamed stage L in workgroups of eight waves (launches of at most one workgroup a compute unit) and of
four: a head gives the same bits alone and beside enough copies of itself that the launch takes the other
kind, for one to twelve query tiles, with plain inputs and with logits that keep rising along the keys
(every chunk raises the softmax references, of one query tile earlier than of another)."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

CASES = {
    # name: (d, f_kv, h, w, b1, b2, chunk): three frames against f_kv
    "1": (128, 18, 13, 12, 13, 12, 0), "2": (64, 12, 30, 8, 30, 8, 3), "3": (128, 9, 47, 9, 47, 9, 0),
    "4": (128, 9, 21, 10, 63, 10, 3), "5": (64, 9, 25, 11, 75, 11, 3), "6": (128, 15, 30, 9, 90, 9, 3),
    "7": (128, 6, 35, 13, 105, 13, 3), "8": (64, 9, 42, 10, 126, 5, 0), "9": (128, 9, 45, 10, 135, 10, 3),
    "12": (64, 6, 61, 8, 183, 8, 0),
}


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_same_bits(name, rising):
    d, f_kv, h, w, b1, b2, chunk = CASES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(len(name))

    def draw(frames):
        return torch.randn(1, 1, frames * h * w, d, generator=gen, device="cuda:0")

    q, k, v = draw(3), draw(f_kv), draw(f_kv)
    if rising:       # rows of a column: the query's first feature grows, the keys' with it, by rows
        rows = torch.arange(f_kv * h * w, device="cuda:0") // w
        k[..., 0] = 0.25 * rows
        q[..., 0] = 1.0 + (rows[:q.shape[2]] % b1) / 16.0
    copies = 256 // (w * (3 * h // b1)) + 1
    args = dict(f_q=3, f_kv=f_kv, h=h, w=w, b1=b1, b2=b2, tile=1, iters=2, causal_chunk=chunk,
                q_frame_offset=f_kv - 3 if chunk else 0, scale=d ** -0.5, head_groups=1)
    q, k, v = (x.bfloat16() for x in (q, k, v))
    print(f"case {name} rising {rising} copies {copies}", flush=True)
    one = pkg.monarch_attn_fwd(q, k, v, **args)
    many = pkg.monarch_attn_fwd(*(x.expand(1, copies, *x.shape[2:]).contiguous() for x in (q, k, v)), **args)
    assert torch.isfinite(one.float()).all()
    for i in (0, copies - 1):
        assert torch.equal(many[:, i:i + 1], one)
