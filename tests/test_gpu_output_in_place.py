"""O in the place of Q: every kernel that writes O has read its rows of Q by then, also where an fp32 workgroup
does its work a second time (one of its products is an infinity).  The same bits as with an O of its own."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

# f, h, w, b1, b2, tile, iters, d, heads, causal chunk
SIZES = {
    "24x24": (1, 24, 24, 24, 24, 0, 2, 64, 1, 0),
    "40x33": (1, 40, 33, 40, 33, 0, 2, 128, 8, 0),
    "90x52": (3, 30, 52, 90, 52, 0, 2, 128, 2, 0),
    "97-rows": (1, 97, 20, 97, 20, 0, 2, 128, 2, 0),
    "156-rows": (1, 156, 12, 156, 12, 0, 1, 128, 2, 0),
    "192-rows": (1, 192, 8, 192, 8, 0, 2, 128, 1, 0),
    "192-rows-d64": (1, 192, 17, 192, 17, 0, 2, 64, 2, 0),
    "streamed": (2, 50, 48, 50, 24, 1, 2, 128, 2, 0),
    "streamed-masked": (6, 40, 10, 120, 10, 1, 2, 64, 2, 3),
    "regular-mask": (6, 7, 34, 42, 34, 0, 2, 64, 4, 2),
    "dense": (2, 9, 13, 0, 0, 0, 0, 128, 2, 0),
    "dense-long": (3, 30, 20, 0, 0, 0, 0, 64, 2, 0),
    "dense-masked": (6, 9, 13, 0, 0, 0, 0, 64, 2, 2),
}


@pytest.mark.parametrize("dtype", ["f32", "f32-infinity", "f32-elements", "bf16"])
@pytest.mark.parametrize("name", list(SIZES))
def test_same_bits(name, dtype):
    f, h, w, b1, b2, tile, iters, d, heads, chunk = SIZES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    q, k, v = (torch.randn(1, heads, f * h * w, d, generator=gen, device="cuda:0") for _ in range(3))
    if dtype == "f32-infinity":
        v[:, 0, v.shape[2] // 2, 3] = float("inf")
    if dtype == "bf16":
        q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    if dtype == "f32-elements":
        q = torch.zeros(q.numel() + 1, device="cuda:0")[1:].view(q.shape).copy_(q)
    print(f"{name} {dtype}", flush=True)

    def call(out):
        args = dict(f_q=f, f_kv=f, h=h, w=w, causal_chunk=chunk, scale=d ** -0.5, out=out)
        if iters == 0:
            return pkg.dense_attn_fwd(q, k, v, **args)
        return pkg.monarch_attn_fwd(q, k, v, b1=b1, b2=b2, tile=tile, iters=iters, **args)
    expect = call(torch.zeros(q.numel() + 1, dtype=q.dtype, device="cuda:0")[1:].view(q.shape)
                  if dtype == "f32-elements" else torch.empty_like(q))
    got = call(q)
    torch.cuda.synchronize()
    assert torch.equal(got.isnan(), expect.isnan()) and torch.equal(got.nan_to_num(), expect.nan_to_num())
