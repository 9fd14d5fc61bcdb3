"""Stage L backward on resident key ranges of five and six tiles, with fewer workgroups than compute units up to more
than two and a half for each (at 128 features and t < T 513 to 640 take two launches, here 40 heads of 15 columns):
all against the fp32 kernels on the same bf16 tensors.  Bar, in the 2-norm: one bf16 rounding is 1.1e-3 rms (2^-9 / sqrt 3), a gradient
crosses about a dozen of them (every intermediate of the forward pass, both factors of every product of
the reverse sweep), 4e-3 in quadrature; four times that.  (The largest single error is no measure here:
it comes from the one near-tied softmax among 40 heads, 2.2e-2 of the largest gradient, whichever
kernels run.)"""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads", [2, 24, 40])
@pytest.mark.parametrize("f,h,w,d,iters", [(3, 30, 15, 128, 2), (1, 65, 14, 64, 1), (2, 48, 13, 64, 2), (1, 81, 16, 128, 1)])
def test_gradients(f, h, w, d, iters, heads):
    gen = torch.Generator(device="cuda:0").manual_seed(f * h + heads)
    q, k, v, do = (torch.randn(1, heads, f * h * w, d, generator=gen, device="cuda:0").bfloat16() for _ in range(4))
    kw = dict(f_q=f, f_kv=f, h=h, w=w, b1=f * h, b2=w, tile=0, iters=iters, scale=d ** -0.5)
    print(f"case {kw} heads {heads}", flush=True)
    got = pkg.monarch_attn_bwd(q, k, v, do, **kw)
    ref = pkg.monarch_attn_bwd(q, k, v, do, compute=pkg.MRT_COMPUTE_F32, **kw)
    for name, x, r in zip(("dQ", "dK", "dV"), got, ref):
        err = ((x - r).norm() / r.norm()).item()
        print(f"  {name}: rel {err:.2e}", flush=True)
        assert err <= 1.6e-2
