"""Stage L backward of resident key ranges, rows and columns in one launch: the numbers of query and key
tiles on either side of what a workgroup's waves own, blocks whose key range is two or three tiles of
fewer query rows, masks, one to three iterations, against the fp32 kernels on the same bf16 tensors.  Bar, in the 2-norm:
about a dozen bf16 roundings of 1.1e-3 rms each (2^-9 / sqrt 3) in quadrature, 4e-3; four times that."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

# f, h, w, b1, b2, tile, iters, d, causal chunk
SIZES = [
    (1, 1, 5, 1, 5, 0, 2, 64, 0),
    (1, 16, 9, 16, 9, 0, 1, 128, 0),
    (1, 17, 18, 17, 18, 0, 2, 128, 0),
    (1, 32, 10, 32, 10, 0, 3, 64, 0),
    (1, 33, 7, 33, 7, 0, 2, 64, 0),
    (2, 24, 20, 48, 20, 0, 1, 128, 0),
    (1, 64, 6, 64, 6, 0, 2, 128, 0),
    (1, 65, 17, 65, 17, 0, 2, 128, 0),
    (1, 80, 33, 80, 33, 0, 2, 64, 0),
    (1, 96, 11, 96, 11, 0, 2, 128, 0),
    (1, 15, 24, 15, 12, 1, 2, 128, 0),
    (1, 17, 24, 17, 12, 1, 2, 64, 0),
    (1, 48, 20, 48, 10, 1, 2, 128, 0),
    (1, 31, 27, 31, 9, 1, 1, 64, 0),
    (3, 20, 12, 20, 12, 1, 2, 128, 1),
    (6, 13, 8, 78, 8, 0, 2, 64, 2),
]


@pytest.mark.parametrize("size", SIZES, ids=str)
def test_gradients(size):
    f, h, w, b1, b2, tile, iters, d, chunk = size
    gen = torch.Generator(device="cuda:0").manual_seed(b1 + w)
    q, k, v, do = (torch.randn(2, 2, f * h * w, d, generator=gen, device="cuda:0").bfloat16() for _ in range(4))
    kw = dict(f_q=f, f_kv=f, h=h, w=w, b1=b1, b2=b2, tile=tile, iters=iters, causal_chunk=chunk, scale=d ** -0.5)
    print(f"case {kw}", flush=True)
    got = pkg.monarch_attn_bwd(q, k, v, do, **kw)
    ref = pkg.monarch_attn_bwd(q, k, v, do, compute=pkg.MRT_COMPUTE_F32, **kw)
    _, saved = pkg.monarch_attn_fwd_save(q, k, v, **kw)
    again = pkg.monarch_attn_bwd_saved(q, k, v, do, saved, **kw)
    for name, x, r, s in zip(("dQ", "dK", "dV"), got, ref, again):
        err = ((x - r).norm() / r.norm()).item()
        print(f"  {name}: rel {err:.2e}", flush=True)
        assert err <= 1.6e-2
        assert torch.equal(x, s)
