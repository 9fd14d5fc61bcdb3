"""Stage L backward from the forward call's row statistics (saved training steps of more than 192 key
rows): one to six query tiles at their edges, key ranges that end anywhere in a wave's 32 keys or leave
waves without any (short visible ranges under the mask), neighbourhood tiles, both feature counts, a second
iteration, two sequences and unpacked tensors.
Gradients against the fp32 kernels with the bar of the bf16 backward pass (2e-2 of the largest entry)."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

CASES = {
    # name: (heads, d, f, h, w, b1, b2, chunk, tile_h)
    "one-row": (1, 128, 13, 16, 6, 1, 3, 0, 0),
    "one-tile": (2, 128, 14, 16, 10, 16, 5, 0, 0),
    "two-tiles-first": (1, 64, 12, 17, 9, 17, 9, 3, 0),
    "two-tiles": (1, 128, 7, 32, 7, 32, 7, 1, 0),
    "three-tiles": (2, 64, 6, 33, 8, 33, 4, 2, 0),
    "four-tiles": (1, 128, 4, 64, 5, 64, 5, 1, 0),
    "five-tiles": (1, 128, 6, 39, 11, 78, 11, 2, 0),
    "five-tiles-first": (2, 64, 5, 65, 6, 65, 6, 0, 0),
    "six-tiles": (1, 128, 12, 32, 10, 96, 10, 3, 0),
    "six-tiles-64": (1, 64, 9, 30, 12, 90, 12, 3, 0),
    "bands": (1, 128, 8, 20, 12, 20, 6, 2, 10),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gradients(name):
    heads, d, f, h, w, b1, b2, chunk, tile_h = CASES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(len(name))
    q, k, v, do = (torch.randn(1, heads, f * h * w, d, generator=gen, device="cuda:0").bfloat16() for _ in range(4))
    args = dict(f_q=f, f_kv=f, h=h, w=w, b1=b1, b2=b2, tile=1, iters=1, causal_chunk=chunk, tile_h=tile_h, scale=d ** -0.5)
    print(f"case {name}", flush=True)
    o, saved = pkg.monarch_attn_fwd_save(q, k, v, **args)
    got = pkg.monarch_attn_bwd_saved(q, k, v, do, saved, **args)
    again = pkg.monarch_attn_bwd_saved(q, k, v, do, saved, **args)
    want = pkg.monarch_attn_bwd(q, k, v, do, compute=pkg.MRT_COMPUTE_F32, **args)
    for which, x, y, z in zip(("dQ", "dK", "dV"), got, again, want):
        err = ((x - z).abs().max() / z.abs().max()).item()
        print(f"  {which} {err:.2e}", flush=True)
        assert torch.equal(x, y) and err <= 2e-2


@pytest.mark.parametrize("name", ["one-tile", "two-tiles-first", "five-tiles", "six-tiles", "six-tiles-64"])
def test_two_iterations_batches_and_strides(name):
    # (the sweep at t = 2 writes the dQ that t = 1 adds to; tokens before heads, two sequences)
    heads, d, f, h, w, b1, b2, chunk, tile_h = CASES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(len(name) + 1)
    q, k, v, do = (torch.randn(2, f * h * w, heads, d, generator=gen, device="cuda:0").bfloat16().permute(0, 2, 1, 3)
                   for _ in range(4))
    args = dict(f_q=f, f_kv=f, h=h, w=w, b1=b1, b2=b2, tile=1, iters=2, causal_chunk=chunk, tile_h=tile_h, scale=d ** -0.5)
    print(f"case {name}", flush=True)
    o, saved = pkg.monarch_attn_fwd_save(q, k, v, **args)
    got = pkg.monarch_attn_bwd_saved(q, k, v, do, saved, **args)
    packed = [x.contiguous() for x in (q, k, v, do)]
    o, saved = pkg.monarch_attn_fwd_save(*packed[:3], **args)
    again = pkg.monarch_attn_bwd_saved(*packed, saved, **args)
    want = pkg.monarch_attn_bwd(*packed, compute=pkg.MRT_COMPUTE_F32, **args)
    for which, x, y, z in zip(("dQ", "dK", "dV"), got, again, want):
        err = ((x - z).abs().max() / z.abs().max()).item()
        print(f"  {which} {err:.2e}", flush=True)
        assert torch.equal(x, y) and err <= 2e-2
