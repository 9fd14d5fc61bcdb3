"""Stage R backward of up to 16 columns, where a wave owns whole key blocks: one to sixteen columns, both
feature counts, more and fewer key blocks than waves, several query tiles a block, blocks that no query
tile sees, two iterations (d abar of the second, dK added to), neighbourhood tiles, packed and unpacked
rows.  Against the fp32 kernels with the bar of the bf16 backward pass (2e-2 of the largest entry)."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

CASES = {
    # name: (heads, d, f_q, f_kv, h, w, b1, b2, tile, iters, chunk, offset, tile_h)
    "one-column": (1, 128, 2, 2, 9, 1, 18, 1, 0, 1, 0, 0, 0),
    "sixteen": (2, 64, 2, 2, 17, 16, 34, 16, 0, 2, 0, 0, 0),
    "fifteen": (1, 128, 3, 3, 20, 15, 60, 15, 0, 2, 0, 0, 0),
    "tiles": (2, 128, 6, 6, 20, 26, 20, 13, 1, 1, 3, 0, 0),
    "tiles-two-iterations": (1, 64, 4, 4, 12, 16, 12, 8, 1, 2, 2, 0, 0),
    "unseen-blocks": (1, 128, 2, 6, 10, 12, 10, 6, 1, 2, 2, 0, 0),
    "unseen-blocks-offset": (2, 64, 2, 6, 10, 12, 20, 12, 1, 1, 2, 2, 0),
    "many-blocks": (3, 64, 8, 8, 30, 32, 30, 16, 1, 1, 2, 0, 0),
    "bands": (1, 128, 4, 4, 20, 24, 20, 12, 1, 1, 2, 0, 10),
}


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_gradients(name, packed):
    heads, d, f_q, f_kv, h, w, b1, b2, tile, iters, chunk, offset, tile_h = CASES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(len(name))

    def draw(frames):
        x = torch.randn(1, heads, frames * h * w, d, generator=gen, device="cuda:0").bfloat16()
        return x if packed else x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)   # tokens before heads

    q, do, k, v = draw(f_q), draw(f_q), draw(f_kv), draw(f_kv)
    args = dict(f_q=f_q, f_kv=f_kv, h=h, w=w, b1=b1, b2=b2, tile=tile, iters=iters, causal_chunk=chunk,
                q_frame_offset=offset, tile_h=tile_h, scale=d ** -0.5)
    print(f"case {name} packed {packed}", flush=True)
    got = pkg.monarch_attn_bwd(q, k, v, do, **args)
    again = pkg.monarch_attn_bwd(q, k, v, do, **args)
    want = pkg.monarch_attn_bwd(q, k, v, do, compute=pkg.MRT_COMPUTE_F32, **args)
    for which, x, y, z in zip(("dQ", "dK", "dV"), got, again, want):
        err = ((x - z).abs().max() / z.abs().max()).item()
        print(f"  {which} {err:.2e}", flush=True)
        assert torch.equal(x, y) and err <= 2e-2
