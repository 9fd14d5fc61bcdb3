"""fp32 products formed from bf16 parts: at every size the kernels that do so differ in, what they return
is what the kernels with fp32 operands return (those run where rows are not 16-byte aligned): infinite
and NaN results in the same places, values near the largest fp32 number (their first part rounds to an
infinity) and tiny ones as accurate.

The bar is that of the other fp32 tests (2-norm, 5e-6): two fp32 results a rounding apart in every stage."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

INF = float("inf")
REL = 5e-6

# name: (f, h, w, b1, b2, tile, iters, d, heads, causal chunk)
SIZES = {
    "two-tiles-39-heads": (1, 24, 24, 24, 24, 0, 2, 64, 39, 0),
    "three-tiles-40x33": (1, 40, 33, 40, 33, 0, 2, 128, 8, 0),
    "wave-of-six-90x52": (3, 30, 52, 90, 52, 0, 2, 128, 2, 0),
    "five-tiles-66x80": (1, 66, 80, 66, 80, 0, 2, 64, 2, 0),
    "96-keys-d36": (1, 96, 49, 96, 49, 0, 3, 36, 2, 0),
    "97-keys-two-parts": (1, 97, 20, 97, 20, 0, 2, 128, 2, 0),
    "tile-pair-45x30": (1, 45, 60, 45, 30, 1, 2, 128, 2, 0),
    "three-parts-180": (1, 180, 20, 180, 20, 0, 2, 128, 2, 0),
    "refine-of-twelve-d64": (1, 192, 17, 192, 17, 0, 2, 64, 2, 0),
    "streamed-four-tiles": (2, 50, 48, 50, 24, 1, 2, 128, 2, 0),
    "streamed-ten-tiles": (2, 150, 18, 150, 9, 1, 2, 64, 2, 0),
    "masked-tiles": (4, 33, 20, 33, 20, 1, 2, 64, 3, 2),
    "regular-mask": (6, 7, 18, 42, 18, 0, 2, 64, 4, 2),
    "dense": (2, 9, 13, 0, 0, 0, 0, 128, 2, 0),
    "dense-masked": (6, 9, 13, 0, 0, 0, 0, 64, 2, 2),
}


def both(size, q, k, v):
    """The call on aligned tensors and on ones that start one element off."""
    f, h, w, b1, b2, tile, iters, d, heads, chunk = size
    outs = []
    for shift in (0, 1):
        dev = [torch.zeros(x.numel() + 4, device="cuda:0")[shift:shift + x.numel()].view(x.shape).copy_(x) for x in (q, k, v)]
        out = torch.zeros(q.numel() + 4, device="cuda:0")[shift:shift + q.numel()].view(q.shape)
        args = dict(f_q=f, f_kv=f, h=h, w=w, causal_chunk=chunk, scale=d ** -0.5, out=out)
        if iters == 0:
            pkg.dense_attn_fwd(*dev, **args)
        else:
            pkg.monarch_attn_fwd(*dev, b1=b1, b2=b2, tile=tile, iters=iters, **args)
        outs.append(out)
    torch.cuda.synchronize()
    return outs


def infinite_value(q, k, v):
    v[:, 0, v.shape[2] // 2, 3] = INF


def infinite_keys(q, k, v):
    # logits of plus or minus infinity by the sign of the query's feature, in one key of the first head
    k[:, 0, k.shape[2] // 3, 5] = INF
    q[:, 0, :, 5] = -q[:, 0, :, 5].abs()


def infinite_query(q, k, v):
    q[:, 0, 7, 0] = -INF


def values_near_the_largest(q, k, v):
    v[:, 0, :, 1] = 3.4e38


def tiny_values(q, k, v):
    v *= 1e-25


def wide_values(q, k, v):
    v *= torch.exp(20 * torch.randn(v.shape, generator=torch.Generator(device="cuda:0").manual_seed(3), device="cuda:0"))


@pytest.mark.parametrize("change", [infinite_value, infinite_keys, infinite_query, values_near_the_largest, tiny_values,
                                    wide_values])
@pytest.mark.parametrize("name", list(SIZES))
def test_as_with_fp32_operands(name, change):
    size = SIZES[name]
    f, h, w, d, heads = size[0], size[1], size[2], size[7], size[8]
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    q, k, v = (torch.randn(1, heads, f * h * w, d, generator=gen, device="cuda:0") for _ in range(3))
    change(q, k, v)
    print(f"{name} {change.__name__}", flush=True)
    split, plain = both(size, q, k, v)
    assert torch.equal(split.isnan(), plain.isnan())
    assert torch.equal(split.isinf(), plain.isinf()) and torch.equal(split[split.isinf()], plain[plain.isinf()])
    # feature by feature: wide values must not hide narrow ones
    a, b = (torch.where(x.isfinite(), x, torch.zeros_like(x)).double().flatten(0, -2) for x in (split, plain))
    assert ((a - b).norm(dim=0) <= REL * b.norm(dim=0)).all()
