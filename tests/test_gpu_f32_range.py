"""The fp32 path over the whole range of fp32 numbers: inputs whose bf16 parts would fall below the smallest
bf16 number, weights of the softmaxes down to the smallest fp32 number.  Products of split operands (aligned
rows) have to return what products of fp32 operands return (rows that start one element off).

Bar of the 2-norm comparisons: that of the other fp32 tests, 5e-6.  Single weights e^-z carry the rounding of
their logit, z 2^-24 relative and as much again per product of the dot product: 1e-4 at z = 87 is 20 of them."""
import pytest
import torch

import paper_2602_12271_amd as pkg

pytestmark = pytest.mark.gpu

REL = 5e-6

# f, h, w, b1, b2, tile, iters, d, heads, causal chunk
SIZES = {
    "three-tiles-40x33": (1, 40, 33, 40, 33, 0, 2, 128, 8, 0),
    "wave-of-six-90x52": (3, 30, 52, 90, 52, 0, 2, 128, 2, 0),
    "97-keys-two-parts": (1, 97, 20, 97, 20, 0, 2, 128, 2, 0),
    "refine-of-twelve-d64": (1, 192, 17, 192, 17, 0, 2, 64, 2, 0),
    "streamed-four-tiles": (2, 50, 48, 50, 24, 1, 2, 128, 2, 0),
    "regular-mask-d36": (6, 7, 34, 42, 34, 0, 2, 36, 4, 2),
    "dense": (2, 9, 13, 0, 0, 0, 0, 128, 2, 0),
    "dense-masked": (6, 9, 13, 0, 0, 0, 0, 64, 2, 2),
}


def call(size, q, k, v, scale, out):
    f, h, w, b1, b2, tile, iters, d, heads, chunk = size
    args = dict(f_q=f, f_kv=f, h=h, w=w, causal_chunk=chunk, scale=scale, out=out)
    if iters == 0:
        return pkg.dense_attn_fwd(q, k, v, **args)
    return pkg.monarch_attn_fwd(q, k, v, b1=b1, b2=b2, tile=tile, iters=iters, **args)


def both(size, q, k, v, scale):
    """The call on aligned tensors and on ones that start one element off."""
    outs = []
    for shift in (0, 1):
        dev = [torch.zeros(x.numel() + 4, device="cuda:0")[shift:shift + x.numel()].view(x.shape).copy_(x) for x in (q, k, v)]
        out = torch.zeros(q.numel() + 4, device="cuda:0")[shift:shift + q.numel()].view(q.shape)
        outs.append(call(size, *dev, scale, out))
    torch.cuda.synchronize()
    return outs


def inputs(size, seed):
    f, h, w, d, heads = size[0], size[1], size[2], size[7], size[8]
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    return [torch.randn(1, heads, f * h * w, d, generator=gen, device="cuda:0") for _ in range(3)]


def assert_same(split, plain):
    assert torch.isfinite(plain).all() and plain.abs().max() > 0
    a, b = (x.double().flatten(0, -2) for x in (split, plain))
    err = ((a - b).norm(dim=0) / b.norm(dim=0)).max().item()
    print(f"  rel {err:.2e}", flush=True)
    assert err <= REL


@pytest.mark.parametrize("factor", [1e-28, 1e-31, 1e-34, 1e-36])
@pytest.mark.parametrize("name", list(SIZES))
def test_tiny_values(name, factor):
    size = SIZES[name]
    q, k, v = inputs(size, 5)
    print(f"{name} {factor}", flush=True)
    assert_same(*both(size, q, k, factor * v, size[7] ** -0.5))


@pytest.mark.parametrize("name", list(SIZES))
def test_a_few_tiny_values_of_one_feature(name):
    size = SIZES[name]
    q, k, v = inputs(size, 6)
    v[:, :, :, 2] *= 3e-36
    v[:, :, ::3, 2] = 0
    print(name, flush=True)
    assert_same(*both(size, q, k, v, size[7] ** -0.5))


@pytest.mark.parametrize("which", ["keys", "queries"])
@pytest.mark.parametrize("name", list(SIZES))
def test_tiny_keys_or_queries_against_huge_ones(name, which):
    # logits of order one
    size = SIZES[name]
    q, k, v = inputs(size, 7)
    q, k = (q * 1e30, k * 1e-35) if which == "keys" else (q * 1e-35, k * 1e30)
    print(f"{name} {which}", flush=True)
    assert_same(*both(size, q, k, v, 1e5 * size[7] ** -0.5))


@pytest.mark.parametrize("name", list(SIZES))
def test_tiny_keys_against_some_huge_queries(name):
    # averages of keys are formed where the queries are small and meet huge ones later
    size = SIZES[name]
    q, k, v = inputs(size, 8)
    q[:, :, 1::3] *= 1e34
    k *= 3e-36
    print(name, flush=True)
    assert_same(*both(size, q, k, v, size[7] ** -0.5))


@pytest.mark.parametrize("d", [64, 128])
def test_every_weight_of_the_dense_softmax(d):
    # value row i has a one at feature i: the output is the matrix of the weights, e^0 .. e^-103
    n = 64
    q = torch.zeros(1, 2, n, d, device="cuda:0")
    k, v = torch.zeros_like(q), torch.zeros_like(q)
    q[..., 0] = 1 + torch.arange(n, device="cuda:0") / n
    k[..., 0] = -51.5 * torch.arange(n, device="cuda:0") / n
    v[:, :, torch.arange(n), torch.arange(n)] = 1
    split, plain = both((1, 8, 8, 0, 0, 0, 0, d, 2, 0), q, k, v, 1.0)
    expect = torch.softmax(torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()), -1)
    for out in (split, plain):
        w = out[..., :n].double()
        normal = expect > 2.0 ** -125
        assert ((w - expect).abs() <= 1e-4 * expect)[normal].all()
        assert ((w - expect).abs() <= 2.0 ** -140)[~normal].all()


@pytest.mark.parametrize("name,rows,cols", [("weights-of-r", 40, 64), ("weights-of-l", 64, 40), ("weights-of-l-streamed", 48, 40),
                                            ("weights-of-l-wide", 128, 40)])
def test_every_weight_of_one_iteration(name, rows, cols):
    # the values of one block column (or row) are ones at their own feature, the others zeros
    f = 3 if name.endswith("streamed") else 1
    d, n = 128, rows * cols
    heads = 8
    x, y = torch.arange(f * n, device="cuda:0") // cols, torch.arange(f * n, device="cuda:0") % cols
    along = y if name == "weights-of-r" else x
    length = cols if name == "weights-of-r" else f * rows
    q = torch.zeros(1, heads, f * n, d, device="cuda:0")
    k, v = torch.zeros_like(q), torch.zeros_like(q)
    q[..., 0] = 1.0
    k[..., 0] = -103.0 * along / length
    v[:, :, torch.arange(f * n), along % d] = 1
    size = (f, rows, cols, rows, cols, 1 if f > 1 else 0, 1, d, heads, 0)
    split, plain = both(size, q, k, v, 1.0)
    assert plain.min() < 1e-30
    normal = plain > 2.0 ** -125
    assert ((split - plain).abs() <= 1e-4 * plain)[normal].all()
    assert ((split - plain).abs() <= 2.0 ** -140)[~normal].all()


@pytest.mark.parametrize("rows,cols,d,heads", [(24, 24, 64, 1), (40, 33, 128, 8), (90, 52, 128, 2), (10, 16, 64, 2)])
def test_logits_near_the_largest_number(rows, cols, d, heads):
    # one key of every block row has the logit 2e38, the others -2e38: R picks it, its entropy is 0, and L weighs
    # the rows alike, so that the output is the mean of those keys' values over the rows
    gen = torch.Generator(device="cuda:0").manual_seed(rows)
    n = rows * cols
    v = torch.randn(1, heads, n, d, generator=gen, device="cuda:0")
    q, k = torch.zeros_like(v), torch.zeros_like(v)
    pick = torch.randint(cols, (heads, rows), generator=gen, device="cuda:0") + cols * torch.arange(rows, device="cuda:0")
    q[..., 0] = 1.4e19
    k[..., 0] = -1.43e19
    k[0, :, :, 0].scatter_(1, pick, 1.43e19)
    expect = torch.gather(v[0].double(), 1, pick[..., None].expand(-1, -1, d)).mean(1, keepdim=True)
    for out in both((1, rows, cols, rows, cols, 0, 1, d, heads, 0), q, k, v, 1.0):
        assert (out[0].double() - expect).norm() <= REL * expect.norm() * n ** 0.5


@pytest.mark.parametrize("rows,cols,d", [(24, 24, 64), (32, 20, 64), (17, 33, 128), (40, 33, 128), (33, 48, 64), (30, 52, 128)])
def test_same_bits_for_any_number_of_heads_and_sequences(rows, cols, d):
    heads = 16
    gen = torch.Generator(device="cuda:0").manual_seed(rows)
    q, k, v = (torch.randn(1, heads, rows * cols, d, generator=gen, device="cuda:0") for _ in range(3))

    def run(*x):
        return pkg.monarch_attn_fwd(*x, f_q=1, f_kv=1, h=rows, w=cols, b1=rows, b2=cols, tile=0, iters=2, scale=d ** -0.5)
    whole = run(q, k, v)
    for some in (1, 5):
        assert torch.equal(run(*(x[:, :some].contiguous() for x in (q, k, v))), whole[:, :some])
    assert torch.equal(run(*(x.transpose(0, 1).contiguous() for x in (q, k, v))).transpose(0, 1), whole)
