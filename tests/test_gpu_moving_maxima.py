"""The online softmaxes whose reference is raised only when a logit exceeds it by more than eight: the
streamed stage L kernels (bf16: output at four and eight waves, first pass of the refine kernel) and the
fp32 kernels' chunk loop (dense, stage L output and refine).  Crafted keys make the logits of a query
rise steadily over the keys (the reference is raised many times, at different chunks for the queries of
one wave), fall, zig-zag or hold one spike; against the fp64 oracle on the same rounded inputs.

Stage L sees the crafted logits themselves: the profile sits in two features that the two columns of a key
row share, so every convex combination alpha_L of them has it unrounded, and c_L (an entropy of two
keys) lies in [-0.7, 0].  With one column (one iteration) alpha_L = K and c_L = 0."""
import numpy as np
import pytest
import torch

import paper_2602_12271_amd as pkg
from workloads import synthetic as syn

from gpu_harness import oracle_dense_head, oracle_monarch_head, run_dense_gpu, run_monarch_gpu, to_device

pytestmark = pytest.mark.gpu

PROFILES = ["rising", "falling", "zigzag", "spike"]


def crafted(wl, profile, seed, cols, noise=0.1):
    """Q and K with logit(i, k) = amp_i shape_k plus noise, amp_i between 31 and 57 natural units at 128
    features and 44 and 80 at 64, shape_k in [-1, 1] over the key rows; bf16-representable."""
    rng = np.random.default_rng(seed)
    nk = wl.n_kv // cols
    x = np.linspace(-1.0, 1.0, nk)
    shape = dict(rising=x, falling=-x, zigzag=np.where(np.arange(nk) % 64 < 32, x, -x),
                 spike=np.where(np.arange(nk) == (2 * nk) // 3, 1.0, -1.0 + 0.05 * rng.standard_normal(nk)))[profile]
    shape = np.repeat(shape, cols)
    Q = noise * rng.standard_normal((1, wl.heads, wl.n_q, wl.head_dim)).astype(np.float32)
    K = noise * rng.standard_normal((1, wl.heads, wl.n_kv, wl.head_dim)).astype(np.float32)
    Q[..., 0] = 24.0 * rng.uniform(0.5, 1.0, size=(1, wl.heads, wl.n_q))
    Q[..., 1] = 8.0
    K[..., 0] = 24.0 * shape
    K[..., 1] = 8.0 * shape
    V = rng.standard_normal(K.shape).astype(np.float32)
    return tuple(syn.round_to_bf16(a) for a in (Q, K, V))


def workload(dtype, d, f_q, f_kv, h, w, iters=1, b1=1, b2=1, tile=0, **kw):
    return syn.Workload("moving", 1, 2, d, f_q, f_kv, h, w, b1, b2, tile, iters, kw.pop("chunk", 0), kw.pop("off", 0),
                        dtype, d ** -0.5, False, **kw)


def distance(wl, arrays, out, oracle):
    num = den = 0.0
    for hd in range(wl.heads):
        ref = oracle(wl, *(x[0, hd] for x in arrays))
        num += (out[0, hd].double().cpu() - ref).pow(2).sum().item()
        den += ref.pow(2).sum().item()
    return (num / den) ** 0.5


# (rows of a tile, key tiles): waves of one tile, waves of two, eight waves; 336, 400 and 450 key rows
SIZES = [(48, 7), (80, 5), (150, 3)]


# bar: four times the 3.7e-3 (2-norm) that the bf16 roundings of the forward pass show
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,tiles", SIZES)
@pytest.mark.parametrize("profile", PROFILES)
def test_bf16_stage_l_output(profile, rows, tiles, d):
    wl = workload("bf16", d, 1, tiles, rows, 1, b1=rows, b2=1, tile=1)
    arrays = crafted(wl, profile, rows + d, 1)
    out = run_monarch_gpu(wl, *to_device(wl, arrays))
    err = distance(wl, arrays, out, oracle_monarch_head)
    print(f"  {profile} {rows} x {tiles}, {d} features: rel {err:.2e}", flush=True)
    assert err <= 1.5e-2


# The statistics of the refine kernel's first pass weigh the query rows of each key's abar, which chooses
# between the two columns of the key row in the second iteration.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,tiles", SIZES)
@pytest.mark.parametrize("profile", PROFILES)
def test_bf16_stage_l_refine(profile, rows, tiles, d):
    wl = workload("bf16", d, 1, tiles, rows, 2, iters=2, b1=rows, b2=2, tile=1)
    arrays = crafted(wl, profile, rows + d, 2, noise=1.0)
    out = run_monarch_gpu(wl, *to_device(wl, arrays))
    err = distance(wl, arrays, out, oracle_monarch_head)
    print(f"  {profile} {rows} x {tiles}, {d} features: rel {err:.2e}", flush=True)
    assert err <= 1.5e-2


# fp32 bar: a logit of 80 carries an fp32 rounding of 4e-6, which is the relative error of its weight;
# with the scaling before it and the stages after it four times that
REL_F32 = 2e-5


@pytest.mark.parametrize("d", [64, 100, 128])
@pytest.mark.parametrize("grid", [(1, 1, 7, 13, 0, 0), (2, 9, 5, 9, 0, 7), (6, 6, 7, 19, 2, 0)])
@pytest.mark.parametrize("profile", PROFILES)
def test_fp32_dense(profile, grid, d):
    f_q, f_kv, h, w, chunk, off = grid
    wl = workload("f32", d, f_q, f_kv, h, w, chunk=chunk, off=off)
    arrays = crafted(wl, profile, h + d, 1)
    err = distance(wl, arrays, run_dense_gpu(wl, *to_device(wl, arrays)), oracle_dense_head)
    print(f"  {profile} {grid}, {d} features: rel {err:.2e}", flush=True)
    assert err <= REL_F32


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,tiles", [(30, 3), (50, 5), (150, 3)])
@pytest.mark.parametrize("iters", [1, 2])
@pytest.mark.parametrize("profile", PROFILES)
def test_fp32_stage_l(profile, iters, rows, tiles, d):
    wl = workload("f32", d, 1, tiles, rows, 2, iters=iters, b1=rows, b2=2, tile=1)
    arrays = crafted(wl, profile, rows + d, 2, noise=1.0)
    err = distance(wl, arrays, run_monarch_gpu(wl, *to_device(wl, arrays)), oracle_monarch_head)
    print(f"  {profile} {rows} x {tiles}, {iters} iterations, {d} features: rel {err:.2e}", flush=True)
    assert err <= REL_F32


# Regular blocks of 129 to 144 rows under the chunk-causal mask: the streamed output kernel with hidden keys
# (whole 32-key chunks hidden from a query row, and its chunk's end inside one), also where it leaves the
# row statistics for the sweep.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("f,h,chunk,off", [(3, 43, 1, 0), (3, 45, 1, 0), (9, 15, 2, 1), (6, 24, 2, 0), (8, 18, 3, 0)])
def test_masked_blocks_of_129_to_144_rows(f, h, chunk, off, d):
    wl = workload("bf16", d, f, f, h, 9, iters=1 + f % 2, b1=f * h, b2=9, tile=0, chunk=chunk, off=off)
    arrays = syn.make_inputs(wl)
    rng = np.random.default_rng(h)
    dO = syn.round_to_bf16(rng.standard_normal(arrays[0].shape).astype(np.float32))
    q, k, v, do = to_device(wl, arrays + (dO,))
    kw = dict(f_q=f, f_kv=f, h=h, w=9, b1=f * h, b2=9, tile=0, iters=wl.iters, causal_chunk=chunk, q_frame_offset=off,
              scale=wl.scale)
    out = pkg.monarch_attn_fwd(q, k, v, **kw)
    assert distance(wl, arrays, out, oracle_monarch_head) <= 1.5e-2
    saved_out, saved = pkg.monarch_attn_fwd_save(q, k, v, **kw)
    assert torch.equal(saved_out, out)
    from oracle import monarch_oracle as mo
    for grads in (pkg.monarch_attn_bwd(q, k, v, do, **kw), pkg.monarch_attn_bwd_saved(q, k, v, do, saved, **kw)):
        for hd in range(wl.heads):
            ref = mo.monarch_attn_grad(*(torch.from_numpy(x[0, hd]) for x in arrays), torch.from_numpy(dO[0, hd]), **kw)
            for name, got, want in zip(("dQ", "dK", "dV"), grads, ref):
                err = ((got[0, hd].double().cpu() - want).norm() / want.norm()).item()
                print(f"  head {hd} {name}: rel {err:.2e}", flush=True)
                assert err <= 1.6e-2
