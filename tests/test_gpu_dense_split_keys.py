"""bf16 dense calls whose keys are split over several workgroups (few queries, many keys): every workgroup
shape at ragged sizes, under the mask with hidden keys, with query ranges whose key counts differ (where
some parts of a workgroup's keys are empty and one workgroup's halves end at different keys), with infinite
values that only the last chunk sees, and with softmax references beyond 2^20.  Against plain torch in float64 with the bar of the
unsplit kernels (output and probabilities rounded once each to 2^-9: 2.4e-3 in the 2-norm; four times
that), and against the unsplit call, whose probabilities are rounded relative to other references: two
roundings of 2^-9 apart in the 2-norm at most."""
import ctypes

import pytest
import torch

import paper_2602_12271_amd as pkg
from paper_2602_12271_amd import binding

from test_gpu_dense_variants import reference

pytestmark = pytest.mark.gpu

CASES = {
    # name (the shape the rule takes): (heads, d, f_q, f_kv, h, w, chunk, offset)
    "64": (2, 128, 3, 12, 16, 17, 3, 9),
    "64-few-steps": (1, 128, 3, 6, 12, 16, 3, 3),
    "64-ragged-steps": (1, 128, 9, 9, 16, 39, 3, 0),
    "128-steps": (1, 128, 9, 9, 16, 40, 3, 0),
    "256": (1, 128, 3, 9, 40, 59, 3, 6),
    "256-no-mask": (1, 128, 3, 3, 45, 61, 0, 0),
    "256-steps": (2, 128, 12, 12, 20, 37, 3, 0),
    "256-hidden": (2, 128, 3, 12, 44, 35, 3, 3),
    "d64-64": (1, 64, 3, 12, 45, 23, 3, 9),
    "d64-64-steps": (2, 64, 9, 9, 20, 37, 3, 0),
    "d64-128": (4, 64, 3, 12, 42, 20, 3, 9),
}


def problem(name, **kw):
    heads, d, f_q, f_kv, h, w, chunk, offset = CASES[name]
    return binding.make_problem(batch=1, heads=heads, head_dim=d, f_q=f_q, f_kv=f_kv, h=h, w=w, q_frame_offset=offset,
                                scale=2.0 * d ** -0.5, **kw), chunk


def inputs(name, packed=True):
    heads, d, f_q, f_kv, h, w, chunk, offset = CASES[name]
    gen = torch.Generator(device="cuda:0").manual_seed(len(name))

    def draw(n):
        x = torch.randn(1, heads, n, d, generator=gen, device="cuda:0").bfloat16()
        return x if packed else x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)

    args = dict(f_q=f_q, f_kv=f_kv, h=h, w=w, causal_chunk=chunk, q_frame_offset=offset, scale=2.0 * d ** -0.5)
    return [draw(f_q * h * w), draw(f_kv * h * w), draw(f_kv * h * w)], args


def unsplit(tensors, args):
    # a workspace too small for the parts is not used
    return pkg.dense_attn_fwd(*tensors, **args, workspace=torch.empty(256, dtype=torch.uint8, device="cuda:0"))


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_split(name, packed):
    tensors, args = inputs(name, packed)
    print(f"case {name} packed {packed}", flush=True)
    nbytes = binding.dense_attn_workspace_bytes(*problem(name))
    assert nbytes > 0
    scratch = torch.full((nbytes // 4,), float("nan"), device="cuda:0")
    out = pkg.dense_attn_fwd(*tensors, **args, workspace=scratch)
    assert torch.equal(out, pkg.dense_attn_fwd(*tensors, **args))
    one = unsplit(tensors, args).double()
    ref = reference(*tensors, args["h"] * args["w"], args["causal_chunk"], args["q_frame_offset"], args["scale"])
    err, apart = ((out.double() - x).norm() / x.norm() for x in (ref, one))
    print(f"  rel {err:.2e}, from the unsplit call {apart:.2e}", flush=True)
    assert err <= 1e-2 and apart <= 2.0 ** -8


@pytest.mark.parametrize("name", ["64-ragged-steps", "128-steps", "256-steps", "d64-64-steps"])
def test_infinite_values_of_the_last_chunk(name):
    # (queries that share a workgroup, or its half, with one that sees them have them times zero in either call)
    (q, k, v), args = inputs(name)
    seen = args["h"] * args["w"] * (args["f_q"] - args["causal_chunk"])     # tokens before the last chunk
    expect = pkg.dense_attn_fwd(q, k, v, **args)[:, :, :seen]
    v[:, :, seen:] = float("inf")
    out, one = pkg.dense_attn_fwd(q, k, v, **args)[:, :, :seen], unsplit((q, k, v), args)[:, :, :seen]
    assert not (out.isnan() & ~one.isnan()).any() and not out.isinf().any()
    assert torch.equal(out[~out.isnan()], expect[~out.isnan()]) and out.isnan().sum() < 128 * q.shape[1] * q.shape[3]


@pytest.mark.parametrize("name", ["64", "64-ragged-steps", "128-steps", "256-steps", "256-hidden", "d64-64-steps", "d64-128"])
def test_references_far_from_zero(name):
    # Logits around 2^22 (their products exact in fp32), where a reference is a rounded logit: of two queries in
    # three the parts of the first keys have such a reference and those of the others zero, the weight lying once
    # on the former and once on the latter, on keys of one logit (the next is 2^18 below); of the third query all
    # logits are zero.  Weights are then equal or zero in any precision; O's rounding is left.
    (q, k, v), args = inputs(name)
    args["scale"] = 1.0
    q.zero_(), k.zero_()
    at = torch.arange(q.shape[2], device="cuda:0")
    q[..., 0] = (at % 3 - 1) * 2.0 ** 12
    at = torch.arange(k.shape[2], device="cuda:0")
    k[..., 0] = torch.where(at < k.shape[2] // 2, 64.0 * (16 - at % 7), torch.zeros(()).to(at.device))
    out, one = pkg.dense_attn_fwd(q, k, v, **args).double(), unsplit((q, k, v), args).double()
    ref = reference(q, k, v, args["h"] * args["w"], args["causal_chunk"], args["q_frame_offset"], 1.0)
    err, apart = ((out - x).norm() / x.norm() for x in (ref, one))
    print(f"case {name}: rel {err:.2e}, from the unsplit call {apart:.2e}", flush=True)
    assert err <= 1e-2 and apart <= 2.0 ** -8


def test_output_in_the_place_of_the_queries():
    (q, k, v), args = inputs("64")
    expect = pkg.dense_attn_fwd(q, k, v, **args)
    assert torch.equal(pkg.dense_attn_fwd(q, k, v, **args, out=q), expect)


def test_captured_and_other_stream_calls():
    tensors, args = inputs("256-steps")
    one, out = unsplit(tensors, args), torch.empty_like(tensors[0])
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    pkg.dense_attn_fwd(*tensors, **args, out=out, stream=other.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(out, one)                     # no scratch of its own on a stream torch does not know of
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pkg.dense_attn_fwd(*tensors, **args, out=out)
    prob, chunk = problem("256-steps")
    scratch = torch.empty(binding.dense_attn_workspace_bytes(prob, chunk), dtype=torch.uint8, device="cuda:0")
    split, with_scratch = torch.empty_like(out), torch.cuda.CUDAGraph()
    with torch.cuda.graph(with_scratch):
        pkg.dense_attn_fwd(*tensors, **args, out=split, workspace=scratch)
    for _ in range(3):
        out.zero_(), split.zero_(), scratch.fill_(255)
        graph.replay(), with_scratch.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, one) and torch.equal(split, pkg.dense_attn_fwd(*tensors, **args))


def test_no_memory_for_the_scratch(monkeypatch):
    # (the allocator's refusal is raised by a stand-in: no memory is filled)
    tensors, args = inputs("64")
    one, out = unsplit(tensors, args), torch.empty_like(tensors[0])

    def refuse(*a, **kw):
        raise torch.cuda.OutOfMemoryError("no memory")

    with monkeypatch.context() as patch:
        patch.setattr(torch, "empty", refuse)
        pkg.dense_attn_fwd(*tensors, **args, out=out)
    assert torch.equal(out, one)


def test_which_calls_are_split():
    assert binding.dense_attn_workspace_bytes(*problem("64")) == 816 * 2 * 9 * 130 * 4
    for kw in (dict(dtype=binding.MRT_F32), dict(compute=binding.MRT_COMPUTE_F32)):
        assert binding.dense_attn_workspace_bytes(*problem("64", **kw)) == 0
    small = binding.make_problem(batch=1, heads=1, head_dim=128, f_q=3, f_kv=3, h=8, w=16)
    full = binding.make_problem(batch=1, heads=12, head_dim=128, f_q=3, f_kv=3, h=30, w=52)
    assert binding.dense_attn_workspace_bytes(small) == binding.dense_attn_workspace_bytes(full) == 0
    lib = binding.load_library()
    prob, chunk = problem("64")
    assert lib.dense_attn_workspace_bytes(ctypes.byref(prob), -1) == 0
    (q, k, v), _ = inputs("64")
    assert lib.dense_attn_fwd_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), q.data_ptr(), ctypes.byref(prob), chunk,
                                 q.data_ptr() + 16, 1 << 30, None) == binding.MRT_ERR_WORKSPACE
