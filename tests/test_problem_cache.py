"""The binding's cache of problem descriptors: a call must describe exactly the problem its arguments
state, whatever was called before, refuse what it refused, and the cache stays bounded."""
import numpy as np
import pytest
import torch

from paper_2602_12271_amd import binding


class Tensor:
    """What the binding reads of a tensor (the checks need no device memory)."""

    def __init__(self, shape, dtype=torch.bfloat16, strides=None, is_cuda=True):
        self.shape, self.dtype, self.is_cuda = torch.Size(shape), dtype, is_cuda
        self._s = strides or tuple(int(np.prod(shape[i + 1:])) for i in range(len(shape)))

    def dim(self):
        return len(self.shape)

    def stride(self, i=None):
        return self._s if i is None else self._s[i]


BASE = dict(f_q=1, f_kv=2, h=3, w=4, q_frame_offset=0, scale=1.0, compute=0, assign="fh_w", tile_h=0, head_groups=0)


def tensors(B=1, H=2, d=64, dtype=torch.bfloat16, f_q=1, f_kv=2, h=3, w=4, transposed=False, **_):
    def one(n):
        if transposed:
            return Tensor((B, H, n, d), dtype, (H * n * d, d, H * d, 1))
        return Tensor((B, H, n, d), dtype)
    return one(f_q * h * w), one(f_kv * h * w), one(f_kv * h * w), one(f_q * h * w)


def describe(kw, fresh):
    args = {k: kw[k] for k in BASE}
    f = binding._torch_problem if fresh else binding._call_problem
    return bytes(f(*tensors(**kw), *args.values()))


VARIANTS = [dict(), dict(B=2), dict(H=3), dict(d=128), dict(dtype=torch.float32), dict(transposed=True), dict(f_q=2),
            dict(f_kv=4), dict(h=4), dict(w=5), dict(q_frame_offset=1), dict(scale=0.5), dict(compute=1),
            dict(assign="fw_h"), dict(tile_h=3), dict(head_groups=2), dict(scale=float(np.float32(0.1)))]


def test_every_argument_reaches_the_descriptor():
    binding._problems.clear()
    for _ in range(2):                                   # the second pass is served from the cache
        seen = set()
        for v in VARIANTS:
            kw = dict(BASE, **v)
            assert describe(kw, False) == describe(kw, True)
            seen.add(describe(kw, False))
        assert len(seen) == len(VARIANTS)


@pytest.mark.parametrize("bad", [dict(is_cuda=False), dict(dtype=torch.float32), dict(shape=(1, 2, 25, 64)),
                                 dict(strides=(2 * 24 * 64, 24 * 64, 64, 2))])
def test_refused_tensors_stay_refused_after_a_hit(bad):
    describe(BASE, False)
    q, k, v, o = tensors()
    k = Tensor(bad.get("shape", k.shape), bad.get("dtype", k.dtype), bad.get("strides", k.stride()), bad.get("is_cuda", True))
    with pytest.raises(AssertionError):
        binding._call_problem(q, k, v, o, *BASE.values())


@pytest.mark.parametrize("name,value", [("f_q", 1.0), ("tile_h", 0.0), ("assign", 0.0), ("assign", "w_h"), ("scale", "1")])
def test_refused_arguments_stay_refused_after_a_hit(name, value):
    describe(BASE, False)
    args = dict(BASE, **{name: value})
    with pytest.raises((TypeError, KeyError)):
        binding._torch_problem(*tensors(), *args.values())
    with pytest.raises((TypeError, KeyError)):
        binding._call_problem(*tensors(), *args.values())


def test_bounded():
    for i in range(3 * binding._MAX_PROBLEMS):
        describe(dict(BASE, scale=1.0 + i), False)
    assert len(binding._problems) <= binding._MAX_PROBLEMS
