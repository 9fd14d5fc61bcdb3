"""Last-iteration stage L for blocks of more than 144 rows (one LDS tile used twice by six waves): the
edges of its query and key tiles, with and without the chunk-causal mask, against the fp64 oracle.
Bar: 2-norm, four times the 3.7e-3 the bf16 roundings of the forward pass show."""
import pytest

from oracle import monarch_oracle as mo  # noqa: F401  (the oracle the harness compares with)
from workloads import synthetic as syn

from gpu_harness import oracle_monarch_head, run_monarch_gpu, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("f,h,chunk", [(5, 29, 0), (1, 160, 0), (7, 23, 0), (2, 88, 0), (3, 59, 1), (2, 96, 0), (4, 48, 2)])
def test_forward(f, h, chunk, d):
    wl = syn.Workload("wide", 1, 2, d, f, f, h, 9, f * h, 9, 0, 2, chunk, 0, "bf16", d ** -0.5, True)
    arrays = syn.make_inputs(wl)
    print(f"case {wl}", flush=True)
    out = run_monarch_gpu(wl, *to_device(wl, arrays))
    num = den = 0.0
    for hd in range(wl.heads):
        ref = oracle_monarch_head(wl, *(x[0, hd] for x in arrays))
        num += (out[0, hd].double().cpu() - ref).pow(2).sum().item()
        den += ref.pow(2).sum().item()
    assert (num / den) ** 0.5 <= 1.5e-2
