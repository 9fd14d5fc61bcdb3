"""Which bf16 dense calls split their keys, asked of the library on the host (256 compute units, the ones of the GPU it
is built for, where there is none).  Splitting the first ones, all under a mask, had made them 11 to 29 % longer; the others gain."""
import pytest

from paper_2602_12271_amd import binding


def scratch(d, heads, f_q, f_kv, h, w, chunk, offset):
    prob = binding.make_problem(batch=1, heads=heads, head_dim=d, f_q=f_q, f_kv=f_kv, h=h, w=w, q_frame_offset=offset,
                                scale=d ** -0.5)
    assert binding.dense_attn_check(prob, chunk) == binding.MRT_OK
    return binding.dense_attn_workspace_bytes(prob, chunk)


@pytest.mark.parametrize("call", [
    # unsplit -> split, us
    (128, 15, 6, 12, 15, 36, 3, 6),      # 173 -> 201
    (128, 7, 6, 6, 35, 42, 3, 0),        # 251 -> 279
    (128, 27, 7, 35, 10, 15, 3, 27),     # 94 -> 121
    (128, 7, 4, 12, 12, 45, 1, 8),       # 82 -> 105
    (128, 20, 3, 9, 22, 42, 1, 6),       # 223 -> 257
])
def test_unsplit(call):
    assert scratch(*call) == 0


@pytest.mark.parametrize("call", [
    (128, 2, 3, 12, 16, 17, 3, 9),       # 43.6 -> 19
    (128, 1, 6, 24, 14, 42, 3, 18),      # 165 -> 60
    (128, 3, 4, 16, 41, 35, 1, 12),      # 369 -> 224
    (128, 9, 3, 9, 34, 18, 0, 6),        # 94 -> 67
    (64, 1, 3, 18, 18, 57, 0, 15),       # 135 -> 35
    (64, 2, 5, 25, 25, 50, 0, 0),        # 241 -> 143
    (64, 4, 2, 12, 26, 28, 1, 10),       # 70 -> 34
])
def test_split(call):
    assert scratch(*call) > 0
