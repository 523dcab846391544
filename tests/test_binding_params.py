"""The packed parameter structure holds what field-by-field assignment stores, in range and out of it."""
import ctypes

import pytest
import torch

from paper_2602_21233_amd import binding


@pytest.mark.parametrize("change", [{}, dict(softmax_scale=None), dict(q=None, out=None), dict(top_k_blocks=2 ** 33 + 5),
                                    dict(kv_prefix_len=-1), dict(softmax_scale=1e300), dict(lists_per_kv_head=True)])
def test_packed_params_equal_assigned_fields(change):
    q = torch.empty((2, 640, 4, 128), dtype=torch.bfloat16).transpose(1, 2)
    kw = dict(batch=2, n_q_heads=4, n_kv_heads=2, seq_len=640, head_dim=128, block_size=64, n_sink_blocks=1, n_local_blocks=2,
              top_k_blocks=3, softmax_scale=0.3, q=q, k=q[:, :2], v=q[:, 2:], out=q, stride_blocks=5, n_dense_q_blocks=6,
              stride_reach_blocks=7, lists_per_kv_head=0, kv_prefix_len=128)
    kw.update(change)
    got = binding.make_params(**kw)
    want = binding.SpaParams()
    for name in ("batch", "n_q_heads", "n_kv_heads", "seq_len", "head_dim", "block_size", "n_sink_blocks", "n_local_blocks",
                 "top_k_blocks", "stride_blocks", "n_dense_q_blocks", "stride_reach_blocks", "kv_prefix_len"):
        setattr(want, name, kw[name])
    want.lists_per_kv_head = int(kw["lists_per_kv_head"])
    want.softmax_scale = kw["softmax_scale"] or 0.0
    for field, t in (("q_stride", kw["q"]), ("k_stride", kw["k"]), ("v_stride", kw["v"]), ("o_stride", kw["out"])):
        setattr(want, field, (ctypes.c_int64 * 3)(*(t.stride()[:3] if t is not None else (0, 0, 0))))
    assert bytes(got) == bytes(want)


def test_a_head_dim_axis_that_is_not_contiguous_is_refused():
    q = torch.empty((1, 2, 128, 64), dtype=torch.bfloat16).transpose(2, 3)
    with pytest.raises(AssertionError):
        binding._params_from(q, q, 64, 1, 1, 1, None)


def test_the_stream_of_a_cpu_tensor_is_refused_by_torch(monkeypatch):
    """Lists on the CPU, say: torch.cuda.current_stream names what is wrong, the raw call only says "invalid argument"."""
    def current_stream(device=None):
        raise ValueError(f"Expected a cuda device, but got: {device}")
    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    with pytest.raises(ValueError, match="Expected a cuda device, but got: cpu"):
        binding._stream(torch.empty(1, dtype=torch.int32))
