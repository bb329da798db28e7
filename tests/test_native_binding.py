"""The native part of the Python binding refuses what the calls refuse, before anything reaches a GPU (no GPU needed)."""
import pytest
import torch

import paper_2210_00129_amd as sbp


def test_arguments_are_checked_before_the_call():
    W = torch.zeros(8, 4)
    dY, idx = torch.zeros(6, 8), torch.zeros(3, dtype=torch.int32)
    with pytest.raises(ValueError, match="M is required when dY is compact"):
        sbp.backward_linear(dY, idx, dY, W, flags=sbp.FLAG_DY_COMPACT)
    with pytest.raises(ValueError, match="dW must be bfloat16"):
        sbp.backward_linear(dY, idx, dY, W, dW=torch.zeros(8, 4), flags=sbp.FLAG_DW_OUT_BF16)
    with pytest.raises(TypeError, match="unsupported dtype"):
        sbp.backward_linear(dY, idx, dY, W.double())
    with pytest.raises(ValueError, match="GPU memory"):
        sbp.backward_linear(dY, idx, dY, W)
    with pytest.raises(ValueError):
        sbp.backward_linear(dY, idx, dY, torch.zeros(8, 4, 1))
    with pytest.raises(TypeError):
        sbp.backward_linear(dY, idx, dY, W, M=6.5)
    with pytest.raises(ValueError, match=r"\[M, C\]"):
        sbp.forward_cache(torch.zeros(5), idx)
    with pytest.raises(ValueError, match="GPU memory"):
        sbp.forward_cache(dY, idx)
    with pytest.raises(TypeError):
        sbp.forward_cache(dY, None)


def test_sizes_of_a_draw_are_checked_first():
    with pytest.raises(sbp.SbpError):
        sbp.sample_indices(2, 0, 4, 4, 9, 1, 1, device="cpu")
    with pytest.raises(sbp.SbpError):
        sbp.sample_indices(2, 0, 4, 4, 9, 1, 1)
    with pytest.raises(ValueError, match="GPU memory"):
        sbp.sample_indices(2, 0, 4, 4, 2, 1, 1, device="cpu")
    with pytest.raises(ValueError, match="GPU memory"):
        sbp.sample_indices(2, 0, 4, 4, 2, 2**64 - 1, -1, idx_out=torch.zeros(16, dtype=torch.int32))


def test_first_allocation_on_a_gpu_initializes_torch(monkeypatch):
    # what torch.empty does before it allocates: without it the fork check is missing (here the check's own error, as in a child
    # forked from a process that has used the GPU)
    if torch.cuda.is_initialized():
        pytest.skip("this process has used the GPU")

    def refuse():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    monkeypatch.setattr(torch.cuda, "_lazy_init", refuse)
    with pytest.raises(RuntimeError, match="forked subprocess"):
        sbp.sample_indices(2, 0, 4, 4, 2, 1, 1)


def test_flags_are_whole_numbers_and_dtypes_are_named_as_torch_names_them():
    W, dY, idx = torch.zeros(8, 4), torch.zeros(6, 8), torch.zeros(3, dtype=torch.int32)
    with pytest.raises(TypeError):
        sbp.backward_linear(dY, idx, dY, W, flags=1.5)
    with pytest.raises(TypeError, match=r"unsupported dtype torch\.float64; use float32 or bfloat16"):
        sbp.backward_linear(dY, idx, dY, W.double())

    class Neither:
        def __bool__(self):
            raise KeyError("neither")
    with pytest.raises(KeyError):
        sbp.sample_indices(2, 0, 4, 4, 2, 1, 1, want_inv=Neither(), idx_out=torch.zeros(16, dtype=torch.int32))
