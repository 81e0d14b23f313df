"""What the Python layer itself refuses, on the CPU: stand-ins for device
tensors whose pointers the C side refuses (not 16-byte aligned), so no call
ever reaches the GPU."""
import ctypes
import os
import subprocess
import sys

import pytest
import torch

wf = pytest.importorskip("paper_2606_07710_amd")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class FakeTensor:
    is_cuda, device = True, "cuda"

    def __init__(self, *shape, dtype=torch.bfloat16):
        self.shape, self.dtype = torch.Size(shape), dtype

    def data_ptr(self):
        return 8

    def is_contiguous(self):
        return True

    def numel(self):
        return self.shape.numel()

    def element_size(self):
        return 8 if self.dtype == torch.int64 else 2


class FakeStream:
    cuda_stream = 0


def _attend(tree, ctx_len, num_splits=0):
    q, k = FakeTensor(4, 8, 128), FakeTensor(2, 64, 128)
    ws = FakeTensor(64 << 20, dtype=torch.uint8)
    if tree:
        return wf.wf_verify_attn_tree(q, k, k, q, ctx_len, FakeTensor(4, dtype=torch.int64),
                                      num_splits=num_splits, workspace=ws, stream=FakeStream)
    return wf.wf_verify_attn(q, k, k, q, ctx_len, num_splits=num_splits, workspace=ws,
                             stream=FakeStream)


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("ctx_len,num_splits", [(5.7, 0), ("5", 0), (5, 1.5)])
def test_attention_takes_whole_numbers_only(tree, ctx_len, num_splits):
    """A context length that is no integer is refused whether or not the
    caller brings a workspace, and never rounded."""
    with pytest.raises((ctypes.ArgumentError, TypeError)):
        _attend(tree, ctx_len, num_splits)


@pytest.mark.parametrize("tree", [False, True])
def test_attention_reaches_the_library(tree):
    with pytest.raises(wf.WfError) as e:
        _attend(tree, 5)
    assert e.value.status == wf.WF_ERR_INVALID_ARG


@pytest.mark.parametrize("missing", ["attn_norm", "w_v", "w_down"])
def test_a_decoder_layer_needs_every_weight(missing):
    w = {n: FakeTensor(*((256,) if n.endswith("norm") else (256, 256)))
         for n in wf.DECODER_WEIGHTS}
    assert wf.decoder_layer(w, 2, 2, 1e-6, 1e4).hidden == 256
    w[missing] = None
    with pytest.raises((ValueError, AttributeError)):
        wf.decoder_layer(w, 2, 2, 1e-6, 1e4)


def test_import_without_torch_private_functions():
    """A torch without the two private stream getters: the package imports and
    takes the stream from torch.cuda.current_stream()."""
    code = """
import torch
for n in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
    if hasattr(torch._C, n):
        delattr(torch._C, n)
import paper_2606_07710_amd as wf
class S: cuda_stream = 77
torch.cuda.current_stream = lambda: S
assert wf._stream(None) == 77
"""
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT, timeout=300)
