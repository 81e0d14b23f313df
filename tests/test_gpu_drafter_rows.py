"""The drafter layer around the token counts where its launches change: K, V
and q in one launch up to 16 tokens, W_o and W_down with their residual in one
kernel up to 11 tokens on layers of at least 256 feature blocks (4096).
Against the fp64 oracle, with the bf16 bar of the other drafter tests."""
import pytest
import torch

import workloads as W
from test_gpu_drafter import _setup, _workload
from test_gpu_drafter import test_forward_matches_oracle as check_forward

pytestmark = pytest.mark.gpu

wf = pytest.importorskip("paper_2606_07710_amd")


@pytest.mark.parametrize("M", [1, 2, 11, 12, 16, 17])
@pytest.mark.parametrize("hidden,nqh,nkvh,hd,inter,pos", [
    (4096, 2, 1, 128, 96, 40),           # exactly 256 feature blocks, short inputs
    (4128, 5, 5, 64, 352, 0),            # more, none a power of two
    (4064, 4, 2, 64, 128, 9),            # 254 blocks: the slices
])
def test_forward_rows(hidden, nqh, nkvh, hd, inter, pos, M):
    check_forward(hidden, nqh, nkvh, hd, inter, pos, M)


# inputs of W_o and W_down of more than one pass of 64 32-dim chunks: whole
# batches of eight chunks a wave, a ragged later batch (305 chunks = 4 passes
# and 49; 65 = one pass and one chunk; 2080 = 65 chunks), and exactly two passes
@pytest.mark.parametrize("M", [2, 8, 11])
@pytest.mark.parametrize("hidden,nqh,nkvh,hd,inter,pos", [
    (4096, 32, 8, 128, 9760, 40),
    (5120, 20, 4, 128, 2080, 0),
    (4096, 65, 5, 64, 4096, 9),
])
def test_forward_long_inputs(hidden, nqh, nkvh, hd, inter, pos, M):
    check_forward(hidden, nqh, nkvh, hd, inter, pos, M)
    # tiled weights: the same sums, bit for bit
    w = _workload(hidden, nqh, nkvh, hd, inter, pos, M, seed_cfg=70 + M + pos)
    t, row, _ = _setup(w)
    tiled = wf.decoder_layer({k: (t[k] if k.endswith("norm") else wf.tile_weights(t[k]))
                              for k in W.DECODER_WEIGHTS}, nqh, nkvh, w.rms_eps, w.rope_base)
    got = []
    for layer in (row, tiled):
        kc, vc = t["k_cache"].clone(), t["v_cache"].clone()
        out = torch.empty((M, hidden), dtype=torch.bfloat16, device="cuda")
        wf.wf_drafter_forward(layer, t["r"], pos, kc, vc, out)
        got.append((out, kc, vc))
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
