"""GPU parity of the LM head's kernels that stream W through LDS, against the
fp64 oracle, at their edges: ragged last vocabulary block and last sub-tile
of a run, one to five sub-tiles, every row-group count, hidden sizes of one
half step (32), half a step over (96) and no multiple of 512 (any of them
without a tiled form); and, where a tiled form exists, the same bits."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from parity import check_argmax, entropy_rel_err

pytestmark = pytest.mark.gpu

wf = pytest.importorskip("paper_2606_07710_amd")
DEV = "cuda"


def _run(h, w):
    g = h.shape[0]
    am = torch.empty(g, dtype=torch.int32, device=DEV)
    ent = torch.empty(g, dtype=torch.float32, device=DEV)
    acc = torch.empty(3, dtype=torch.int32, device=DEV)
    draft = torch.zeros(max(g - 1, 1), dtype=torch.int32, device=DEV)
    wf.wf_lmhead_accept_entropy(h, w, None, draft, 1.0, am, ent, acc)
    torch.cuda.synchronize()
    return am, ent, acc


CASES = [
    # gamma, d, vocab
    (1, 32, 17), (64, 32, 40000), (5, 96, 1000), (16, 96, 32769), (17, 160, 33000),
    (33, 2080, 1025), (48, 96, 70001), (61, 288, 32768),          # any hidden size
    (1, 512, 1), (16, 512, 129), (20, 512, 33000), (33, 512, 65537), (61, 1024, 70001),
    (64, 512, 163841), (49, 512, 4096), (32, 512, 34000),         # multiples of 512
]


@pytest.mark.parametrize("gamma,d,vocab", CASES)
def test_matches_oracle(gamma, d, vocab):
    print(f"lmhead rows gamma={gamma} d={d} vocab={vocab}", flush=True)
    h = W.normal((gamma, d), 1.0, 1 + vocab, torch.bfloat16, DEV)
    w = W.normal((vocab, d), 0.05, 2 + vocab, torch.bfloat16, DEV)
    am, ent, acc = _run(h, w)
    am_ref, ent_ref, margin, z = oracle.lmhead_rows(W.to_oracle(h), W.to_oracle(w),
                                                    want_logits=True)
    check_argmax(am.cpu().numpy(), am_ref, margin, z, "bf16")
    # fp32 sums of up to 2080 products and of the row states: a few hundred
    # roundings of 6e-8, none of them correlated
    assert entropy_rel_err(ent.cpu().numpy(), ent_ref) <= 1e-5
    if d % 512 == 0:
        for a, b in zip(_run(h, wf.tile_weights(w)), (am, ent, acc)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("gamma,d", [(7, 160), (40, 512)])
def test_masked_and_infinite_logits(gamma, d):
    """An infinite weight row gives that row's logits +inf, -inf or NaN-free
    sums as the definition has them: rows whose logit is -inf count nothing."""
    vocab = 900
    h = W.normal((gamma, d), 1.0, 5, torch.bfloat16, DEV).abs() + 0.01
    w = W.normal((vocab, d), 0.05, 6, torch.bfloat16, DEV)
    w[3] = float("-inf")
    w[899] = float("-inf")
    am, ent, _ = _run(h, w)
    keep = [v for v in range(vocab) if v not in (3, 899)]
    am_ref, ent_ref, margin, z = oracle.lmhead_rows(W.to_oracle(h),
                                                    W.to_oracle(w[keep].contiguous()),
                                                    want_logits=True)
    got = np.array([keep.index(int(a)) for a in am.cpu()])
    check_argmax(got, am_ref, margin, z, "bf16")
    assert entropy_rel_err(ent.cpu().numpy(), ent_ref) <= 1e-5


@pytest.mark.parametrize("gamma,d,vocab,tiled", [
    (64, (1 << 25) + (1 << 22), 20, False),     # 64 rows of h span more than 4 GB
    (64, (1 << 25) + (1 << 22), 20, True),
    (2, 150000000, 16, False),                  # a 16-row block of W does
    (2, 150000000, 5, False),
    (17, 320000000, 16, False),                 # eight rows do
    (17, 320000000, 16, True),
    (9, 320000032, 14, False),
])
def test_rows_more_than_4gb_apart(gamma, d, vocab, tiled):
    """Byte offsets past 32 bits, with inputs that are zero but for a few
    whole numbers, so that every logit is exact in any order of sums."""
    print(f"lmhead far rows gamma={gamma} d={d} vocab={vocab} tiled={tiled}", flush=True)
    gen = torch.Generator().manual_seed(d)
    cols = torch.tensor([0, 31, 515, d // 2 + 7, d - 33, d - 1])
    hs = torch.randint(-3, 4, (gamma, len(cols)), generator=gen).double()
    ws = torch.randint(-3, 4, (vocab, len(cols)), generator=gen).double()
    h = torch.zeros(gamma, d, dtype=torch.bfloat16, device=DEV)
    w = torch.zeros(vocab, d, dtype=torch.bfloat16, device=DEV)
    h[:, cols.to(DEV)] = hs.to(DEV, torch.bfloat16)
    w[:, cols.to(DEV)] = ws.to(DEV, torch.bfloat16)
    am, ent, _ = _run(h, wf.tile_weights(w) if tiled else w)
    z = hs @ ws.t()
    # equal logits: the lowest index
    assert torch.equal(am.cpu(), (z == z.amax(1, keepdim=True)).int().argmax(1).int())
    lp = torch.log_softmax(z, 1)
    assert entropy_rel_err(ent.cpu().numpy(), (-(lp.exp() * lp).sum(1)).numpy()) <= 1e-5
