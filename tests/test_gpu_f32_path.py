"""The fp32 verify kernels where their tiling can go wrong: one pass and two of
8 verify rows, more rows, and hidden sizes that are, and are not, a multiple of the four
floats a load takes (LM head); whole and ragged 64-key blocks, one and several
a split (attention).  Against the fp64 oracle; the tolerance is the fp32 bar of
the other kernel tests (1e-4 entropy, attention 1e-5: a few hundred fp32
roundings of 6e-8 in random order)."""
import pytest
import torch


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma", [1, 4, 5, 8, 9, 16, 17, 64])
@pytest.mark.parametrize("d,vocab", [(512, 64), (260, 131), (255, 200), (1, 65), (1028, 70)])
def test_lmhead_f32(gamma, d, vocab):
    import paper_2606_07710_amd as wf
    gen = torch.Generator().manual_seed(1000 * gamma + d)
    h = torch.randn(gamma, d, generator=gen)
    w = torch.randn(vocab, d, generator=gen) * 0.3
    z = h.double() @ w.double().t()
    top = z.topk(2, dim=1).values
    logp = torch.log_softmax(z, -1)
    ent = -(logp.exp() * logp).sum(-1)
    argmax = torch.full((gamma,), -1, dtype=torch.int32, device="cuda")
    entropy = torch.zeros(gamma, device="cuda")
    accept = torch.zeros(4, dtype=torch.int32, device="cuda")
    draft = z.argmax(1)[: gamma - 1].to(torch.int32).cuda() if gamma > 1 else None
    wf.wf_lmhead_accept_entropy(h.cuda(), w.cuda(), None, draft, 1.0, argmax, entropy, accept)
    torch.cuda.synchronize()
    clear = (top[:, 0] - top[:, 1]) > 1e-4
    assert torch.equal(argmax.cpu()[clear], z.argmax(1).to(torch.int32)[clear])
    err = ((entropy.cpu().double() - ent).abs() / ent.abs().clamp(min=1e-3)).max()
    assert err <= 1e-4, float(err)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("gamma,ctx,splits", [(1, 0, 0), (1, 63, 0), (1, 64, 1), (8, 55, 0),
                                              (8, 56, 0), (8, 57, 1), (5, 250, 2), (16, 1000, 3),
                                              (64, 500, 8)])
def test_attention_f32(gamma, ctx, splits, dh):
    import paper_2606_07710_amd as wf
    hq, hkv = 4, 2
    gen = torch.Generator().manual_seed(gamma + 100 * ctx + dh)
    q = torch.randn(gamma, hq, dh, generator=gen)
    cap = ctx + gamma + 3
    k = torch.randn(hkv, cap, dh, generator=gen)
    v = torch.randn(hkv, cap, dh, generator=gen)
    k[:, ctx + gamma:] = float("nan")          # rows past the block are never used
    v[:, ctx + gamma:] = float("nan")
    n = ctx + gamma
    see = torch.arange(n)[None, :] <= ctx + torch.arange(gamma)[:, None]
    ref = torch.empty(gamma, hq, dh, dtype=torch.float64)
    for h in range(hq):
        z = q[:, h].double() @ k[h // 2, :n].double().t() / dh ** 0.5
        ref[:, h] = torch.softmax(z.masked_fill(~see, -torch.inf), -1) @ v[h // 2, :n].double()
    out = torch.empty(gamma, hq, dh, device="cuda")
    wf.wf_verify_attn(q.cuda(), k.cuda(), v.cuda(), out, ctx, num_splits=splits)
    err = ((out.cpu().double() - ref).abs().amax(-1) / ref.abs().amax(-1)).max()
    assert err <= 1e-5, float(err)
