"""GPU parity of the KV-only prefill's LDS-tiled kernel (many tokens, many
layers) against the fp64 oracle at the edges of its tiles: the token counts
where the tile changes, ragged last token and feature blocks, input
dimensions that end in half a 64-dim step, row-major and tiled weights,
head_dim 64, and the tiled rows a long drafter catch-up hands it."""
import pytest
import torch

import oracle
import workloads as W
from parity import TOL, host64, max_vec_rel_err

pytestmark = pytest.mark.gpu

wf = pytest.importorskip("paper_2606_07710_amd")
DEV = "cuda"
BF = torch.bfloat16


def _check(L, n, d, hkv, dh, start, tiled, check):
    print(f"prefill gemm L={L} n={n} d={d} hkv={hkv} dh={dh} tiled={tiled}", flush=True)
    cap = start + n + 2
    x = W.normal((L, n, d), 1.0, 11, BF, DEV)
    wk = W.normal((L, hkv * dh, d), 0.02, 12, BF, DEV)
    wv = W.normal((L, hkv * dh, d), 0.02, 13, BF, DEV)
    kc = W.normal((L, hkv, cap, dh), 1.0, 14, BF, DEV)
    vc = W.normal((L, hkv, cap, dh), 1.0, 15, BF, DEV)
    k0, v0 = kc.clone(), vc.clone()
    a, b = (wf.tile_weights(wk), wf.tile_weights(wv)) if tiled else (wk, wv)
    wf.wf_kv_only_prefill_layers(x, a, b, kc, vc, start, 1e6)
    torch.cuda.synchronize()
    rows = slice(start, start + n)
    for l in check:
        kr, vr = oracle.kv_only_prefill(W.to_oracle(x[l]), W.to_oracle(wk[l]),
                                        W.to_oracle(wv[l]), start, hkv, dh, 1e6)
        # bf16 results of fp32 sums: half an ulp (2^-9) of each element, well
        # inside the bar of the parity tests
        assert max_vec_rel_err(host64(kc[l][:, rows]), kr) <= TOL["bf16"] / 4
        assert max_vec_rel_err(host64(vc[l][:, rows]), vr) <= TOL["bf16"] / 4
    for got, old in ((kc, k0), (vc, v0)):
        assert torch.equal(got[:, :, :start], old[:, :, :start])
        assert torch.equal(got[:, :, start + n:], old[:, :, start + n:])


# one layer: n around the lines where the tile changes (256 workgroups), the
# last token block ragged; d ends in half a step where d % 64 == 32
ONE = [
    # n, d, hkv, dh, tiled
    (81, 64, 8, 128, False), (81, 96, 8, 128, True), (256, 160, 8, 128, False),
    (257, 128, 8, 128, True), (513, 96, 8, 128, False), (1025, 96, 8, 128, True),
    (1030, 64, 8, 128, False), (2049, 96, 8, 128, False), (4096, 64, 8, 128, True),
    (130, 224, 3, 64, False), (700, 96, 1, 64, True), (1300, 1056, 5, 64, False),
]


@pytest.mark.parametrize("n,d,hkv,dh,tiled", ONE)
def test_one_layer(n, d, hkv, dh, tiled):
    _check(1, n, d, hkv, dh, 70001, tiled, (0,))


# more tokens, but few heads and long inputs: the kernel that splits the input
# dimension takes them back.  Both sides of that line, for one layer (units of
# two pairs, three and four token blocks) and for two to four
FEW_HEADS = [
    # layers, n, d, hkv, dh, tiled, layers checked
    (1, 81, 4096, 2, 128, True, (0,)), (1, 97, 4096, 2, 128, False, (0,)),
    (1, 160, 4096, 1, 128, True, (0,)), (1, 161, 4096, 1, 128, True, (0,)),
    (1, 301, 4096, 1, 128, True, (0,)), (1, 200, 8192, 2, 64, True, (0,)),
    (1, 175, 8192, 2, 64, False, (0,)), (1, 640, 4096, 1, 128, True, (0,)),
    (2, 65, 4096, 1, 128, False, (1,)), (3, 80, 4096, 1, 64, True, (0, 2)),
    (4, 129, 4096, 1, 64, True, (3,)), (2, 250, 4096, 1, 128, True, (1,)),
    (2, 65, 512, 1, 128, True, (1,)),
]


@pytest.mark.parametrize("L,n,d,hkv,dh,tiled,check", FEW_HEADS)
def test_few_heads(L, n, d, hkv, dh, tiled, check):
    _check(L, n, d, hkv, dh, 500, tiled, check)


# many layers: every token-block count of the streaming tiles, the lines at
# 384, 512, 1024 and 2048 units of 32 features, and two token blocks
MANY = [
    # layers, n, d, hkv, dh, tiled, layers checked
    (8, 1, 96, 8, 128, False, (0, 7)), (16, 16, 64, 8, 128, True, (3, 15)),
    (6, 17, 96, 8, 128, True, (0, 5)), (16, 32, 64, 8, 128, False, (15,)),
    (6, 40, 160, 8, 128, False, (5,)), (8, 64, 96, 8, 128, True, (7,)),
    (32, 64, 64, 8, 128, False, (31,)), (16, 65, 96, 8, 128, False, (15,)),
    (36, 80, 96, 8, 128, True, (35,)), (20, 96, 64, 8, 128, True, (19,)),
    (33, 100, 96, 8, 128, False, (32,)), (8, 128, 96, 8, 128, False, (7,)),
    (40, 128, 64, 8, 128, True, (39,)), (37, 33, 96, 5, 64, False, (36,)),
    (75, 120, 96, 3, 64, True, (74,)), (36, 129, 96, 8, 128, False, (35,)),
    (3, 200, 96, 8, 128, True, (2,)),
    # one token block around the unit counts of short tiled inputs and of four stages
    (16, 16, 1056, 8, 64, True, (15,)), (20, 16, 1056, 8, 64, True, (0, 19)),
    (24, 9, 96, 8, 128, False, (23,)), (25, 9, 96, 8, 128, False, (24,)),
    (24, 16, 2080, 8, 128, True, (23,)), (25, 3, 2080, 8, 128, True, (24,)),
]


@pytest.mark.parametrize("L,n,d,hkv,dh,tiled,check", MANY)
def test_many_layers(L, n, d, hkv, dh, tiled, check):
    _check(L, n, d, hkv, dh, 1000, tiled, check)


@pytest.mark.parametrize("n", [768, 769, 850])
def test_catchup_hands_over_tiled_rows(n):
    """A drafter catch-up around the backlog from which its K/V run in the
    LDS-tiled kernel, reading the RMSNorm launch's tiled rows."""
    _check_catchup(n, 288, False)


@pytest.mark.parametrize("n,hid,tiled", [(512, 288, False), (513, 288, False), (768, 288, True),
                                         (769, 288, True), (1024, 2048, True),
                                         (1025, 2048, True)])
def test_catchup_changes_over(n, hid, tiled):
    """The backlogs at which the launches change, per weight layout and width."""
    _check_catchup(n, hid, tiled)


def _check_catchup(n, hid, tiled):
    print(f"catch-up n={n} hidden={hid} tiled={tiled}", flush=True)
    hq, hkv, dh, inter, pos = 4, 2, 64, 320, 9
    shapes = {"attn_norm": (hid,), "w_q": (hq * dh, hid), "w_k": (hkv * dh, hid),
              "w_v": (hkv * dh, hid), "w_o": (hid, hq * dh), "mlp_norm": (hid,),
              "w_gate": (inter, hid), "w_up": (inter, hid), "w_down": (hid, inter)}
    w = {k: W.normal(s, 0.05, 30 + i, BF, DEV) + (1 if k.endswith("norm") else 0)
         for i, (k, s) in enumerate(shapes.items())}
    r = W.normal((n, hid), 1.0, 50, BF, DEV)
    kc = W.normal((hkv, pos + n + 1, dh), 1.0, 51, BF, DEV)
    vc = W.normal((hkv, pos + n + 1, dh), 1.0, 52, BF, DEV)
    kh, vh = W.to_oracle(kc), W.to_oracle(vc)
    out = torch.empty(hid, dtype=BF, device=DEV)
    given = {k: v if k.endswith("norm") or not tiled else wf.tile_weights(v) for k, v in w.items()}
    wf.wf_drafter_catchup(wf.decoder_layer(given, hq, hkv, 1e-6, 1e6), r, pos, kc, vc, out)
    torch.cuda.synchronize()
    ref, kref, vref = oracle.catchup(W.to_oracle(r), pos, {k: W.to_oracle(v) for k, v in w.items()},
                                     kh, vh, hq, hkv, 1e-6, 1e6)
    rows = slice(pos, pos + n)
    assert max_vec_rel_err(host64(kc[:, rows]), kref[:, rows]) <= TOL["bf16"]
    assert max_vec_rel_err(host64(vc[:, rows]), vref[:, rows]) <= TOL["bf16"]
    assert max_vec_rel_err(host64(out)[None], ref[None]) <= TOL["bf16"]
