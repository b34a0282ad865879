"""dK and dV of key tiles whose row list is divided into parts (few groups,
long lists), next to tiles that are not, against the fp64 oracle.  A part is
whole chunks of 64 rows; at these sizes, with scratch for every part, it holds
at most 4 of them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_13141_amd import configs, inputs, sas

from helpers import assert_close, f64

pytestmark = pytest.mark.gpu

#        n    H Hkv dh   B   K  mode
CASES = [(900, 3, 1, 128, 64, 8, "gated"), (700, 2, 1, 64, 16, 12, "gated"), (769, 2, 2, 64, 128, 2, "sparse")]


@pytest.mark.parametrize("n,H,Hkv,dh,B,K,mode", CASES)
def test_divided_row_lists(n, H, Hkv, dh, B, K, mode):
    print(f"\n[case] backward parts n={n} H={H}/{Hkv} dh={dh} B={B} K={K} {mode}", flush=True)
    w = configs.L7B_1K.with_(seq_len=n, n_heads=H, n_kv_heads=Hkv, head_dim=dh, block_size=B, top_k=K, mode=mode,
                             segments=(("txt", n),), index=112)
    q, k, v = inputs.qkv(w)
    d_o = inputs.normal(w, "d_o", q.shape, 1.0)
    cfg = sas.make_config(w)
    dev = [sas.to_device(a, "bf16") for a in (q, k, v, d_o)]
    fw = sas.attention_prefill(cfg, *dev[:3], log_gate=True)
    bw = [sas.attention_backward(cfg, *dev[:3], fw["o"], dev[3], fw["lse"], fw["sel_idx"], fw["log_gate"])
          for _ in range(2)]
    st = oracle.select(f64(q[0]), f64(k[0]), B, K, "bf16")
    # the lists of 64-key tiles: own rows and every later row that selected one of the tile's blocks
    longest = 0
    for g in range(Hkv):
        for j in range(-(-n // 64)):
            m = set(range(64 * j // B, min(n - 1, 64 * j + 63) // B + 1))
            longest = max(longest, sum(t >= 64 * j and (t // B in m or bool(m & set(st["sel"][g, t].tolist())))
                                       for t in range(n)))
    assert longest > 4 * 64, longest
    dQ, dK, dV, _ = oracle.sas_attention_backward(f64(q[0]), f64(k[0]), f64(v[0]), f64(d_o[0]), B, mode, st["sel"],
                                                  st["log_gate"])
    assert_close(bw[0]["dq"][0].float().cpu().numpy(), dQ, "bf16", "dQ")
    assert_close(bw[0]["dk"][0].float().cpu().numpy(), dK, "bf16", "dK")
    assert_close(bw[0]["dv"][0].float().cpu().numpy(), dV, "bf16", "dV")
    for f in ("dk", "dv"):  # the parts are added in a fixed order
        assert torch.equal(bw[0][f], bw[1][f])
